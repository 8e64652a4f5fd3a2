"""GPU parity of the attention kernels at the edges of the rules that pick one.

One sequence of 33 to 64 query rows per KV head takes the register path with two row waves up to
20 KV tiles per CU (of 256) over the heads, and the streaming kernel in four key groups above;
batches take the streaming kernel, in two key groups for 128-column heads and, up to 12 tiles per
CU, for 64-column ones, else in four.  Where one split holds a sequence (short caches, more than 64
sequences) the register path writes its outputs without a merge.

Tolerance: that of the streaming kernel's other cases (2^-18 max|V| for the two-part
probabilities, 2e-6 for the float32 sums and the exponential).
"""
import numpy as np
import pytest

import respec_synth as synth
import workload

from test_gpu_parity import check_x, rt, _depth  # noqa: F401 (rt is a fixture)
from test_gpu_stream_attention import _rows_in_use, _tree

pytestmark = pytest.mark.gpu

CASES = {
    # name: (Hq, Hkv, D, nodes per sequence, prefix lengths[, dtype])
    # one split per sequence: the attention kernel writes x itself (one or four key-group waves,
    # one and two 16-row blocks, more rows than a workgroup holds)
    "direct-one-node": (4, 4, 64, [1], [0]),
    "direct-short": (2, 2, 128, [26], [37]),
    "direct-grouped": (12, 4, 64, [9], [70]),
    "direct-batch": (4, 4, 128, [1 + k % 12 for k in range(70)], [(53 * k) % 300 for k in range(70)]),
    "direct-batch-d64": (8, 8, 64, [16 - k % 16 for k in range(65)], [(31 * k) % 200 for k in range(65)]),
    "direct-f32": (4, 2, 64, [30], [60], "f32"),
    "direct-f32-two-blocks": (4, 1, 64, [61], [20], "f32"),
    "direct-f32-batch": (4, 4, 128, [1 + k % 9 for k in range(66)], [(41 * k) % 90 for k in range(66)], "f32"),
    "one-33-rows": (2, 2, 128, [33], [1]),
    "one-64-rows": (2, 2, 128, [64], [1023]),
    "one-63-rows-grouped": (18, 2, 128, [7], [320]),
    "one-48-rows-d64": (8, 2, 64, [12], [0]),
    "one-at-20-tiles": (64, 64, 64, [34], [80 * 32 - 34]),
    "one-past-20-tiles": (64, 64, 64, [34], [80 * 32 - 33]),
    "one-long-d128": (32, 32, 128, [40], [5300]),
    "batch-two-groups": (4, 2, 128, [17, 32, 1, 5], [70, 2000, 0, 31]),
    "batch-two-groups-d64": (4, 2, 64, [17, 1, 32, 5, 9], [2000, 0, 31, 32, 650]),
    "batch-four-groups-d64": (32, 32, 64, [34, 5, 60, 1], [700, 0, 31, 90]),
}


@pytest.mark.timeout(300)
@pytest.mark.parametrize("name", list(CASES))
def test_attention_routes(rt, name):  # noqa: F811
    hq, hkv, d, nodes, kv, dtype = (*CASES[name], "bf16")[:6]
    parents = [_tree(n, 2 + i % 3) for i, n in enumerate(nodes)]
    big, far = int(np.argmax(nodes)), int(np.argmax(kv))
    parents[big], parents[far] = parents[far], parents[big]
    depth = max(8, max(_depth(p) for p in parents))
    shp = synth.Shape("edge", dtype, hq * d, hq, hkv, d, 520, len(nodes), max(nodes), depth, 8)
    w = synth.custom(shp, parents, kv, seed=613, poison_tail=True)
    print(f"[routes {name}] building", flush=True)
    case = workload.finish(w)
    print(f"[routes {name}] running GPU step", flush=True)
    from paper_2511_01282_amd import binding
    out = rt.run(case.w, x_out=True, stop_after=binding.STOP_ATTN)
    v = _rows_in_use(case.w)
    v = synth.bf16_bits_to_f32(v) if dtype == "bf16" else v
    atol = 2.0 ** -18 * float(np.abs(v).max()) + 2e-6
    err = np.abs(out["attn_out"] - case.attn).max()
    print(f"[routes {name}] max|dO| = {err:.3e} (at most {atol:.3e})", flush=True)
    assert err <= atol
    check_x(case, out["x_out"], f"routes {name}")
