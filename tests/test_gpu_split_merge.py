"""GPU parity of the split merge on both sides of its two forms.

Up to 16 splits of a row are added up by one thread per (row, 4 columns), more by four waves that
share them.  The cases have 16, 17, 33 and up to 64 splits, of every kind: splits of one sequence
(register path), pieces of a batch on the register path, and pieces of the streaming kernel for
one sequence (whose count the merge works out by itself) and for a batch, and a plan larger than
the step.

Tolerance: that of the attention kernels' other cases (2^-18 max|V| for the two-part
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
    # name: (Hq, Hkv, D, nodes per sequence, prefix lengths, dtype, plan's nodes, path)
    "16-splits": (2, 2, 128, [5], [16 * 128 - 5], "bf16", 5, "split"),
    "17-splits": (2, 2, 128, [5], [16 * 128 - 4], "bf16", 5, "split"),
    "33-splits-d64": (4, 4, 64, [13], [33 * 128 - 13], "bf16", 61, "split"),
    "17-splits-f32": (4, 4, 64, [16], [16 * 128 - 15], "f32", 16, "split"),
    "33-splits-f32-d128": (4, 2, 128, [20], [1100], "f32", 61, "split"),
    "pieces-of-a-batch": (4, 2, 64, [9, 3], [31000, 700], "f32", 9, "flat"),
    "stream-16": (4, 1, 128, [40], [32 * 32 - 40], "bf16", 40, "stream"),
    "stream-17": (4, 1, 128, [40], [34 * 32 - 40], "bf16", 40, "stream"),
    "stream-64-larger-plan": (28, 4, 64, [17], [64 * 64 - 17], "bf16", 100, "stream"),
    "stream-of-a-batch": (4, 1, 128, [33, 40], [900, 2500], "bf16", 40, "stream"),
}


@pytest.mark.timeout(300)
@pytest.mark.parametrize("name", list(CASES))
def test_split_merge(rt, name):  # noqa: F811
    hq, hkv, d, nodes, kv, dtype, plan_nodes, _ = CASES[name]
    parents = [_tree(n, 2 + i % 3) for i, n in enumerate(nodes)]
    depth = max(8, max(_depth(p) for p in parents))
    shp = synth.Shape("edge", dtype, hq * d, hq, hkv, d, 520, len(nodes), max(nodes), depth, 8)
    w = synth.custom(shp, parents, kv, seed=617, poison_tail=True)
    print(f"[merge {name}] building", flush=True)
    case = workload.finish(w)
    print(f"[merge {name}] running GPU step", flush=True)
    from paper_2511_01282_amd import binding
    out = rt.run(case.w, plan=rt.make_plan(case.w, max_nodes=plan_nodes), x_out=True, stop_after=binding.STOP_ATTN)
    v = _rows_in_use(case.w)
    v = synth.bf16_bits_to_f32(v) if dtype == "bf16" else v
    atol = 2.0 ** -18 * float(np.abs(v).max()) + 2e-6
    err = np.abs(out["attn_out"] - case.attn).max()
    print(f"[merge {name}] max|dO| = {err:.3e} (at most {atol:.3e})", flush=True)
    assert err <= atol
    check_x(case, out["x_out"], f"merge {name}")
