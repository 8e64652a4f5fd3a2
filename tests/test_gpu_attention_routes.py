"""GPU parity of the attention kernels at the edges of the rules that pick one.

Each case names its path (tests/test_attention_route_rule.py checks on the CPU that it takes it):
  whole    the register path with one split per sequence, which writes its outputs without a merge;
  split    the register path with several;
  flat     the register path over pieces of the whole batch;
  shared   KV tiles shared through LDS, splits of each sequence;
  stream   KV tiles shared through LDS, pieces of the whole batch (two key groups for batches of
           128-column heads and, up to 12 tiles per CU of 256, for 64-column ones, else four).

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
    # name: (Hq, Hkv, D, nodes per sequence, prefix lengths, path[, dtype])
    # one split per sequence: four key-group waves, two, one; one and two 16-row blocks; more rows
    # than a workgroup holds
    "direct-one-node": (4, 4, 64, [1], [0], "whole"),
    "direct-short": (2, 2, 128, [26], [37], "whole"),
    "direct-grouped": (12, 4, 64, [9], [70], "whole"),
    "direct-batch": (4, 4, 128, [1 + k % 12 for k in range(70)], [(53 * k) % 300 for k in range(70)], "whole"),
    "direct-batch-d64": (8, 8, 64, [16 - k % 16 for k in range(65)], [(31 * k) % 200 for k in range(65)], "whole"),
    "direct-batch-full": (32, 32, 64, [1, 12, 5, 32, 20, 3, 9, 27], [900, 3, 500, 1300, 31, 0, 32, 77], "whole"),
    "one-48-rows-d64": (8, 2, 64, [12], [0], "whole"),
    "direct-64-rows": (8, 2, 64, [16], [40], "whole"),
    "direct-one-wave-column": (8, 2, 128, [17, 5], [14, 0], "whole"),
    "direct-f32": (4, 2, 64, [20], [20], "whole", "f32"),
    "direct-f32-one-wave-column": (4, 1, 64, [32], [0], "whole", "f32"),
    "direct-f32-two-blocks": (8, 1, 64, [20], [12], "whole", "f32"),
    "direct-f32-batch": (4, 4, 128, [1 + k % 9 for k in range(66)], [(41 * k) % 90 for k in range(66)], "whole", "f32"),
    # splits of each sequence, of one or a batch
    "one-33-rows": (2, 2, 128, [33], [90], "split"),
    "one-64-rows": (2, 2, 128, [64], [1023], "split"),
    "one-63-rows-grouped": (18, 2, 128, [7], [320], "split"),
    "one-f32-61-nodes": (4, 1, 64, [61], [20], "split", "f32"),
    "one-f32-two-tiles-more": (4, 2, 64, [30], [60], "split", "f32"),
    "one-at-20-tiles": (64, 64, 64, [34], [80 * 32 - 34], "split"),
    "batch-of-splits": (8, 8, 128, [16, 32, 9], [500, 1234, 0], "split"),
    "batch-of-splits-grouped": (4, 2, 128, [17, 32, 1, 5], [70, 2000, 0, 31], "split"),
    "batch-of-splits-d64": (4, 2, 64, [17, 1, 32, 5, 9], [2000, 0, 31, 32, 650], "split"),
    "batch-of-splits-128-rows": (16, 2, 64, [16, 9, 2], [1000, 0, 33], "split"),
    "batch-f32": (4, 2, 64, [8, 16, 3], [300, 100, 0], "split", "f32"),
    # pieces of a batch on the register path
    "pieces": (16, 16, 128, [6, 1, 12, 3, 2, 5, 4, 9], [700, 0, 3800, 31, 32, 33, 100, 5], "flat"),
    "pieces-grouped": (16, 8, 128, [3, 16, 8, 1, 2, 7, 5, 9], [64, 7700, 0, 900, 31, 32, 33, 2000], "flat"),
    "pieces-f32": (8, 8, 64, [9, 30, 4, 1, 2, 3, 6, 5], [64, 2100, 0, 900, 31, 32, 33, 500], "flat", "f32"),
    "pieces-f32-two-waves": (16, 8, 64, [9, 30, 4, 1, 2, 3, 6, 5], [64, 1100, 0, 900, 31, 32, 33, 500], "flat", "f32"),
    # shared tiles: one sequence whose last row wave is at most half live, a few short sequences, one per
    # CU, many of 64-column heads
    "shared-97-rows": (32, 32, 128, [97], [1500], "shared"),
    "shared-112-rows-grouped": (32, 16, 128, [56], [3100], "shared"),
    "shared-65-rows": (32, 32, 128, [65], [1600], "shared"),
    "shared-65-rows-rotated": (32, 32, 128, [65], [16400], "shared"),
    "shared-33-rows": (32, 32, 128, [33], [5120], "shared"),
    "shared-a-few": (32, 32, 64, [41, 1, 33], [700, 0, 1100], "shared"),
    "shared-a-few-grouped": (32, 16, 128, [9, 40, 2], [33, 700, 0], "shared"),
    "shared-per-cu": (32, 32, 128, [33, 64, 1, 17, 40, 5, 12, 60], [300, 1100, 31, 32, 150, 0, 7, 200], "shared"),
    "shared-per-cu-128-rows-d64": (64, 32, 64, [33, 64, 1, 17, 40, 5, 12, 60], [300, 600, 31, 32, 150, 0, 7, 200], "shared"),
    "shared-many-d64": (8, 4, 64, [17] + [1 + k % 5 for k in range(269)], [150] + [(37 * k) % 120 for k in range(269)],
                        "shared"),
    "shared-many-32-rows": (8, 4, 64, [16] + [1 + k % 5 for k in range(199)], [300] + [(37 * k) % 200 for k in range(199)],
                            "shared"),
    # streams
    "one-past-20-tiles": (64, 64, 64, [34], [80 * 32 - 33], "stream"),
    "one-long-d128": (32, 32, 128, [50], [5300], "stream"),
    "batch-two-groups": (4, 2, 128, [17, 32, 1, 5], [70, 2100, 0, 31], "stream"),
    "batch-two-groups-d64": (4, 2, 64, [17, 1, 32, 5, 9], [2100, 0, 31, 32, 650], "stream"),
    "batch-four-groups-d64": (32, 32, 64, [34, 5, 60, 1, 2], [800, 0, 31, 90, 7], "stream"),
}


def shape(hq, hkv, d):
    """Heads of a case: a hidden row is a multiple of 512 bytes."""
    return (hq, hkv, d) if hq * d * 2 % 512 == 0 else (2 * hq, 2 * hkv, d)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("name", list(CASES))
def test_attention_routes(rt, name):  # noqa: F811
    hq, hkv, d, nodes, kv, _, dtype = (*CASES[name], "bf16")[:7]
    hq, hkv, d = shape(hq, hkv, d)
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
