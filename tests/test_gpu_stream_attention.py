"""GPU parity of the streaming attention kernel (bf16; tests/test_attention_route_rule.py checks on
the CPU that every case takes it).

Attention output and residual against the CPU oracle, at the edges of the kernel's dispatch:
query rows per KV head on both sides of every wave and key-group count (65 and 128: three and four
row waves in two key groups; 129 and 256: five and eight in one; 260 and 455: two row blocks, the
latter cut inside a node's heads; 33-64 rows of batches: two waves in two key groups or, with many
tiles of 64 columns, four), prefixes that end on, before and after a 32-row tile, sequences shorter
than the key groups, ragged batches whose pieces span several sequences (and sequences that span
several pieces), more sequences than a slice of 256 holds, and plans larger than the step.

Tolerance: the probabilities are the sum of two bf16 parts, off by at most 2^-18 of themselves
(the second part rounds a remainder of at most 2^-9), and the weights of a row sum to one, so O
is off by at most 2^-18 max|V|; 2e-6 more for the float32 sums and the exponential.
"""
import numpy as np
import pytest

import respec_synth as synth
import workload

from test_gpu_parity import check_x, rt, _depth  # noqa: F401 (rt is a fixture)

pytestmark = pytest.mark.gpu


def _tree(n, arity=2):
    return [-1] + [(j - 1) // arity for j in range(1, n)]


CASES = {
    # name: (Hq, Hkv, D, nodes per sequence, prefix lengths[, nodes of the plan])
    "65-rows": (2, 2, 128, [65], [995]),
    "65-rows-larger-plan": (2, 2, 128, [65], [995], 128),
    "128-rows-d64": (8, 1, 64, [16], [33]),
    "129-rows": (3, 1, 128, [43], [700]),
    "256-rows": (8, 2, 128, [64], [95]),
    "256-rows-of-a-batch": (4, 2, 64, [128, 65], [200, 40]),
    "260-rows-two-blocks": (8, 2, 128, [65], [300]),
    "455-rows-two-blocks-inside-a-node": (14, 2, 128, [65], [300]),
    "455-rows-of-a-batch": (14, 2, 128, [65, 1, 40, 37], [600, 0, 31, 90]),
    "455-rows-of-a-batch-d64-larger-plan": (14, 2, 64, [65, 1, 40, 37], [600, 0, 31, 90], 128),
    "empty-prefix": (8, 1, 128, [17, 1], [0, 0]),
    "ragged-two-groups": (4, 2, 128, [17, 1, 32, 5, 9], [2100, 0, 31, 32, 650]),
    "ragged-two-groups-larger-plan": (4, 2, 128, [17, 1, 32, 5, 9], [2100, 0, 31, 32, 650], 128),
    "ragged-one-group": (8, 2, 64, [60, 1, 33, 7], [97, 3000, 1, 512]),
    "ragged-one-group-larger-plan": (8, 2, 64, [60, 1, 33, 7], [97, 3000, 1, 512], 100),
    "two-slices": (4, 2, 128, [17] + [1 + k % 5 for k in range(269)], [150] + [(37 * k) % 120 for k in range(269)]),
}


def _rows_in_use(w):
    """V rows that some node sees (the cache's tail is poisoned)."""
    n = np.diff(w.node_off)
    return np.concatenate([w.v_cache[b][:, :int(w.kv_len[b]) + int(n[b])].reshape(-1) for b in range(len(n))])


@pytest.mark.timeout(300)
@pytest.mark.parametrize("name", list(CASES))
def test_stream_attention_parity(rt, name):  # noqa: F811
    hq, hkv, d, nodes, kv, plan_nodes = (*CASES[name], 0)[:6]
    parents = [_tree(n, 2 + i % 3) for i, n in enumerate(nodes)]
    # (the cache holds the longest prefix plus the largest tree)
    big, far = int(np.argmax(nodes)), int(np.argmax(kv))
    parents[big], parents[far] = parents[far], parents[big]
    depth = max(8, max(_depth(p) for p in parents))
    # (a hidden row is a multiple of 512 bytes)
    hq, hkv = (hq, hkv) if hq * d * 2 % 512 == 0 else (2 * hq, 2 * hkv)
    shp = synth.Shape("edge", "bf16", hq * d, hq, hkv, d, 520, len(nodes), max(nodes), depth, 8)
    w = synth.custom(shp, parents, kv, seed=611, poison_tail=True)
    print(f"[stream {name}] building", flush=True)
    case = workload.finish(w)
    print(f"[stream {name}] running GPU step", flush=True)
    from paper_2511_01282_amd import binding
    plan = rt.make_plan(case.w, max_nodes=plan_nodes) if plan_nodes else None
    out = rt.run(case.w, plan=plan, x_out=True, stop_after=binding.STOP_ATTN)
    atol = 2.0 ** -18 * float(np.abs(synth.bf16_bits_to_f32(_rows_in_use(case.w))).max()) + 2e-6
    err = np.abs(out["attn_out"] - case.attn).max()
    print(f"[stream {name}] max|dO| = {err:.3e} (at most {atol:.3e})", flush=True)
    assert err <= atol
    check_x(case, out["x_out"], f"stream {name}")
