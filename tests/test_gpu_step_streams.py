"""Stage events and graph capture of a step, over the attention paths.

Stage events: every path records the four of them, in order (the one that ends the attention stage
goes with the merge or, where one split per sequence writes its outputs, with the attention kernel
itself), and the outputs are those of a step without events.

Capture: a plan whose first step took one path has a step of another captured, the path's first, and
replayed with eager steps in between; every replay's outputs are the eager step's, bit for bit.
"""
import numpy as np
import pytest

import attn_paths
import respec_synth as synth

from test_gpu_parity import rt  # noqa: F401 (rt is a fixture)
from test_gpu_stream_attention import _tree

pytestmark = pytest.mark.gpu

STEPS = {
    # path: (nodes per sequence, prefix lengths) of 32 heads, 64 columns
    "whole": ([9], [60]),
    "split": ([9], [2000]),
    "flat": ([5, 9, 2, 1, 3, 8, 4, 6], [100, 6200, 0, 1, 33, 64, 700, 31]),
    "shared": ([33, 5], [700, 31]),
    "stream": ([65], [3000]),
}


def _step(name, vocab=1003):
    import torch
    nodes, kv = STEPS[name]
    assert attn_paths.of(32, 32, 64, nodes, kv) == name
    parents = [_tree(n, 2 + i % 3) for i, n in enumerate(nodes)]
    gen = torch.Generator(device="cuda:0").manual_seed(len(nodes) + sum(kv))
    m, cap = sum(nodes), max(kv) + 65
    off = np.concatenate([[0], np.cumsum(nodes)])

    def rand(*shape):
        return torch.randn(*shape, generator=gen, device="cuda:0").bfloat16()

    def ints(v):
        return torch.tensor(np.asarray(v), dtype=torch.int32, device="cuda:0")

    ins = dict(node_off=ints(off), kv_len=ints(kv), hidden=rand(m, 2048), k_cache=rand(len(nodes), 32, cap, 64),
               v_cache=rand(len(nodes), 32, cap, 64), lm_head=rand(vocab, 2048),
               parent=ints([p for t in parents for p in t]), token=ints([7] * m),
               src=torch.zeros(m, dtype=torch.uint8, device="cuda:0"))
    call = dict(batch=len(nodes), total_nodes=m, max_nodes_in_batch=max(nodes), max_kv_len_in_batch=max(kv),
                kv_capacity=cap, topk=8)
    return ins, call


def _plan(vocab=1003):
    from paper_2511_01282_amd import binding
    return binding.Plan(hidden=2048, n_q_heads=32, n_kv_heads=32, head_dim=64, vocab=vocab, dtype=binding.BF16,
                        max_batch=8, max_nodes=65, max_depth=64, max_kv_len=6200, topk_out=8)


def _outputs(call, vocab=1003):
    import torch
    from paper_2511_01282_amd import binding
    return binding.alloc_outputs(total_nodes=call["total_nodes"], batch=call["batch"], hidden=2048, vocab=vocab, topk_out=8,
                                 max_depth=64, x_dtype=torch.bfloat16)


def _check(got, want, label):
    import torch
    for k, v in want.items():
        if v is not None and k != "sample":
            assert torch.equal(got[k], v), (label, k)


@pytest.mark.timeout(120)
@pytest.mark.parametrize("name", list(STEPS))
def test_stage_events(rt, name):  # noqa: F811
    import torch
    print(f"[events {name}]", flush=True)
    ins, call = _step(name)
    plan, want, got = _plan(), _outputs(call), _outputs(call)
    plan.step(ins, want, **call)
    events = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    for e in events:
        e.record()  # (creates it)
    torch.cuda.synchronize()
    plan.step(ins, got, stage_events=events, **call)
    torch.cuda.synchronize()
    stages = [events[k].elapsed_time(events[k + 1]) for k in range(3)]
    print(f"[events {name}] attention, LM head, vocabulary pass: {stages} ms", flush=True)
    assert all(0.0 < t < 50.0 for t in stages)
    _check(got, want, name)


@pytest.mark.timeout(120)
@pytest.mark.parametrize("name", list(STEPS))
def test_capture_of_a_paths_first_step(rt, name):  # noqa: F811
    import torch
    print(f"[capture {name}]", flush=True)
    other = "split" if name != "split" else "stream"
    ins, call = _step(name)
    want = _outputs(call)
    _plan().step(ins, want, **call)
    ins2, call2 = _step(other)
    want2, got2 = _outputs(call2), _outputs(call2)
    plan = _plan()
    plan.step(ins2, want2, **call2)
    torch.cuda.synchronize()
    got, graph = _outputs(call), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.step(ins, got, **call)
    for k in range(4):
        for v in got.values():
            if v is not None:
                v.zero_()
        graph.replay()
        torch.cuda.synchronize()
        _check(got, want, f"replay {k}")
        plan.step(ins2, got2, **call2)  # (the same workspace)
        torch.cuda.synchronize()
        _check(got2, want2, f"eager after replay {k}")
