"""GPU parity of the LM head's DMA-fed kernels (bf16), at the edges of their tiles.

The token rows lie on both sides of every tile height the dispatch takes over these vocabularies
(128, 192 and 256 by 128, then 128 to 256 by 256 in steps of 32), in one and several tiles; the
vocabularies end inside a tile (one row, and odd counts that rule out 16-byte stores); up to 64 rows, the vocabulary
leaves a last round of tiles of every height (64 to 256 rows), alone and after whole tiles; the hidden
sizes give the shortest K loop (4 steps, as long as or shorter than the request rings hold) and
longer ones.

Tolerance: the products are exact in float32 and summed over K in some order, each sum off by at
most 2^-23 of the partial sums, so a logit is off by at most K 2^-23 sum |x||w|.  The statistics
are compared with those of the returned logits: sums of V float32 terms whose exponentials are off
by at most about 2^-20 (the argument's rounding, |z - max| < 32): 1e-5 on the log-sum-exp; the
entropy weights each term's logarithm with it, 1e-5 times log V (at most 11) and a rounding.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [
    # (token rows, hidden, vocab)
    (1, 256, 16449), (33, 512, 20001), (17, 256, 33001), (64, 768, 49153), (61, 256, 66003), (5, 512, 65600),
    (40, 256, 90004), (9, 4096, 41001), (20, 8192, 33001), (48, 256, 70000), (64, 256, 130001),
    (65, 256, 32001), (128, 512, 520), (129, 256, 32001), (192, 768, 32004), (193, 256, 32001), (224, 512, 20001), (256, 1024, 32003),
    (257, 256, 32004), (320, 512, 32001), (321, 256, 32002), (384, 768, 32001), (385, 256, 32001), (448, 512, 32004),
    (449, 256, 32257), (512, 768, 32001), (897, 512, 32001), (1025, 256, 1537),
]


@pytest.mark.timeout(120)
@pytest.mark.parametrize("m,hidden,vocab", CASES)
def test_lmhead_tiles(m, hidden, vocab):
    from paper_2511_01282_amd import binding
    print(f"[lmhead] {m} rows, hidden {hidden}, vocab {vocab}", flush=True)
    dev = "cuda:0"
    gen = torch.Generator(device=dev).manual_seed(m)
    heads, d = hidden // 64, 64
    batch = -(-m // 64)
    nodes = [m // batch + (1 if b < m % batch else 0) for b in range(batch)]
    off = [sum(nodes[:b]) for b in range(batch + 1)]

    def rand(*shape, std=1.0):
        return (torch.randn(*shape, generator=gen, device=dev) * std).bfloat16()

    def ints(v):
        return torch.tensor(v, dtype=torch.int32, device=dev)

    w = rand(vocab, hidden, std=0.1)
    ins = dict(node_off=ints(off), kv_len=ints([0] * batch), hidden=rand(m, hidden), k_cache=rand(batch, heads, 64, d),
               v_cache=rand(batch, heads, 64, d), lm_head=w,
               parent=ints([j - 1 for n in nodes for j in range(n)]), token=ints([7] * m),
               src=torch.zeros(m, dtype=torch.uint8, device=dev))
    plan = binding.Plan(hidden=hidden, n_q_heads=heads, n_kv_heads=heads, head_dim=d, vocab=vocab, dtype=binding.BF16,
                        max_batch=batch, max_nodes=64, max_depth=64, max_kv_len=0, topk_out=8)
    out = binding.alloc_outputs(total_nodes=m, batch=batch, hidden=hidden, vocab=vocab, topk_out=8, max_depth=64,
                                x_dtype=torch.bfloat16)
    out["logits"].fill_(float("nan"))
    plan.step(ins, out, batch=batch, total_nodes=m, max_nodes_in_batch=max(nodes), max_kv_len_in_batch=0,
              kv_capacity=64, topk=8, stop_after=binding.STOP_STATS)
    torch.cuda.synchronize()
    x, z = out["x_out"].double(), out["logits"]
    w64 = w.double().t().contiguous()
    err = (z.double() - x @ w64).abs() / (x.abs() @ w64.abs())
    print(f"[lmhead] largest error {float(err.max()) * 2 ** 23 / hidden:.3f} of its bound", flush=True)
    assert bool((err <= hidden * 2.0 ** -23).all())
    z = z.double()
    lse = torch.logsumexp(z, 1)
    logp = z - lse[:, None]
    assert torch.equal(out["argmax"].long(), z.argmax(1))
    assert torch.equal(out["max_logit"].double(), z.max(1).values)
    assert float((out["lse"] - lse).abs().max()) <= 1e-5 + 2.0 ** -23 * float(lse.abs().max())
    assert float((out["entropy"] + (logp.exp() * logp).sum(1)).abs().max()) <= 1.2e-4
    top = z.topk(8, 1)
    assert float((out["topk_logprob"] - (top.values - lse[:, None])).abs().max()) <= 3e-5
