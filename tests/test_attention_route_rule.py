"""The rule that picks the attention kernel, and the cut into splits (host code, on the CPU).

Every GPU parity case names the path it is there for: this checks that it takes it, so that a later
change of the rule cannot leave a kernel without its cases.
"""
import random

import pytest

import attn_paths
import test_gpu_attention_routes as routes
import test_gpu_split_merge as merge
import test_gpu_stream_attention as stream


@pytest.mark.parametrize("name", list(routes.CASES))
def test_routes_cases(name):
    hq, hkv, d, nodes, kv, want, dtype = (*routes.CASES[name], "bf16")[:7]
    assert attn_paths.of(*routes.shape(hq, hkv, d), nodes, kv, dtype) == want


@pytest.mark.parametrize("name", list(stream.CASES))
def test_stream_cases(name):
    hq, hkv, d, nodes, kv = stream.CASES[name][:5]
    assert attn_paths.of(*routes.shape(hq, hkv, d), nodes, kv) == "stream"


@pytest.mark.parametrize("name", list(merge.CASES))
def test_merge_cases(name):
    hq, hkv, d, nodes, kv, dtype, _, want = merge.CASES[name]
    assert attn_paths.of(hq, hkv, d, nodes, kv, dtype) == want


EDGES = [
    # (bytes per element, D, KV heads, sequences, rows, tiles): path
    ((2, 128, 32, 1, 64, 160), "split"), ((2, 128, 32, 1, 64, 161), "stream"),
    ((2, 128, 32, 1, 48, 160), "split"), ((2, 128, 32, 1, 48, 161), "shared"), ((2, 128, 32, 1, 49, 161), "stream"),
    ((2, 128, 32, 1, 96, 100), "stream"), ((2, 128, 32, 1, 97, 100), "shared"), ((2, 128, 32, 1, 97, 48), "stream"),
    ((2, 128, 32, 1, 112, 512), "shared"), ((2, 128, 32, 1, 112, 513), "stream"), ((2, 128, 32, 1, 113, 100), "stream"),
    ((2, 128, 32, 1, 65, 513), "shared"), ((2, 128, 40, 1, 80, 4000), "shared"), ((2, 128, 32, 1, 81, 100), "stream"),
    ((2, 128, 32, 1, 48, 512), "shared"), ((2, 128, 32, 1, 48, 513), "stream"), ((2, 64, 32, 1, 65, 513), "stream"),
    ((2, 64, 32, 1, 97, 100), "stream"), ((2, 128, 32, 1, 129, 100), "stream"),
    ((2, 128, 16, 4, 33, 40), "shared"), ((2, 128, 16, 4, 33, 41), "stream"), ((2, 128, 16, 4, 33, 20), "stream"),
    ((2, 128, 16, 5, 33, 40), "stream"), ((2, 64, 32, 2, 112, 21), "shared"), ((2, 64, 32, 2, 113, 21), "stream"),
    ((2, 128, 32, 2, 129, 40), "stream"),
    ((2, 128, 32, 8, 32, 96), "split"), ((2, 128, 32, 8, 32, 97), "flat"), ((2, 64, 32, 8, 32, 192), "split"),
    ((2, 64, 32, 8, 32, 193), "flat"), ((2, 128, 32, 65, 32, 500), "split"), ((2, 128, 8, 8, 16, 236), "split"),
    ((2, 128, 8, 8, 16, 240), "flat"), ((2, 128, 8, 17, 16, 96), "split"), ((2, 128, 8, 17, 16, 97), "flat"),
    ((2, 64, 32, 24, 17, 12), "shared"), ((2, 64, 32, 24, 17, 13), "split"), ((2, 64, 32, 24, 16, 12), "split"),
    ((2, 128, 8, 4, 128, 64), "split"), ((2, 128, 8, 4, 128, 65), "stream"), ((2, 128, 8, 4, 129, 64), "stream"),
    ((2, 128, 32, 8, 128, 40), "shared"), ((2, 128, 32, 8, 128, 41), "stream"), ((2, 128, 8, 32, 64, 40), "stream"),
    ((2, 64, 32, 12, 64, 64), "shared"), ((2, 64, 32, 12, 64, 65), "stream"), ((2, 64, 32, 12, 65, 64), "stream"),
    ((2, 64, 32, 11, 64, 20), "stream"),
    ((4, 64, 8, 8, 32, 60), "split"), ((4, 64, 8, 8, 32, 61), "flat"), ((4, 64, 8, 8, 33, 29), "flat"),
    ((4, 64, 8, 65, 33, 500), "split"), ((4, 64, 8, 1, 500, 500), "split"),
]


@pytest.mark.parametrize("args,want", EDGES)
def test_rule_edges(args, want):
    assert attn_paths.path(*args) == want


ROTATED = [
    # (D, sequences, KV capacity): rotated
    ((128, 1, 16449), False), ((128, 1, 16512), True), ((128, 1, 16256), True), ((128, 1, 20608), True),
    ((128, 1, 16384), False), ((128, 1, 16463), False), ((128, 1, 16464), True), ((128, 1, 16584), True),
    ((128, 1, 16585), False), ((128, 1, 18273), True), ((128, 1, 18593), True), ((128, 1, 18432), False), ((128, 4, 1061), False), ((128, 5, 1061), True), ((64, 2, 8320), False),
    ((64, 2, 8448), True), ((128, 1, 2147483647), False),
]


@pytest.mark.parametrize("args,want", ROTATED)
def test_rotation_edges(args, want):
    assert attn_paths.rotated(*args) is want


def test_splits_cover_every_tile():
    """Any sizes: the splits cover the tiles, none is empty, and the workspace holds them."""
    rng = random.Random(3)
    for _ in range(20000):
        wgs, batch, heads = rng.choice([256, 512]), rng.randint(1, 400), rng.randint(1, 300)
        tiles, least = rng.randint(1, 5000), rng.randint(1, 4)
        held = rng.choice([1, 2, 7, 64, 1 << 40])
        n, per = attn_paths.splits(wgs, batch, heads, tiles, least, held)
        assert 1 <= n <= held and per >= least
        assert (n - 1) * per < tiles <= n * per


def test_row_geometry():
    """Any rows: the waves own them all, and a workgroup has four waves at most."""
    for rows in range(1, 2000):
        g = attn_paths.row_geometry(rows)
        assert g["rows_per_wg"] == 16 * g["nb"] * g["wr"] and g["threads"] == 64 * g["wr"] * g["wk"] <= 256
        assert (g["n_rowblk"] - 1) * g["rows_per_wg"] < rows <= g["n_rowblk"] * g["rows_per_wg"]


@pytest.mark.parametrize("dtype,batch,nodes", [(0, 64, 1), (1, 64, 1), (1, 1, 61)])
def test_workspace_holds_no_spans_where_no_stream_has_them(dtype, batch, nodes):
    """float32, at most 32 rows per KV head, one sequence: the vocabulary's statistics alone grow with it."""
    import ctypes
    from paper_2511_01282_amd import binding

    def size(vocab):
        h = ctypes.c_void_p()
        s = binding.Shape(64 * 128, 64, 64, 128, vocab, dtype, batch, nodes, 8, 4000, 1)
        assert binding.lib().respec_verify_create(ctypes.byref(s), ctypes.byref(h)) == binding.OK
        n = binding.lib().respec_verify_workspace_bytes(h)
        binding.lib().respec_verify_destroy(h)
        return n

    def aligned(n):
        return -(-n // 256) * 256

    rows = batch * nodes
    for tiles in range(1, 40):
        assert size(64 * tiles + 64) - size(64 * tiles) == aligned(16 * rows * (tiles + 1)) - aligned(16 * rows * tiles)
