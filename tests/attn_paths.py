"""The library's rule for the attention kernel of a step (attn_route.hpp, host code), for the tests."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_01282_amd", "csrc")
NAMES = ("split", "flat", "shared", "stream")

_SOURCE = """
#include "attn_route.hpp"
using namespace respec;
extern "C" int path(int es, int d, int hkv, int batch, int rows, long long tiles) {
  return (int)attn_path(es, d, hkv, batch, rows, tiles);
}
extern "C" void splits(int wgs, int batch, int heads, long long tiles, int least, long long held, int* out) {
  const Splits s = kv_splits(wgs, batch, heads, tiles, least, (size_t)held);
  out[0] = s.n;
  out[1] = s.tiles;
}
extern "C" int rotated(int d, int batch, int cap) { return tiles_rotated(d, batch, cap); }
extern "C" void row_geometry(int rows, int* out) {
  const RowGeom g = row_geom(rows);
  const int v[6] = {g.nb, g.wr, g.wk, g.rows_per_wg, g.n_rowblk, g.threads};
  for (int i = 0; i < 6; ++i) out[i] = v[i];
}
"""


@functools.lru_cache(None)
def lib():
    with tempfile.TemporaryDirectory() as d:
        src, out = os.path.join(d, "route.cpp"), os.path.join(d, "route.so")
        with open(src, "w") as f:
            f.write(_SOURCE)
        subprocess.check_call([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                               "-I", CSRC, src, "-o", out])
        L = ctypes.CDLL(out)
    L.path.argtypes = [ctypes.c_int] * 5 + [ctypes.c_longlong]
    L.splits.argtypes = [ctypes.c_int] * 3 + [ctypes.c_longlong, ctypes.c_int, ctypes.c_longlong, ctypes.c_void_p]
    L.row_geometry.argtypes = [ctypes.c_int, ctypes.c_void_p]
    return L


def path(es, d, hkv, batch, rows, tiles):
    return NAMES[lib().path(es, d, hkv, batch, rows, tiles)]


def rotated(d, batch, cap):
    return bool(lib().rotated(d, batch, cap))


def splits(wgs, batch, heads, tiles, least, held):
    out = (ctypes.c_int * 2)()
    lib().splits(wgs, batch, heads, tiles, least, held, out)
    return out[0], out[1]


def row_geometry(rows):
    out = (ctypes.c_int * 6)()
    lib().row_geometry(rows, out)
    return dict(zip(("nb", "wr", "wk", "rows_per_wg", "n_rowblk", "threads"), out))


def of(hq, hkv, d, nodes, kv, dtype="bf16"):
    """The path of a step, or "whole" where one split per sequence writes its outputs itself."""
    es, rows = (2 if dtype == "bf16" else 4), max(nodes) * (hq // hkv)
    tiles = (max(kv) + max(nodes) + 31) // 32
    name = path(es, d, hkv, len(nodes), rows, tiles)
    if name == "split":
        g = row_geometry(rows)
        n, _ = splits(1024 // (g["threads"] // 64), len(nodes), hkv * g["n_rowblk"], tiles, g["wk"], 1 << 40)
        name = "whole" if n == 1 else name
    return name
