// Which attention kernel a step takes, and how the KV rows are cut (host side, plain C++).
#pragma once

#include <limits.h>
#include <stddef.h>

namespace respec {

constexpr int kCUs = 256;    // compute units of an MI355X
constexpr int kKvTile = 32;  // KV rows per tile of the attention kernels

enum class AttnPath {
  kSplit,   // tree_attn_kernel: splits of each sequence (one split: no merge follows)
  kFlat,    // tree_attn_kernel: equal pieces of the whole batch
  kShared,  // tree_attn_shared_kernel: splits of each sequence, KV tiles shared through LDS
  kStream   // tree_attn_stream_kernel: equal pieces of the whole batch, as one stream per workgroup
};

// `rows` query rows per KV head of the largest tree, `tiles` KV tiles of the longest sequence (the
// shorter ones are known to the device alone).  Figures: us per attention layer, merge included.
inline AttnPath attn_path(int es, int head_dim, int n_kv_heads, int batch, int rows, long long tiles) {
  const long long heads = (long long)batch * n_kv_heads;  // workgroups of one sequence and KV head each
  const bool pieces_fit = batch > 1 && batch <= 64;       // (kFlat: a lane per sequence)
  const long long splits = heads >= kCUs ? 1 : kCUs / heads, split_tiles = (tiles + splits - 1) / splits;
  // A piece starts anew at every sequence it touches, 8 us each, and the partials are merged; a
  // split that holds a whole sequence is not, but the longest sequence ends alone.  So the rows of a
  // split decide.
  if (es != 2) {
    // 8 sequences, 8 heads of 64 columns, over 100-600 rows (splits of 150) splits 1.1 times as
    // fast, over 300-2000 (500) the same, 24 sequences (2000) 0.7 times; with two row waves 4
    // sequences over 300-2000 (250) 0.9 times.
    return pieces_fit && split_tiles > (rows <= 32 ? 15 : 7) ? AttnPath::kFlat : AttnPath::kSplit;
  }
  if (rows <= 32) {
    // 64-column heads fit two shared rings on a CU: many short sequences of 17-32 rows (64 of 32
    // heads over 100-500 rows: shared 66, splits 79, pieces 132).
    if (head_dim == 64 && rows > 16 && heads >= 3 * kCUs && 64 * tiles <= heads) return AttnPath::kShared;
    // 8 sequences of 32 nodes, 32 heads, splits / pieces: over 50-300 rows 14.8 / 33.9, 200-1000
    // 23 / 34, 500-4000 62.8 / 62.8, 4000-16000 249 / 214.  With two pieces per sequence or more, as
    // few KV heads leave, a piece seldom starts anew: 8 sequences of 8 heads of 4 over 1000-8000
    // rows (splits of 2000) 34 / 31.  64 columns take half the time per row.
    const bool many = n_kv_heads <= 16 && 2 * heads <= kCUs;
    return pieces_fit && split_tiles * head_dim > (many ? 7600 : 12288) ? AttnPath::kFlat : AttnPath::kSplit;
  }
  const bool half_idle = (rows - 1) % 32 < 16;  // the last wave of 32 rows
  if (batch == 1) {
    // Two waves of rows while a CU has few tiles: the register path starts 3-4 us sooner, and the
    // second read of each tile comes from L2.  34 nodes of 32 heads over 1000 rows 14.0 against 17.0
    // us in a stream, over 4000 21.6 / 22.9, over 8000 (32 tiles per CU) 31.9 / 30.3; 12 nodes on 8
    // heads of 4 over 4000 rows 11.4 / 15.0.
    const long long cu_tiles = tiles * n_kv_heads;
    if (rows <= 64 && cu_tiles <= 20ll * kCUs) return AttnPath::kSplit;
    // A last row wave with 16 live rows or fewer is half idle in the stream, whose products are 32
    // rows high (32 heads, shared / stream: 65 nodes over 2100-3000 rows 0.92, 100 over 4000 28.1 / 31.3,
    // over 8000 43.7 / 43.8; 96 over 3000 0.94, over 4000 1.12; 128 over 32000 1.15).
    // 65-80 rows at any length (with tiles_rotated; 65 nodes over 16384 rows 61.0 / 63.4, over 48000 150 / 157,
    // 40 heads 188 / 199; 33 over 17000 59.7 / 60.7 and 40 over 24000 80.0 / 79.3; 97 over 17000 1.04).
    const bool any_length = rows > 64 && rows <= 80;
    if (head_dim == 128 && rows <= 128 && half_idle && cu_tiles > 6ll * kCUs && (any_length || cu_tiles <= 64ll * kCUs))
      return AttnPath::kShared;
    return AttnPath::kStream;
  }
  if (rows <= 128) {
    // Few KV heads: 2-4 sequences of 17 nodes on 8 heads of 4 over up to 1000 rows 15-22 us in
    // splits, 17-24 in a stream.
    if (heads <= 32 && tiles <= 64) return AttnPath::kSplit;
    // A few short ones whose last row wave is half idle (2 of 48 nodes, 32 heads, over 200-1000 rows
    // 20.4 shared, 22.7 in a stream; 2 of 61 25.3 and 23.5, 48 nodes over 100-500 21.1 and 17.9).
    if (batch <= 4 && n_kv_heads >= 16 && half_idle && tiles > 20 && tiles <= 40) return AttnPath::kShared;
    // One short sequence per CU: 8 of 61 nodes, 32 heads, over 200-1000 rows 28.4 shared, 36.8 in a
    // stream, 8 of 48 over 300-2000 49.6 and 44.5 (12 of 61 over 200-1000 54 and 46.8).
    if (heads == kCUs && batch <= 8 && tiles <= 40) return AttnPath::kShared;
    // Two shared rings on a CU hide each other's starts and ends: 32 of 48 nodes, 32 heads of 64
    // columns, over 100-500 rows 41 shared and 69 in a stream, over 500-4000 (24 sequences) 96 and
    // 104; 12 sequences over 500-4000 73 and 59.
    if (head_dim == 64 && rows <= 64 && 2 * heads >= 3 * kCUs && 6 * tiles <= heads) return AttnPath::kShared;
  }
  return AttnPath::kStream;
}

// Whether the shared-tile kernel takes a split's tiles in rotated order (tile_rotation in attention.hpp).  In
// order, the splits of a few sequences meet on the same memory channels where the heads lie near a multiple
// of 512 KB plus or minus 32 KB apart (65 nodes of 32 heads over 16384 rows, in order / rotated: capacity
// 16512 68.0 / 61.7 us, 20608 64.4 / 60.6, at six others 59.6-61.8 / 60.2-61.7; in order, of 170 capacities up
// to 20800 those above 63 us lie 28-48 KB off a multiple); elsewhere they keep out of each other's way, and a short split ends with its masked tiles (over 48000 rows 150 / 155; 2 sequences of 48
// nodes over 200-1000 rows 19.6 / 21.4).  More sequences, of unlike lengths: rotated (24 of 48 nodes, 32
// heads of 64 columns, over 500-4000 rows 105 / 101).
inline bool tiles_rotated(int head_dim, int batch, int kv_capacity) {
  const long long span = 1 << 19, stride = 2ll * head_dim * kv_capacity, off = (stride + span / 2) % span - span / 2;
  const long long apart = off < 0 ? -off : off;
  return batch > 4 || (apart >= 20480 && apart <= 51200);
}

inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }
inline int clampi(int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); }

// Register-path attention (tree_attn_kernel) of `rows` query rows per KV head:
// rows are (node, head-in-group) pairs; a wave owns at most 32 of them (more
// would not fit the registers next to a ring of tiles); above 4 waves' worth a
// head's KV rows are read once per row block.
struct RowGeom {
  int nb, wr, wk, rows_per_wg, n_rowblk, threads;
};
inline RowGeom row_geom(int rows) {
  RowGeom g;
  g.nb = rows <= 16 ? 1 : 2;
  const int rb = 16 * g.nb, rg = cdiv(rows, rb);
  g.wr = rg < 4 ? rg : 4;
  g.n_rowblk = cdiv(rg, g.wr);
  g.rows_per_wg = g.wr * rb;
  const int by_waves = 4 / g.wr, by_rows = 128 / g.rows_per_wg;
  g.wk = clampi(by_waves < by_rows ? by_waves : by_rows, 1, 4);
  g.threads = 64 * g.wr * g.wk;
  return g;
}

// Splits of each sequence: as many as fill `wgs` workgroups over `heads` (KV head, row block) pairs
// of `batch` sequences, of `least` tiles or more (one per key-group wave: fewer, fuller splits for
// short caches), at most `held`.
struct Splits {
  int n, tiles;  // splits, tiles of each
};
inline Splits kv_splits(int wgs, int batch, int heads, long long tiles, int least, size_t held) {
  const int most = held < (size_t)tiles ? (int)held : (int)tiles;
  const int target = clampi((int)(wgs / ((long long)batch * heads)), 1, most);
  Splits s;
  s.tiles = cdiv(tiles, target);
  if (s.tiles < least) s.tiles = least;
  s.n = cdiv(tiles, s.tiles);
  return s;
}

}  // namespace respec
