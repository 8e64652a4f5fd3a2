// Device helpers shared by the attention kernels.
#pragma once

#include "common.hpp"
#include "kernels.hpp"

namespace respec {

// Rows of sequence b's KV range (prefix + tree); invalid device data degrades
// to an empty sequence.  The merge computes the same, so both agree on the
// flat partition.
struct SeqRows {
  int node0, n_nodes, L;
};
__device__ __forceinline__ SeqRows seq_rows(const AttnArgs& a, int b) {
  const int node0 = a.node_off[b], node1 = a.node_off[b + 1];
  int n_nodes = node1 - node0;
  if (node0 < 0 || node1 > a.total_nodes || n_nodes < 1 || n_nodes > a.max_nodes) n_nodes = 0;
  int L = a.kv_len[b];
  L = max(0, min(L, a.kv_cap - n_nodes));
  return SeqRows{node0, n_nodes, n_nodes > 0 ? L : 0};
}

// A workgroup's KV tiles are taken in rotated order, from a start that differs from
// workgroup to workgroup: heads and pieces lie at regular distances, and
// workgroups that all walk their tiles from the first one meet on the same
// memory channels where a head's rows take near a multiple of 512 KB plus or minus
// 32 KB.  The start is quadratic in the head: one that is linear (or none) moves
// the meeting to other cache capacities.  33 nodes of 32 heads over 15800 rows, us per
// attention layer at 50 capacities of 15872 to 16656 rows: by 5 x alone 55.4-69.3, by
// 5 x + 3 y 55.7-68.4, by 5 x + 17 y 55.0-61.5, this 56.0-58.4 (KV tiles in order, in a
// kernel of per-sequence splits: 57.5-77.5); 65 nodes 58.8-72.8, 58.2-71.2, 59.2-64.3,
// 59.2-61.6 (59.7-80.3).
__device__ __forceinline__ int tile_rotation(int n_tiles) {
  return (int)((blockIdx.x * 5 + blockIdx.y * blockIdx.y * 3) % (uint32_t)n_tiles);
}

// Pieces of the streaming kernel's only sequence (of `tiles` KV tiles).
__device__ __forceinline__ int stream_pieces_of_one(const AttnArgs& a, int tiles) {
  return min(a.pieces, max(1, tiles >> a.piece_shift));
}

}  // namespace respec
