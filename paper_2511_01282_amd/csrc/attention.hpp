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

// Pieces of the streaming kernel's only sequence (of `tiles` KV tiles).
__device__ __forceinline__ int stream_pieces_of_one(const AttnArgs& a, int tiles) {
  return min(a.pieces, max(1, tiles >> a.piece_shift));
}

}  // namespace respec
