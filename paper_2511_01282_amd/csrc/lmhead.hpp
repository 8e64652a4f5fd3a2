// Shared by the LM head's DMA-fed kernels (lmhead.hip, lmhead_pair.hip).
#pragma once

#include "common.hpp"
#include "kernels.hpp"

namespace respec {

constexpr int kGmStep = 128;                    // bytes of a row per K step (64 elements)
constexpr int kGmWaves = 8;                     // waves per workgroup

// One 1 KB DMA request (8 rows of 128 bytes): lane l fills chunk position l % 8
// of row 8 q + l / 8 with the chunk that belongs there.
__device__ __forceinline__ void gm_dma(uint32_t lds_dst, uint64_t base, uint32_t off) {
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %2, %3\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(lds_dst), "v"(off), "s"(base)
      : "memory");
}

// Statistics {max, sum, entropy sum, argmax} of one token row's logits z of the 64-row statistics tile at vh
// (entries at or past V are not logits), by one thread.
__device__ __forceinline__ void tile_row_stats(const f32x4* z4, int vh, int vocab, float* dst) {
  float z[kLmTileRows];
#pragma unroll
  for (int q = 0; q < kLmTileRows / 4; ++q) {
    const f32x4 v = z4[q];
    z[4 * q] = v[0];
    z[4 * q + 1] = v[1];
    z[4 * q + 2] = v[2];
    z[4 * q + 3] = v[3];
  }
  const int nv = vocab - vh;
  float mx = kNegInf;
#pragma unroll
  for (int i = 0; i < kLmTileRows; ++i) mx = i < nv ? fmaxf(mx, z[i]) : mx;
  float S = 0.f, T = 0.f;
  int am = 0x7FFFFFFF;
#pragma unroll
  for (int i = kLmTileRows - 1; i >= 0; --i) {
    const bool ok = i < nv;
    const float d = z[i] - mx;
    const float e = ok ? __expf(d) : 0.f;
    S += e;
    T += ok ? e * d : 0.f;
    am = (ok && z[i] == mx) ? vh + i : am;
  }
  *reinterpret_cast<u32x4*>(dst) = u32x4{__float_as_uint(mx), __float_as_uint(S), __float_as_uint(T), (uint32_t)am};
}

// Tiles of the paired kernel: lmhead_pair.hip.
hipError_t launch_lmhead_pair(LmTile tile, const LmArgs& a, hipStream_t s, hipEvent_t ev_stop);

}  // namespace respec
