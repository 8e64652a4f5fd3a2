// LM head for more token rows than one tile of the kernels in lmhead.hip (bf16):
// tiles of VR = 64 WV vocabulary rows by MT = 16 NB WT token rows (WT = 8 / WV),
// logits and tile statistics as there.
//
// What bounds it: matrix-core time, and at a steady load the card's power (256 x 256
// tiles over 128256 x 4096 columns by 510 rows: 435 us for the first steps after a
// pause, 455-490 us later; the 256-token by 128-row tiles of one barrier per step
// took 560 and 630-650 us).  At 256 tokens by 128 vocabulary rows a CU's LDS moves
// 176 KB per 64-column step (128 KB of fragments, 48 KB of DMA), more cycles than
// the step's products; at 256 x 256 it moves 256 KB for twice the products, as many
// cycles as the products take.  (One round of the former is bound by what a CU takes
// in and stays in the kernel of one barrier per step: lm_tile.)
//
//   - Eight waves, two per SIMD, in two groups of four (waves w and w + 4 share a
//     SIMD).  A phase is a load part (fragments from LDS, DMA requests, the wait for
//     the next phase's rows) and a product part (both W halves times one token half),
//     each ended by a workgroup barrier; group 1 runs one part behind group 0, so
//     that on every SIMD one wave's products run under the other's loads.  (Both
//     groups in step: 600 against 505 us with four phases per step; two phases per
//     step instead of four, half the barriers: 475.)
//   - Group 0 requests the W rows, group 1 the x rows, in rings of their own (SW and
//     SX steps), so that a wait for x, which comes from L2, does not wait for the
//     newer W requests, which come from HBM.  A ring slot is requested again one
//     phase (x) or two (W) after its last read.
//   - Requests are spread over both phases: a wave that issues all of a step's
//     requests at once waits on the CU's address path (435 against 455 us; in a form
//     of four waves with 128 x 128 products each, 155 against 120 us per tile).
//   - v_mfma_f32_16x16x32_bf16: 3-4 % faster than 32x32x16 here.
//   - Stage rows as in lmhead_gemm_kernel (128 bytes, chunk c of row r at c ^ (r >> 1 & 7)).
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "lmhead.hpp"

namespace respec {
namespace {

template <int WV_, int NB, int SW_, int SX_>
struct PairShape {
  static constexpr int WV = WV_, WT = 8 / WV_, SW = SW_, SX = SX_;
  static constexpr int VR = 64 * WV, MT = 16 * NB * WT;
  static constexpr int NB0 = (NB + 1) / 2, NB1 = NB / 2;            // token blocks per wave in each half
  static constexpr int M0 = 16 * NB0 * WT;                          // token rows of the first half
  static constexpr int kW = VR * kGmStep, kX = MT * kGmStep;        // bytes per stage
  static constexpr int kXBase = SW * kW;
  static constexpr int RW = VR / 64;                                // DMA requests per W wave and half
  static constexpr int RX0 = NB0 * WT / 2, RX1 = NB1 * WT / 2;      // ... per x wave and half
  static constexpr int kTileRowB = VR * 4 + 16;                     // LDS row stride of the logit tile
  static constexpr int kRing = SW * kW + SX * kX;
  static constexpr int kLds = kRing > M0 * kTileRowB ? kRing : M0 * kTileRowB;
  static_assert(kLds <= 163840 && SW >= 3 && SW <= 4 && SX >= 2 && SX <= 4, "LDS of a CU");
  static_assert((NB0 * WT) % 2 == 0 && (NB1 * WT) % 2 == 0, "every x wave issues whole DMA requests");
};

// Wait until at most the requests of k newer regions are pending (their sizes alternate F, S, F, ...).
template <int F, int S>
__device__ __forceinline__ void wait_newer(int k) {
  switch (k) {
    case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    case 1: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(F) : "memory"); break;
    case 2: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(F + S) : "memory"); break;
    case 3: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * F + S) : "memory"); break;
    case 4: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * F + 2 * S) : "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * F + 2 * S) : "memory"); break;
  }
}

template <int WV_, int NB, int SW_, int SX_>
__global__ __launch_bounds__(64 * kGmWaves) void lmhead_pair_kernel(LmArgs a) {
  using G = PairShape<WV_, NB, SW_, SX_>;
  constexpr int WV = G::WV, WT = G::WT, SW = G::SW, SX = G::SX, VR = G::VR, MT = G::MT;
  __shared__ __align__(1024) unsigned char sm[G::kLds];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)sm;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave >> 2, w4 = wave & 3;
  const int lr = lane & 15, lg = lane >> 4;
  const int n_mt = a.n_mtiles;
  const int id = blockIdx.x;
  const int g8 = id / (8 * n_mt), rem = id % (8 * n_mt);
  const int vt = g8 * 8 + rem % 8, mt = rem / 8;  // the M tiles of a vocabulary tile share an XCD
  if (vt * VR >= a.vocab) return;
  const int v0 = vt * VR;
  const int m0 = mt * MT;
  const size_t row_bytes = (size_t)a.hidden_size * 2;
  const int n = (int)(row_bytes / kGmStep);  // steps; >= 4 (checked)
  const int rot = ((vt >> 3) & 3) * (n / 4);  // start of the K walk (lmhead_gemm_kernel)

  // DMA sources: waves 0-3 request W, waves 4-7 x; request j of half h covers 8 rows
  constexpr int RMAX = G::RW > G::RX0 ? G::RW : G::RX0;
  uint32_t off[2][RMAX];
  const int pos = lane & 7;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < RMAX; ++j) {
      const int per = grp == 0 ? G::RW : (h == 0 ? G::RX0 : G::RX1);
      const int base = grp == 0 ? h * (VR / 2) : h * G::M0;
      const int r = base + 8 * (w4 * per + j) + (lane >> 3);
      const int top = grp == 0 ? a.vocab - 1 - v0 : a.m_rows - 1 - m0;  // rows past the end: that row, not stored
      off[h][j] = (uint32_t)((size_t)min(r, top) * row_bytes + ((pos ^ ((r >> 1) & 7)) * 16));
    }
  const uint64_t src = grp == 0 ? reinterpret_cast<uint64_t>(a.w) + (uint64_t)v0 * row_bytes
                                : reinterpret_cast<uint64_t>(a.x) + (uint64_t)m0 * row_bytes;
  // request half h of step c (W waves: ring slot c % SW, x waves: c % SX)
  auto issue = [&](int h, int c, int slot) {
    const int kc = c + rot < n ? c + rot : c + rot - n;
    const uint64_t sb = uniform_u64(src + (uint64_t)kc * kGmStep);
    if (grp == 0) {
      const uint32_t d = lds0 + (uint32_t)(slot * G::kW + h * (VR / 2) * kGmStep + w4 * G::RW * 1024);
#pragma unroll
      for (int j = 0; j < G::RW; ++j) gm_dma(__builtin_amdgcn_readfirstlane(d + j * 1024), sb, off[h][j]);
    } else if (h == 0) {
      const uint32_t d = lds0 + (uint32_t)(G::kXBase + slot * G::kX + w4 * G::RX0 * 1024);
#pragma unroll
      for (int j = 0; j < G::RX0; ++j) gm_dma(__builtin_amdgcn_readfirstlane(d + j * 1024), sb, off[0][j]);
    } else {
      const uint32_t d = lds0 + (uint32_t)(G::kXBase + slot * G::kX + G::M0 * kGmStep + w4 * G::RX1 * 1024);
#pragma unroll
      for (int j = 0; j < G::RX1; ++j) gm_dma(__builtin_amdgcn_readfirstlane(d + j * 1024), sb, off[1][j]);
    }
  };

  const int wv = wave % WV, wt = wave / WV;
  uint32_t kof[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) kof[ks] = (uint32_t)(lr * kGmStep + ((4 * ks + lg) ^ (lr >> 1)) * 16);
  u32x4 af[2][2][2];        // [half][block][slice]
  u32x4 bf[G::NB0][2];      // one half
  f32x4 acc[4][NB];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[i][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto read_a = [&](auto H, int slot) {
    constexpr int h = decltype(H)::value;
    const unsigned char* p = sm + slot * G::kW + (h * (VR / 2) + 32 * wv) * kGmStep;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) af[h][i][ks] = *reinterpret_cast<const u32x4*>(p + 16 * i * kGmStep + kof[ks]);
  };
  auto read_b = [&](auto H, int slot) {
    constexpr int h = decltype(H)::value;
    constexpr int nb = h ? G::NB1 : G::NB0;
    const unsigned char* p = sm + G::kXBase + slot * G::kX + (h * G::M0 + 16 * nb * wt) * kGmStep;
#pragma unroll
    for (int b = 0; b < nb; ++b)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) bf[b][ks] = *reinterpret_cast<const u32x4*>(p + 16 * b * kGmStep + kof[ks]);
  };
  // both W halves times token half hb
  auto mma = [&](auto HB) {
    constexpr int hb = decltype(HB)::value;
    constexpr int nb = hb ? G::NB1 : G::NB0;
    asm volatile("s_barrier\n\ts_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ha = 0; ha < 2; ++ha)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int b = 0; b < nb; ++b)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            acc[2 * ha + i][hb * G::NB0 + b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, af[ha][i][ks]), __builtin_bit_cast(bf16x8, bf[b][ks]),
                acc[2 * ha + i][hb * G::NB0 + b], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
  };
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, 1>;

  if (grp == 0) {
#pragma unroll
    for (int c = 0; c < SW; ++c) {
      issue(0, c, c);
      issue(1, c, c);
    }
    wait_newer<G::RW, G::RW>(2 * SW - 2);
  } else {
#pragma unroll
    for (int c = 0; c < SX; ++c) {
      issue(0, c, c);
      issue(1, c, c);
    }
    wait_newer<G::RX1, G::RX0>(2 * SX - 1);
  }
  asm volatile("s_barrier" ::: "memory");
  if (grp == 1) asm volatile("s_barrier" ::: "memory");  // half a phase behind waves 0-3

  int sw = 0, sx = 0, sw_p = SW - 1, sx_p = SX - 1;  // ring slots of steps c and c - 1
  for (int c = 0; c < n; ++c) {
    // phase 2c
    read_a(H0{}, sw);
    read_a(H1{}, sw);
    read_b(H0{}, sx);
    if (grp == 0) {
      if (c > 0 && c - 1 + SW < n) issue(0, c - 1 + SW, sw_p);
    } else {
      if (c > 0 && c - 1 + SX < n) issue(1, c - 1 + SX, sx_p);
      // the second half of step c
      if (c + SX < n)
        wait_newer<G::RX0, G::RX1>(2 * SX - 2);
      else
        wait_newer<G::RX0, G::RX1>(2 * (n - 1 - c));
    }
    mma(H0{});
    // phase 2c + 1
    read_b(H1{}, sx);
    if (grp == 0) {
      if (c > 0 && c - 1 + SW < n) issue(1, c - 1 + SW, sw_p);
      // both halves of step c + 1
      if (c - 1 + SW < n)
        wait_newer<G::RW, G::RW>(2 * (SW - 2));
      else if (c + 1 < n)
        wait_newer<G::RW, G::RW>(2 * (n - 2 - c));
    } else {
      if (c + SX < n) issue(0, c + SX, sx);
      // the first half of step c + 1
      if (c + SX < n)
        wait_newer<G::RX1, G::RX0>(2 * SX - 2);
      else if (c + 1 < n)
        wait_newer<G::RX1, G::RX0>(2 * (n - 2 - c) + 1);
    }
    mma(H1{});
    sw_p = sw;
    sx_p = sx;
    sw = sw + 1 == SW ? 0 : sw + 1;
    sx = sx + 1 == SX ? 0 : sx + 1;
  }
  if (grp == 0) asm volatile("s_barrier" ::: "memory");

  // logits through LDS, one token half at a time
  const bool vec_ok = (a.vocab & 3) == 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int nb = h ? G::NB1 : G::NB0;
    const int mh = m0 + h * G::M0;
    const int rows = min(16 * nb * WT, a.m_rows - mh);
    if (rows <= 0) break;  // (uniform)
    __syncthreads();       // the ring, or the first half's tile, is no longer read
#pragma unroll
    for (int b = 0; b < nb; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * nb * wt + 16 * b + lr, col = (i >> 1) * (VR / 2) + 32 * wv + 16 * (i & 1) + 4 * lg;
        *reinterpret_cast<f32x4*>(sm + row * G::kTileRowB + col * 4) = acc[i][h * G::NB0 + b];
      }
    __syncthreads();
    {
      constexpr int LPR = VR / 4 < 64 ? VR / 4 : 64;  // lanes per token row of the store
      constexpr int RPW = 64 / LPR;                   // token rows a wave stores per pass
      const int col = 4 * (lane % LPR), vv = v0 + col;
      for (int row = RPW * wave + lane / LPR; row < rows; row += RPW * kGmWaves) {
        const f32x4 q = *reinterpret_cast<const f32x4*>(sm + row * G::kTileRowB + col * 4);
        float* dst = a.logits + (size_t)(mh + row) * a.vocab + vv;
        if (vec_ok && vv + 3 < a.vocab) {
          *reinterpret_cast<f32x4*>(dst) = q;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (vv + e < a.vocab) dst[e] = q[e];
        }
      }
    }
    if (!a.partials) continue;
    for (int u = threadIdx.x; u < 16 * nb * WT * WV; u += 64 * kGmWaves) {
      const int row = u % (16 * nb * WT), hs = u / (16 * nb * WT);
      const int vh = v0 + kLmTileRows * hs;
      if (row < rows && vh < a.vocab)
        tile_row_stats(reinterpret_cast<const f32x4*>(sm + row * G::kTileRowB + hs * kLmTileRows * 4), vh, a.vocab,
                       a.partials + ((size_t)(mh + row) * a.n_vtiles + vh / kLmTileRows) * kTileWords);
    }
  }
}

template <int WV, int NB, int SW, int SX>
hipError_t go(const LmArgs& a, hipStream_t s, hipEvent_t ev_stop) {
  const int n_vt = (a.vocab + 64 * WV - 1) / (64 * WV);
  return launch_k(lmhead_pair_kernel<WV, NB, SW, SX>, dim3((n_vt + 7) / 8 * 8 * a.n_mtiles), dim3(64 * kGmWaves), 0, s,
                  nullptr, ev_stop, a);
}

}  // namespace

hipError_t launch_lmhead_pair(LmTile tile, const LmArgs& a, hipStream_t s, hipEvent_t ev_stop) {
  switch (tile) {
    case LmTile::kPair192x128: return go<2, 3, 4, 3>(a, s, ev_stop);
    case LmTile::kPair128x256: return go<4, 4, 3, 3>(a, s, ev_stop);
    case LmTile::kPair160x256: return go<4, 5, 3, 2>(a, s, ev_stop);
    case LmTile::kPair192x256: return go<4, 6, 3, 2>(a, s, ev_stop);
    case LmTile::kPair224x256: return go<4, 7, 3, 2>(a, s, ev_stop);
    case LmTile::kPair256x256: return go<4, 8, 3, 2>(a, s, ev_stop);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace respec
