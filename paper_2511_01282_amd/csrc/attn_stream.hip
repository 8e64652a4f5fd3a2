// Tree-masked attention, bf16: every KV head's tiles over the whole batch as
// one stream per workgroup.
//
// The contract is that of tree_attn_kernel (attention.hip): S^T = K Q^T, online
// softmax with a lazily raised reference maximum, O^T += V^T P^T with P split
// into hi + lo bf16 parts, unnormalised partials (O, m, l) for the split merge.
//
// Work split.  A head's 32-row KV tiles over all sequences of the batch are cut
// into `pieces` intervals of equal cost, one workgroup each, so that neither a
// ragged batch nor an odd split count leaves CUs idle.  pieces * heads * row
// blocks is at most the CU count, one workgroup per CU, with two exceptions:
// more heads * row blocks than CUs have one piece each, and every 256 sequences
// of a larger batch (a slice) have pieces of their own; those workgroups follow
// one another.  A piece is a list of segments (sequence, tile range); a
// sequence's partials are numbered piece + sequence, which is unique and compact
// (consecutive sequences share at most one piece).
//
// Stream.  A ring of S LDS slots (32 rows of K and of V each) is filled by DMA
// (global_load_lds, 16 bytes per lane).  A segment is a sequence of passes, one
// barrier each: first its query rows (two waves' 32 rows per slot), then its KV
// tiles, TP = KG * TPG per pass (the remainder in the first one).  The slots of a
// pass are requested again as soon as the next pass's barrier shows that they
// are done with, and the ring runs on across segments: the next segment's
// queries and tiles are in flight while this one ends, and nothing but the DMA
// requests waits on memory.  The first PW waves request the K and V halves of
// every slot and wait, before a pass's barrier, until only newer slots' requests
// are pending.
//
// Waves.  wr row waves own 32 query rows each, (node, head-in-group) pairs; KG
// key groups of wr waves take the tiles of a pass in turn, and at a segment's
// end hand their (m, l, O) to group 0 through the slots of the last pass.
// A pass of four tiles with one or two key groups: the barriers are half as
// many as with one tile per group, and the waves of a SIMD drift apart inside
// a pass by themselves (65 nodes of 32 heads, attention layer over 16384 rows:
// 66.0 us with one tile per group, 63.6 with two; 32 heads of 64 columns 47.2
// and 41.6).  Holding waves 4-7 half a tile behind instead costs registers and
// gains nothing: 12 sequences of 24-61 nodes on 8 heads of 4 over 500-16000
// rows 121.0 with it, 114.5 without.
//
// What bounds it: with 8 row waves (256 rows) the arithmetic of two waves per
// SIMD, 1.3 us per tile of which the matrix products are 0.7 (a DMA-less copy
// takes the same), with one or two row waves the DMA ring.  Against per-sequence
// splits of 32-key, 16-row products (the earlier kernel): 12 sequences of 24-61
// nodes over 500-16000 rows, 8 KV heads of 4: 323 -> 120 us (its two splits per
// sequence left the longest sequence alone on 16 CUs); 32 sequences of 8-48 nodes
// over 300-4000 rows, 32 heads: attention + merge 200 -> 194 us (4.2 TB/s).  One
// tree of 64 nodes over 32768 rows, 8 heads of 4, gains little: 67.6 us then,
// 62.4-65.3 in four traces of this kernel on other cards.
//
// Matrix cores: v_mfma_f32_32x32x16_bf16.  A lane then holds 16 scores of ONE
// query row (the other 16 keys of the tile are in lane ^ 32), so the row
// maximum takes 8 three-operand maxima and one lane swap, and the reference
// maximum, its test and its rescale exist once per lane.
#include "attention.hpp"
#include "common.hpp"
#include "kernels.hpp"

namespace respec {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Headroom of the lazily raised softmax reference maximum (log2 units).
constexpr float kLazyMargin = 8.f;
constexpr int kMaxSegs = kStreamSlice;  // a piece holds at most one segment per sequence of its slice
constexpr int kParentAreas = 8;         // segments whose parents are in LDS at once

struct Seg {
  int b, node0, n_nodes, L, lo, hi, tiles, pad;
};

template <int D>
__device__ __forceinline__ int k_swz(int r) {  // chunk swizzle of K and query rows
  return D == 128 ? (r & 15) : ((r >> 1) & 7);
}
template <int D>
__device__ __forceinline__ int v_swz(int r) {  // ... of V rows: a half-wave of a transposing read (4 rows of
  return D == 128 ? ((r & 3) << 2) : ((r & 2) << 1);  // 64 bytes) touches every bank once
}

__device__ __forceinline__ f32x16 mma32(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
// Maximum as v_med3 with +inf (the operands are no signalling NaNs; fmaxf would
// canonicalise each first).  A compiler-visible instruction: it carries the
// wait states that the matrix cores' results and the lane swaps need.
__device__ __forceinline__ float max2(float a, float b) {
  return __builtin_amdgcn_fmed3f(a, b, __builtin_huge_valf());
}

// N DMA requests of 1 KB (global_load_lds_dwordx4, 16 bytes per lane): request i
// moves 16 bytes per lane from base + off[i] + 1024 i into LDS at dst + 1024 i
// (the instruction's offset counts on both sides; dst and base uniform).
template <int N>
__device__ __forceinline__ void dma16(uint32_t dst, uint64_t base, const uint32_t* off) {
  uint32_t saved;
  dst = __builtin_amdgcn_readfirstlane(dst);
  base = uniform_u64(base);
  if constexpr (N == 2) {
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
        "global_load_lds_dwordx4 %2, %4\n\t"
        "global_load_lds_dwordx4 %3, %4 offset:1024\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "s"(dst), "v"(off[0]), "v"(off[1]), "s"(base)
        : "memory");
  } else {
    static_assert(N == 4, "requests per producer and slot");
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
        "global_load_lds_dwordx4 %2, %6\n\t"
        "global_load_lds_dwordx4 %3, %6 offset:1024\n\t"
        "global_load_lds_dwordx4 %4, %6 offset:2048\n\t"
        "global_load_lds_dwordx4 %5, %6 offset:3072\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "s"(dst), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base)
        : "memory");
  }
}
__device__ __forceinline__ void dma4(uint32_t dst, uint64_t base, uint32_t off) {  // 4 bytes per lane
  uint32_t saved;
  dst = __builtin_amdgcn_readfirstlane(dst);
  base = uniform_u64(base);
  asm volatile(
      "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
      "global_load_lds_dword %2, %3\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(dst), "v"(off), "s"(base)
      : "memory");
}

// Ancestor-or-self bitset of this lane's query node, walked up the parents in
// LDS (a walk ends at the root or at an invalid parent; parents strictly decrease).
__device__ __forceinline__ u32x4 ancestor_set(const int32_t* par, int node, int n_nodes) {
  u32x4 anc = {0u, 0u, 0u, 0u};
  int x = node;
  for (int step = 0; step < kMaxNodes; ++step) {
    const uint32_t bit = x >= 0 ? 1u << (x & 31) : 0u;
    const int w = x >> 5;
    anc[0] |= w == 0 ? bit : 0u;
    anc[1] |= w == 1 ? bit : 0u;
    anc[2] |= w == 2 ? bit : 0u;
    anc[3] |= w == 3 ? bit : 0u;
    const int p = par[max(x, 0)];
    x = (x > 0 && p >= 0 && p < x) ? p : -1;
    if (!__any(x >= 0)) break;
  }
  return anc;
}

template <int D, int S, int KG, int TPG>
struct StreamShape {
  static constexpr int TP = KG * TPG;                    // slots per pass
  static constexpr int PW = 4;                           // producer waves
  static constexpr int kHalf = kKvTile * D * 2;          // bytes of a K or V half slot
  static constexpr int kSlot = 2 * kHalf;
  static constexpr int NR = kHalf / 1024 / (PW / 2);     // DMA requests of a producer per slot
  static constexpr int kMaxWr = KG == 1 ? 8 : (KG == 2 ? 4 : 2);
  static constexpr int kPar = S * kSlot;                 // parents: kParentAreas x kMaxNodes int32
  static constexpr int kSeg = kPar + kParentAreas * kMaxNodes * 4;
  static constexpr int kMl = kSeg + kMaxSegs * (int)sizeof(Seg);  // (m, l) handed to group 0
  static constexpr int kCtl = kMl + (KG - 1) * kMaxWr * 64 * 8;
  static constexpr int kLds = kCtl + 16;
  static_assert(S > TP && S > 4 && 7 * NR <= 63, "a pass is part of the ring; vmcnt holds at most 63 pending requests");
  // the groups with tiles hand half of their columns over through the half slots of the last pass (c tiles,
  // c >= the groups with tiles)
  static_assert((KG - 1) * kMaxWr <= 2 * KG, "hand-over space");
  static_assert(S / 2 + 2 <= kParentAreas, "parents of every segment in flight (at least two slots each)");
  static_assert(kLds <= 163840, "LDS of a CU");
};

template <int D, int S, int KG, int TPG>
__global__ __launch_bounds__(512) void tree_attn_stream_kernel(AttnArgs a) {
  using G = StreamShape<D, S, KG, TPG>;
  constexpr int NR = G::NR;
  constexpr int TP = G::TP;
  constexpr int PW = G::PW;
  constexpr int KS = D / 16;   // 16-element slices of a head row
  constexpr int DB = D / 32;   // 32-column blocks of O
  constexpr int DH = DB / 2;   // ... per hand-over round
  constexpr int CPR = D / 8;   // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;  // rows per DMA request

  extern __shared__ __align__(1024) unsigned char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)smem;
  Seg* segs = reinterpret_cast<Seg*>(smem + G::kSeg);
  int* ctl = reinterpret_cast<int*>(smem + G::kCtl);

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = KG == 1 ? 0 : wave / a.wr, rw = KG == 1 ? wave : wave % a.wr;
  const int r32 = lane & 31, hi = lane >> 5;
  const int g = blockIdx.y / a.n_rowblk, rb = blockIdx.y % a.n_rowblk;
  const int row_wg = rb * a.rows_per_wg;
  const int b0 = blockIdx.z * kStreamSlice, nb = min(kStreamSlice, a.batch - b0);

  // ---- this piece's segments ----
  // A tile costs 1, or 2 where a SIMD carries two row waves of one key group's
  // tiles.  Piece p of P covers the costs [c(p), c(p + 1)), c(p) = floor(p * total / P),
  // and takes the tiles whose cost begins there.  A piece holds at least one tile
  // per key group and the largest tile cost: then none inside a sequence's range is empty.
  constexpr int kLeast = KG == 1 ? 1 : (KG == 2 ? 1 : 2);  // log2 of a piece's least cost
  const int p = blockIdx.x;
  auto first_tile = [&](long long c0, long long pre, int sh, int tiles) {
    return c0 <= pre ? 0 : (int)min((long long)tiles, (c0 - pre + ((1 << sh) - 1)) >> sh);
  };
  auto span_of = [&](int b) { return a.span + 2 * (((size_t)b * a.n_kv_heads + g) * a.n_rowblk + rb); };
  if (a.batch == 1) {  // one sequence: every wave works it out (no hand-over through LDS)
    const SeqRows sr = seq_rows(a, 0);
    const int rows = sr.n_nodes * a.group - row_wg;
    if (rows <= 0) return;
    const int tiles = (sr.L + sr.n_nodes + kKvTile - 1) / kKvTile;
    const int P = stream_pieces_of_one(a, tiles);
    if (p >= P) return;
    const int q = tiles / P, r = tiles - q * P;
    const int lo = p * q + p * r / P, hi_t = (p + 1) * q + (p + 1) * r / P;
    if (lane == 0) {  // (every wave writes the same words)
      segs[0] = Seg{0, sr.node0, sr.n_nodes, sr.L, lo, hi_t, tiles, 0};
      ctl[0] = 1;
    }
    wave_lds_sync();
  } else {
    if (wave == 0) {
      int tiles[kStreamSlice / 64], sh[kStreamSlice / 64];
      long long pre[kStreamSlice / 64];
      long long total = 0;
#pragma unroll
      for (int c = 0; c < kStreamSlice / 64; ++c) {
        tiles[c] = 0;
        sh[c] = 0;
        pre[c] = 0;
        if (c * 64 < nb) {
          const int i = c * 64 + lane;
          if (i < nb) {
            const SeqRows sr = seq_rows(a, b0 + i);
            const int rows = sr.n_nodes * a.group - row_wg;
            if (rows > 0) {
              tiles[c] = (sr.L + sr.n_nodes + kKvTile - 1) / kKvTile;
              sh[c] = KG == 1 && rows > 128 ? 1 : 0;
            }
          }
          long long incl = (long long)tiles[c] << sh[c];
          const long long own = incl;
#pragma unroll
          for (int o = 1; o < 64; o <<= 1) {
            const long long y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
          }
          pre[c] = total + incl - own;
          total += __shfl(incl, 63, 64);
        }
      }
      const int P = (int)min((long long)a.pieces, max(1ll, total >> kLeast));
      int n = 0;
      if (p < P) {
        const long long q = total / P;
        const int r = (int)(total - q * P);
        const long long c0 = p * q + p * r / P, c1 = (p + 1) * q + (p + 1) * r / P;
#pragma unroll
        for (int c = 0; c < kStreamSlice / 64; ++c) {
          if (c * 64 < nb) {
            const int lo = first_tile(c0, pre[c], sh[c], tiles[c]), hi_t = first_tile(c1, pre[c], sh[c], tiles[c]);
            const uint64_t mask = __ballot(lo < hi_t);
            if (lo < hi_t) {
              const int at =
                  n + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
              const int b = b0 + c * 64 + lane;
              const SeqRows sr = seq_rows(a, b);
              segs[at] = Seg{b, sr.node0, sr.n_nodes, sr.L, lo, hi_t, tiles[c], 0};
              if (lo == 0) span_of(b)[0] = p;
              if (hi_t == tiles[c]) span_of(b)[1] = p;
            }
            n += __builtin_popcountll(mask);
          }
        }
      }
      if (lane == 0) ctl[0] = n;
    }
    __syncthreads();
  }
  const int n_seg = __builtin_amdgcn_readfirstlane(ctl[0]);
  if (n_seg == 0) return;

  auto seg_word = [&](int s, int w) { return __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(segs + s)[w]); };

  auto tile_row = [&](int lo, int n_t, int rot, int t) {
    const int x = t + rot;
    return (lo + (x >= n_t ? x - n_t : x)) * kKvTile;
  };

  // ---- producers (waves 0 .. PW-1): position after position into slot after slot ----
  // wave w requests part w / 2 of the K (w even) or V (w odd) half of every slot
  const bool v_half = wave & 1;
  const int row_p = (wave >> 1) * NR * RPI + lane / CPR;  // this lane's row of the part's first request
  const char* cache = reinterpret_cast<const char*>(v_half ? a.v_cache : a.k_cache);
  uint32_t toff[NR];  // source offsets within a whole tile (less 1024 per request)
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int r = row_p + q * RPI, pos = lane % CPR;
    toff[q] = (uint32_t)((wave >> 1) * NR * 1024 + (lane / CPR) * D * 2 + (pos ^ (v_half ? v_swz<D>(r) : k_swz<D>(r))) * 16);
  }
  struct {
    int seg, pos, n_q, n_t, node0, rows, L, t_rows, lo, rot;
    uint64_t base;  // row 0 of the sequence's half (K or V) of this head
  } pr;
  int p_slot = 0;
  int produced = 0, consumed = 0;  // slots requested so far, and consumed by the passes before this one
  auto p_open = [&](int s) {  // (s < n_seg)
    pr.seg = s;
    pr.pos = 0;
    const int b = seg_word(s, 0), n_nodes = seg_word(s, 2);
    pr.node0 = seg_word(s, 1);
    pr.L = seg_word(s, 3);
    pr.lo = seg_word(s, 4);
    pr.n_t = seg_word(s, 5) - pr.lo;
    pr.rot = tile_rotation(pr.n_t);
    pr.t_rows = pr.L + n_nodes;
    pr.rows = n_nodes * a.group - row_wg;
    const int wr_live = min(a.wr, (pr.rows + 31) >> 5);
    pr.n_q = (wr_live + 1) >> 1;
    pr.base = reinterpret_cast<uint64_t>(cache) + ((uint64_t)b * a.n_kv_heads + g) * (uint64_t)a.kv_cap * (D * 2);
  };
  auto produce = [&]() {
    if (pr.seg < n_seg) {
      const uint32_t dst =
          lds0 + (uint32_t)(p_slot * G::kSlot) + (v_half ? (uint32_t)G::kHalf : 0u) + (uint32_t)((wave >> 1) * NR * 1024);
      p_slot = p_slot + 1 == S ? 0 : p_slot + 1;
      ++produced;
      const int t = pr.pos - pr.n_q;
      if (t < 0) {
        // query rows of row wave q_wave: row r is (node, head-in-group)
        const int q_wave = 2 * pr.pos + (v_half ? 1 : 0);
        if (pr.pos == 0 && wave == 0 && (pr.lo + pr.n_t) * kKvTile > pr.L) {  // the tree's own rows: parents
          const uint64_t pb = reinterpret_cast<uint64_t>(a.parent + pr.node0);
          const uint32_t area = lds0 + G::kPar + (uint32_t)(pr.seg % kParentAreas) * (kMaxNodes * 4);
          const int last = pr.t_rows - pr.L - 1;
          dma4(area, pb, (uint32_t)min(lane, last) * 4);
          dma4(area + 256, pb, (uint32_t)min(lane + 64, last) * 4);
        }
        {
          // rows past the last, and the second half of an odd last slot: that row again (never merged)
          // (base - 8192: an offset less its request's 1024 q may be negative)
          const uint64_t qb = reinterpret_cast<uint64_t>(a.hidden) +
                              ((uint64_t)pr.node0 * a.hidden_size + (uint64_t)g * a.group * D) * 2 - 8192;
          uint32_t off[NR];
#pragma unroll
          for (int q = 0; q < NR; ++q) {
            const int r = row_p + q * RPI, pos = lane % CPR;
            const int rr = row_wg + min(32 * q_wave + r, pr.rows - 1);
            const int node = rr / a.group, hh = rr - node * a.group;
            off[q] = ((uint32_t)node * (uint32_t)a.hidden_size + (uint32_t)(hh * D)) * 2 + (uint32_t)(pos ^ k_swz<D>(r)) * 16 +
                     8192u - 1024u * q;
          }
          dma16<NR>(dst, qb, off);
        }
      } else {
        const int t0 = tile_row(pr.lo, pr.n_t, pr.rot, t);
        const uint64_t tb = pr.base + (uint64_t)t0 * (D * 2);
        if (t0 + kKvTile <= pr.t_rows) {
          dma16<NR>(dst, tb, toff);
        } else {  // rows past the sequence's last row: that row (masked, or weighted by zero)
          const int last = pr.t_rows - 1 - t0;
          uint32_t off[NR];
#pragma unroll
          for (int q = 0; q < NR; ++q)
            off[q] = toff[q] + 8192u - (uint32_t)(max(row_p + q * RPI - last, 0) * D * 2);
          dma16<NR>(dst, tb - 8192, off);
        }
      }
      if (++pr.pos == pr.n_q + pr.n_t) {
        if (pr.seg + 1 < n_seg)
          p_open(pr.seg + 1);
        else
          pr.seg = n_seg;
      }
    }
  };
  if (wave < PW) {
    p_open(0);
#pragma unroll 1
    for (int i = 0; i < S; ++i) produce();
  }

  // ---- consumer ----
  int s_next = 0;   // slot of the next pass's first position
  int s_cur = 0;    // ... of the current pass's
  int c_cur = 0;    // slots of the current pass
  // Start of a pass of c slots: they have landed (a producer waits until only the
  // requests of newer slots are pending; fewer where a parents request or a
  // partial's store is among them) and every wave is done with the previous
  // pass, whose slots are requested again.
  auto begin_pass = [&](int c) {
    if (wave < PW) {
      switch (produced - consumed - c) {
        case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
        case 1: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NR) : "memory"); break;
        case 2: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NR) : "memory"); break;
        case 3: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * NR) : "memory"); break;
        case 4: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * NR) : "memory"); break;
        case 5: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(5 * NR) : "memory"); break;
        case 6: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(6 * NR) : "memory"); break;
        default: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(7 * NR) : "memory"); break;  // 7 or more
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (wave < PW) {
#pragma unroll 1
      for (int q = 0; q < c_cur; ++q) produce();
    }
    consumed += c;
    c_cur = c;
    s_cur = s_next;
    s_next += c;
    s_next = s_next >= S ? s_next - S : s_next;
  };
  auto slot_of = [&](int q) {
    const int s = s_cur + q;
    return s >= S ? s - S : s;
  };

  for (int sg = 0; sg < n_seg; ++sg) {
    const int b = seg_word(sg, 0), n_nodes = seg_word(sg, 2), L = seg_word(sg, 3), lo = seg_word(sg, 4),
              n_t = seg_word(sg, 5) - lo;
    const int rows = n_nodes * a.group - row_wg;
    const int wr_live = min(a.wr, (rows + 31) >> 5);
    const bool live = rw < wr_live;  // this wave owns a live row
    const int t_rows = L + n_nodes;
    u32x4 qf[KS];
    begin_pass((wr_live + 1) >> 1);
    if (live) {
      const unsigned char* qs = smem + slot_of(rw >> 1) * G::kSlot + (rw & 1) * G::kHalf + r32 * D * 2;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        qf[ks] = *reinterpret_cast<const u32x4*>(qs + (((2 * ks + hi) ^ k_swz<D>(r32)) << 4));
    }
    const bool tail = (lo + n_t) * kKvTile > L;  // the segment reaches the tree's own rows
    u32x4 anc = {0u, 0u, 0u, 0u};
    if (tail && live) {
      const int rr = 32 * rw + r32;
      const int node = rr < rows ? (row_wg + rr) / a.group : -1;
      anc = ancestor_set(reinterpret_cast<const int32_t*>(smem + G::kPar) + (sg % kParentAreas) * kMaxNodes, node,
                         n_nodes);
    }
    float m_run = kNegInf, l_run = 0.f;
    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = f32x16{};

    // passes of TP tiles, the first one of the remainder (so that the last is whole, or the only one)
    const int rem = n_t % TP, rot = tile_rotation(n_t);
    int c = rem ? rem : TP;
    for (int j = 0; j < n_t; j += c, c = TP) {
      begin_pass(c);
#pragma unroll
      for (int u = 0; u < TPG; ++u) {
        const int t = j + KG * u + grp;
        if (KG * u + grp < c && live) {
          const unsigned char* kt = smem + slot_of(KG * u + grp) * G::kSlot;
          // S^T = K Q^T: lane holds, of query row r32, keys 8 (i / 4) + 4 hi + i % 4
          f32x16 s = f32x16{};
          {
            const unsigned char* kr = kt + r32 * D * 2;
            u32x4 kf[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
              kf[ks] = *reinterpret_cast<const u32x4*>(kr + (((2 * ks + hi) ^ k_swz<D>(r32)) << 4));
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) s = mma32(kf[ks], qf[ks], s);
          }
          // V^T fragments: A operand rows d = 32 db + (lane & 31), keys 16 k2 + {0..3, 8..11} + 4 hi, by
          // transposing reads (lane j of a 16-lane group addresses row + j / 4, columns 4 (j % 4) ..
          // and receives column j of the four rows)
          u32x4 vf[DB][2];
          {
            typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
            typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
            const int lr = lane & 15, dh = (lane >> 4) & 1;
            const int r = 4 * hi + lr / 4;  // rows + 8 and + 16 share the swizzle
            const unsigned char* vr = kt + G::kHalf + r * D * 2;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
              const int col = 32 * db + 16 * dh + 4 * (lr % 4);
              const unsigned char* p = vr + ((col >> 3) ^ v_swz<D>(r)) * 16 + (col & 7) * 2;
#pragma unroll
              for (int k2 = 0; k2 < 2; ++k2) {
                const u32x2 h0 = __builtin_bit_cast(
                    u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + (16 * k2) * D * 2)));
                const u32x2 h1 = __builtin_bit_cast(
                    u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + (16 * k2 + 8) * D * 2)));
                vf[db][k2] = u32x4{h0.x, h0.y, h1.x, h1.y};
              }
            }
          }
          const int t0 = tile_row(lo, n_t, rot, t);
          if (t0 + kKvTile > L) {  // tree rows (or the end of the sequence) in this tile
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const int p = t0 + 8 * (i >> 2) + 4 * hi + (i & 3);
              const int ai = p - L;
              const uint32_t word = ai < 64 ? (ai < 32 ? anc[0] : anc[1]) : (ai < 96 ? anc[2] : anc[3]);
              const bool vis = p < t_rows && (ai < 0 || ((word >> (ai & 31)) & 1u));
              s[i] = vis ? s[i] : kNegInf;
            }
          }
          // row maximum: the first one is compiler-visible and every other is ordered behind it (the
          // wait states behind the matrix product are inserted before visible instructions only)
          float x = max2(s[14], s[15]);
          asm("" : "+v"(x), "+v"(s));
          x = max3(x, s[0], s[1]);
          const float x1 = max3(s[2], s[3], s[4]), x2 = max3(s[5], s[6], s[7]), x3 = max3(s[8], s[9], s[10]);
          x = max3(x, s[11], max3(s[12], s[13], x1));
          x = max2(x, max2(x2, x3));
          const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
          const float tmax = max2(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * a.scale_log2;
          // m_run is a reference maximum: raised only when a score exceeds it by more than
          // kLazyMargin (so p <= 2^kLazyMargin); the accumulators are rescaled only then
          const bool raise = tmax > m_run + kLazyMargin;
          if (__any(raise)) {
            const float mn = raise ? tmax : m_run;
            const float alpha = raise && m_run != kNegInf ? __builtin_amdgcn_exp2f(m_run - mn) : 1.f;
            l_run *= alpha;
            m_run = mn;
#pragma unroll
            for (int db = 0; db < DB; ++db) o[db] *= alpha;
          }
          const float mb = m_run == kNegInf ? 0.f : m_run;
          u32x4 phi[2], plo[2];
          float ps = 0.f;
#pragma unroll
          for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
              const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * k2 + 2 * w], a.scale_log2, -mb));
              const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * k2 + 2 * w + 1], a.scale_log2, -mb));
              ps += p0;
              ps += p1;
              const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{p0, p1}, bf16x2));
              const float r0 = p0 - __uint_as_float(h << 16), r1 = p1 - __uint_as_float(h & 0xFFFF0000u);
              phi[k2][w] = h;
              plo[k2][w] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{r0, r1}, bf16x2));
            }
          l_run += ps;
#pragma unroll
          for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
              o[db] = mma32(vf[db][k2], phi[k2], o[db]);
              o[db] = mma32(vf[db][k2], plo[k2], o[db]);
            }
        }
      }
    }

    // ---- segment end: hand-over to key group 0, partials ----
    l_run += xchg<5>(l_run);
    const int pb = blockIdx.z * (a.pieces - 1) + blockIdx.x + b;  // this segment's partial block of the head
    const size_t prow = ((size_t)blockIdx.y * a.part_blocks + pb) * a.part_rows + 32 * rw + r32;
    const bool store = live && grp == 0 && 32 * rw + r32 < rows;
    float w_own = 1.f, w_k[KG > 1 ? KG - 1 : 1];
    if constexpr (KG > 1) {
      // O = sum_k 2^(m_k - M) O_k, l likewise, M = max_k m_k, half of the columns per round
      float2* ml = reinterpret_cast<float2*>(smem + G::kMl);
#pragma unroll
      for (int rd = 0; rd < 2; ++rd) {
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (live && grp > 0 && grp < n_t) {
          const int h = (grp - 1) * a.wr + rw;
          f32x4* xo = reinterpret_cast<f32x4*>(smem + slot_of(h >> 1) * G::kSlot + (h & 1) * G::kHalf) + lane;
#pragma unroll
          for (int db = 0; db < DH; ++db)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              xo[(db * 4 + q) * 64] = f32x4{o[rd * DH + db][4 * q], o[rd * DH + db][4 * q + 1],
                                            o[rd * DH + db][4 * q + 2], o[rd * DH + db][4 * q + 3]};
          if (rd == 0) ml[h * 64 + lane] = make_float2(m_run, l_run);
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (live && grp == 0) {
          if (rd == 0) {
            float mk[KG - 1], M = m_run;
#pragma unroll
            for (int k = 0; k < KG - 1; ++k) {
              mk[k] = k + 1 < n_t ? ml[(k * a.wr + rw) * 64 + lane].x : kNegInf;
              M = fmaxf(M, mk[k]);
            }
            w_own = m_run == kNegInf ? 0.f : __builtin_amdgcn_exp2f(m_run - M);
            l_run *= w_own;
#pragma unroll
            for (int k = 0; k < KG - 1; ++k) {
              w_k[k] = mk[k] == kNegInf ? 0.f : __builtin_amdgcn_exp2f(mk[k] - M);
              if (k + 1 < n_t) l_run += w_k[k] * ml[(k * a.wr + rw) * 64 + lane].y;
            }
            m_run = M;
          }
#pragma unroll
          for (int db = 0; db < DH; ++db)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              f32x4 v;
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = o[rd * DH + db][4 * q + e] * w_own;
#pragma unroll
              for (int k = 0; k < KG - 1; ++k) {
                if (k + 1 >= n_t) break;  // (uniform) groups without a tile hand nothing over
                const int h = k * a.wr + rw;
                const f32x4* xi =
                    reinterpret_cast<const f32x4*>(smem + slot_of(h >> 1) * G::kSlot + (h & 1) * G::kHalf) + lane;
                v += xi[(db * 4 + q) * 64] * w_k[k];
              }
              if (store)
                *reinterpret_cast<f32x4*>(a.part_o + prow * D + 32 * (rd * DH + db) + 8 * q + 4 * hi) = v;
            }
        }
      }
    } else if (store) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<f32x4*>(a.part_o + prow * D + 32 * db + 8 * q + 4 * hi) =
              f32x4{o[db][4 * q], o[db][4 * q + 1], o[db][4 * q + 2], o[db][4 * q + 3]};
    }
    if (store && hi == 0) {
      a.part_m[prow] = m_run;
      a.part_l[prow] = l_run;
    }
  }
  // the requests past the last pass land before the workgroup's LDS is released
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int D, int S, int KG, int TPG>
hipError_t go(bool launch, dim3 grid, int threads, const AttnArgs& a, hipStream_t s, hipEvent_t ev_start) {
  using G = StreamShape<D, S, KG, TPG>;
  if (!launch)
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&tree_attn_stream_kernel<D, S, KG, TPG>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, G::kLds);
  if (a.wr < 1 || a.wr > G::kMaxWr || threads != 64 * a.wr * KG || threads < 64 * G::PW) return hipErrorInvalidValue;
  return launch_k(tree_attn_stream_kernel<D, S, KG, TPG>, grid, dim3(threads), G::kLds, s, ev_start, nullptr, a);
}

template <int D>
hipError_t go_kg(int kg, bool launch, dim3 grid, int threads, const AttnArgs& a, hipStream_t s, hipEvent_t ev_start) {
  switch (kg) {
    case 1: return go<D, 9, 1, 4>(launch, grid, threads, a, s, ev_start);
    case 2: return go<D, 9, 2, 2>(launch, grid, threads, a, s, ev_start);
    case 4: return go<D, 9, 4, 1>(launch, grid, threads, a, s, ev_start);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_tree_attn_stream(int head_dim, int kg, dim3 grid, const AttnArgs& a, hipStream_t s,
                                   hipEvent_t ev_start) {
  const int threads = 64 * a.wr * kg;
  if (head_dim == 128) return go_kg<128>(kg, true, grid, threads, a, s, ev_start);
  if (head_dim == 64) return go_kg<64>(kg, true, grid, threads, a, s, ev_start);
  return hipErrorInvalidValue;
}

hipError_t set_tree_attn_stream_lds_limit(int head_dim) {
  const AttnArgs none{};
  for (int kg : {1, 2, 4}) {
    const hipError_t e = head_dim == 128 ? go_kg<128>(kg, false, dim3(), 0, none, nullptr, nullptr)
                                         : go_kg<64>(kg, false, dim3(), 0, none, nullptr, nullptr);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace respec
