// Host side of the respec_verify C ABI: plan creation (tiling choices and
// workspace layout), argument validation and the launch sequence of one
// verification step.  See include/respec_verify.h for the contract.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <new>

#include "../../include/respec_verify.h"
#include "kernels.hpp"

using namespace respec;

struct respec_verify_plan {
  respec_verify_shape s;
  int es;                 // bytes per element of the workload dtype
  int group;              // Hq / Hkv
  // vocabulary statistics: tiles of the LM head and the top-K width (8 or 16)
  int ko, n_vtiles;
  // workspace layout (bytes)
  size_t off_po, off_pm, off_pl, off_x, off_part, off_flag, off_cnt, off_stoch, off_rank;
  size_t off_span;        // first and last piece of each sequence (dead before the LM head's statistics and the flags)
  size_t part_total;      // rows of attention partials that the workspace holds
  size_t n_cnt_seq, total;
  // kernel families (LdsUser bits) whose LDS limits are raised: on their first step (plan creation stays GPU-free)
  mutable std::atomic<uint32_t> lds_ready{0};
};

namespace {

constexpr int kTargetWaves = 1024;  // attention: one wave per SIMD on a 256-CU MI355X

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
// LDS of the register path's workgroup.
size_t row_lds(int es, int head_dim, const RowGeom& g) {
  const int nwaves = g.wr * g.wk;
  // per wave: one row-major, swizzled V tile (bf16) or one transposed, padded V tile (float32)
  const size_t vt = es == 2 ? (size_t)nwaves * kKvTile * head_dim * es
                            : (size_t)nwaves * head_dim * (kKvTile + kVtPad) * es;
  // wave merge: every wave's O lane-major (D/16 x NB blocks of 64 x 16 bytes) plus its m and l
  const size_t merge =
      g.wk > 1 ? (size_t)nwaves * ((size_t)(head_dim / 16) * g.nb * 64 * 16 + (size_t)2 * g.nb * 64 * 4) : 0;
  return std::max(vt, merge);
}
bool aligned(const void* p, size_t n) { return ((uintptr_t)p % n) == 0; }

}  // namespace

extern "C" {

const char* respec_status_string(respec_status st) {
  switch (st) {
    case RESPEC_OK: return "ok";
    case RESPEC_ERR_NULL: return "a required pointer is NULL";
    case RESPEC_ERR_SHAPE: return "sizes out of the supported range or inconsistent";
    case RESPEC_ERR_DTYPE: return "unknown dtype";
    case RESPEC_ERR_PARAM: return "acceptance parameters out of range";
    case RESPEC_ERR_TREE: return "malformed draft tree";
    case RESPEC_ERR_CAPACITY: return "batch, nodes or KV length above the plan's capacity";
    case RESPEC_ERR_HIP: return "HIP call or kernel launch failed";
    case RESPEC_ERR_WORKSPACE: return "workspace missing or not 256-byte aligned";
    case RESPEC_ERR_TOKEN: return "draft token or source tag out of range";
    case RESPEC_ERR_SCRATCH: return "plan needs more workspace or sequences than the static scratch of the allocation-free step holds";
  }
  return "unknown status";
}

respec_status respec_verify_check_tree(const int32_t* parent, int32_t n, int32_t max_depth) {
  if (!parent) return RESPEC_ERR_NULL;
  if (n < 1 || n > RESPEC_MAX_NODES || max_depth < 0) return RESPEC_ERR_SHAPE;
  if (parent[0] != -1) return RESPEC_ERR_TREE;
  int depth[RESPEC_MAX_NODES];
  depth[0] = 0;
  for (int j = 1; j < n; ++j) {
    if (parent[j] < 0 || parent[j] >= j) return RESPEC_ERR_TREE;
    depth[j] = depth[parent[j]] + 1;
    if (depth[j] > max_depth) return RESPEC_ERR_TREE;
  }
  return RESPEC_OK;
}

respec_status respec_verify_create(const respec_verify_shape* shape, respec_verify_plan** out) {
  if (!shape || !out) return RESPEC_ERR_NULL;
  *out = nullptr;
  const respec_verify_shape& s = *shape;
  if (s.dtype != RESPEC_F32 && s.dtype != RESPEC_BF16) return RESPEC_ERR_DTYPE;
  if (s.head_dim != 64 && s.head_dim != 128) return RESPEC_ERR_SHAPE;
  if (s.n_q_heads < 1 || s.n_kv_heads < 1 || s.n_q_heads % s.n_kv_heads != 0) return RESPEC_ERR_SHAPE;
  if ((long long)s.n_q_heads * s.head_dim != s.hidden) return RESPEC_ERR_SHAPE;
  const int es = s.dtype == RESPEC_BF16 ? 2 : 4;
  if (((long long)s.hidden * es) % 512 != 0) return RESPEC_ERR_SHAPE;
  if (s.topk_out < 1 || s.topk_out > RESPEC_MAX_TOPK_OUT || s.vocab < s.topk_out) return RESPEC_ERR_SHAPE;
  if (s.max_batch < 1 || s.max_nodes < 1 || s.max_nodes > RESPEC_MAX_NODES) return RESPEC_ERR_SHAPE;
  if (s.max_depth < 0 || s.max_depth > RESPEC_MAX_DEPTH || s.max_kv_len < 0) return RESPEC_ERR_SHAPE;
  if ((long long)s.max_batch * s.max_nodes > (1ll << 24)) return RESPEC_ERR_SHAPE;

  respec_verify_plan* p = new (std::nothrow) respec_verify_plan();
  if (!p) return RESPEC_ERR_SHAPE;
  p->s = s;
  p->es = es;
  p->group = s.n_q_heads / s.n_kv_heads;

  // attention partials: rows of every split (or piece) of the largest tree
  const int rmax = s.max_nodes * p->group;
  const long long t_cap = (long long)s.max_kv_len + s.max_nodes;
  int rows_per_wg, n_rowblk, slots;
  if (es == 2 && rmax > 32) {
    const int rg = cdiv(rmax, 32), wr = rg < 8 ? rg : 8;
    n_rowblk = cdiv(rg, wr);
    rows_per_wg = 32 * wr;
    slots = clampi(kCUs / (s.n_kv_heads * n_rowblk), 1, cdiv(t_cap, kKvTile));
  } else {
    const RowGeom ge = row_geom(rmax);
    n_rowblk = ge.n_rowblk;
    rows_per_wg = ge.rows_per_wg;
    const int target = kTargetWaves / (ge.threads / 64) / (s.n_kv_heads * n_rowblk);
    slots = max(clampi(target, 1, cdiv(t_cap, kKvTile)), clampi(target, 1, 64));
  }

  p->ko = s.topk_out <= 8 ? 8 : 16;
  p->n_vtiles = cdiv(s.vocab, kLmTileRows);

  // workspace
  const size_t mcap = (size_t)s.max_batch * s.max_nodes;
  const size_t prow = (size_t)s.max_batch * s.n_kv_heads * n_rowblk * slots * rows_per_wg;
  size_t off = 0;
  p->off_po = off; off = align256(off + prow * s.head_dim * 4);
  p->off_pm = off; off = align256(off + prow * 4);
  p->off_pl = off; off = align256(off + prow * 4);
  p->off_x = off; off = align256(off + mcap * s.hidden * es);
  p->part_total = prow;
  const size_t part_bytes = mcap * p->n_vtiles * kTileWords * 4;
  p->off_part = off; off = align256(off + part_bytes);
  p->off_flag = off; off = align256(off + mcap * 4);
  // the streaming kernel's spans lie over the LM head's statistics and the flags, which are written
  // after the split merge has read them (one sequence has none)
  const bool spans = es == 2 && rmax > 32 && s.max_batch > 1;
  p->off_span = p->off_part;
  if (spans) off = std::max(off, align256(p->off_span + (size_t)s.max_batch * s.n_kv_heads * cdiv(rmax, 256) * 8));
  p->n_cnt_seq = s.max_batch;
  p->off_cnt = off; off = align256(off + p->n_cnt_seq * 4);
  p->off_stoch = off; off = align256(off + 2 * mcap * 4);  // stochastic walk: next child, draw
  p->off_rank = off; off = align256(off + mcap * 4);       // rank requests: parent row per node
  p->total = off;

  *out = p;
  return RESPEC_OK;
}

void respec_verify_destroy(respec_verify_plan* plan) { delete plan; }

size_t respec_verify_workspace_bytes(const respec_verify_plan* plan) { return plan ? plan->total : 0; }

respec_status respec_verify_workspace_init(const respec_verify_plan* plan, void* workspace, void* stream) {
  if (!plan) return RESPEC_ERR_NULL;
  if (!workspace || !aligned(workspace, 256)) return RESPEC_ERR_WORKSPACE;
  int32_t* cnt = reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + plan->off_cnt);
  const size_t n = plan->n_cnt_seq;
  return launch_zero_i32(cnt, n, static_cast<hipStream_t>(stream)) == hipSuccess ? RESPEC_OK : RESPEC_ERR_HIP;
}

}  // extern "C"

namespace {

// Streaming attention of a step whose largest tree has n nodes and longest prefix max_kv rows: row
// waves, key groups, row blocks, rows of a partial block, pieces per (head, row block) and slice of
// kStreamSlice sequences.
struct StreamGeom {
  int wr, kg, n_rowblk, part_rows, pieces, slices;
};
StreamGeom stream_geom(const respec_verify_plan* p, int n, int max_kv, int batch) {
  StreamGeom g;
  const int rows = n * p->group, rg = cdiv(rows, 32);
  g.n_rowblk = cdiv(rg, 8);
  g.wr = cdiv(rg, g.n_rowblk);
  // Two row waves in two key groups leave more of the ring in flight per pass than in four
  // and start and end a segment sooner (12 sequences of 8 KV heads and 5-10 nodes over 300-3000
  // rows 24.1 -> 21.4 us; 2 of 32 heads over 200 rows 16.1 -> 12.1).  Four where a 64-column
  // head's tiles, half as large, go by in long streams (32 of 32 heads over 300-1500 rows 78 us
  // in four groups, 88 in two; 3 over 500-1000 rows, 12 tiles per CU, 18.1 and 16.7), and for one
  // sequence.
  const long long tiles = (long long)batch * cdiv((long long)max_kv + n, kKvTile) * p->s.n_kv_heads;
  const bool deep = batch > 1 && (p->s.head_dim == 128 || tiles <= 12ll * kCUs);
  g.kg = g.wr <= 2 && !deep ? 4 : g.wr <= 4 ? 2 : 1;
  g.part_rows = g.n_rowblk == 1 ? rows : g.wr * 32;
  g.slices = cdiv(batch, kStreamSlice);
  const int heads = p->s.n_kv_heads * g.n_rowblk;
  // one workgroup per CU and slice (one per head and row block at least), within the partial rows
  // that the workspace holds
  const long long blocks = (long long)(p->part_total / ((size_t)heads * g.part_rows));
  g.pieces = (int)std::max(1ll, std::min((long long)(kCUs / heads), (blocks - batch) / g.slices + 1));
  return g;
}

constexpr int kMaxDevices = 64;

// Raise the LDS limits of the attention kernels that a path of this dtype and head size may launch, on
// the current device, once (calls into the runtime that also load the kernels: the first step that
// takes the path pays them, not every plan's).
enum LdsUser { kLdsRegister, kLdsShared, kLdsStream };
bool raise_lds_limits(LdsUser user, int dtype, int es, int head_dim) {
  static std::atomic<uint64_t> done[3][2][2];  // [user][dtype][head size], a bit per device
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return false;
  std::atomic<uint64_t>& d = done[user][dtype == RESPEC_BF16][head_dim == 128];
  const uint64_t bit = dev < kMaxDevices ? 1ull << dev : 0;  // (past the last: every plan raises them)
  if (d.load(std::memory_order_acquire) & bit) return true;
  if (user == kLdsRegister) {
    for (int rows : {16, 32}) {  // (both row block counts; more row waves need no more)
      const RowGeom ge = row_geom(rows);
      if (set_tree_attn_lds_limit(dtype, head_dim, ge.nb, row_lds(es, head_dim, ge)) != hipSuccess) return false;
    }
  } else if ((user == kLdsShared ? set_tree_attn_shared_lds_limit(head_dim) : set_tree_attn_stream_lds_limit(head_dim)) !=
             hipSuccess) {
    return false;
  }
  d.fetch_or(bit, std::memory_order_release);
  return true;
}

// One step on workspace `ws` (the plan's layout) with the sequences' completion
// counters at `cnt` (zero between steps).
respec_status step_impl(const respec_verify_plan* plan, const respec_verify_args* args, char* ws, int32_t* cnt,
                        void* stream) {
  const respec_verify_shape& s = plan->s;
  const respec_verify_args& a = *args;
  if (a.stop_after < RESPEC_STOP_ALL || a.stop_after > RESPEC_STOP_STATS) return RESPEC_ERR_PARAM;
  if (a.batch < 0) return RESPEC_ERR_SHAPE;
  if (a.batch > s.max_batch) return RESPEC_ERR_CAPACITY;
  const bool full = a.stop_after == RESPEC_STOP_ALL;
  const bool stats_only = a.stop_after == RESPEC_STOP_STATS;
  const bool vocab_pass = full || stats_only;  // statistics and predicates run
  const bool need_logits = a.stop_after != RESPEC_STOP_ATTN;
  if (vocab_pass) {
    const respec_accept_params& q = a.accept;
    if (q.topk < 1 || q.topk > s.topk_out || !(q.tau >= 0.f) || isinf(q.tau) || q.min_lookahead < 0 ||
        q.max_relaxed < 0 || (q.stochastic != 0 && q.stochastic != 1))
      return RESPEC_ERR_PARAM;
    if (q.stochastic && (!(q.temperature > 0.f) || isinf(q.temperature))) return RESPEC_ERR_PARAM;
    if (q.stochastic && s.vocab > kMaxStochVocab) return RESPEC_ERR_SHAPE;
  }
  const bool stochastic = full && a.accept.stochastic;
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipEvent_t* ev = static_cast<hipEvent_t*>(a.stage_events);
  if (a.batch == 0) {
    if (ev)
      for (int k = 0; k < 4; ++k)
        if (hipEventRecord(ev[k], st) != hipSuccess) return RESPEC_ERR_HIP;
    return RESPEC_OK;
  }
  if (a.max_nodes_in_batch < 1 || a.max_kv_len_in_batch < 0) return RESPEC_ERR_SHAPE;
  if (a.max_nodes_in_batch > s.max_nodes || a.max_kv_len_in_batch > s.max_kv_len) return RESPEC_ERR_CAPACITY;
  if (a.total_nodes < a.batch || (long long)a.total_nodes > (long long)a.batch * a.max_nodes_in_batch)
    return RESPEC_ERR_SHAPE;
  if ((long long)a.kv_capacity < (long long)a.max_kv_len_in_batch + a.max_nodes_in_batch) return RESPEC_ERR_SHAPE;
  if (!a.node_off || !a.kv_len || !a.hidden || !a.k_cache || !a.v_cache || !a.parent) return RESPEC_ERR_NULL;
  if (need_logits && (!a.lm_head || !a.logits)) return RESPEC_ERR_NULL;
  if (vocab_pass && (!a.token || !a.src || !a.max_logit || !a.lse || !a.entropy || !a.argmax || !a.topk_id ||
                     !a.topk_logprob || !a.tok_logprob || !a.flags))
    return RESPEC_ERR_NULL;
  if (full && (!a.leaf_acc_len || !a.path || !a.acc_len || !a.bonus || !a.winner_leaf || !a.seq_status))
    return RESPEC_ERR_NULL;
  if (stochastic && !a.uniform) return RESPEC_ERR_NULL;
  if (stochastic && a.draft_prob && !aligned(a.draft_prob, 16)) return RESPEC_ERR_SHAPE;
  if (!aligned(a.hidden, 16) || !aligned(a.k_cache, 16) || !aligned(a.v_cache, 16) ||
      (need_logits && (!aligned(a.lm_head, 16) || !aligned(a.logits, 16))) || (a.attn_out && !aligned(a.attn_out, 16)))
    return RESPEC_ERR_SHAPE;
  const bool rank = vocab_pass && a.tok_rank != nullptr;

  // ---- tree-masked attention + residual ----
  AttnArgs at;
  at.hidden = a.hidden;
  at.k_cache = a.k_cache;
  at.v_cache = a.v_cache;
  at.node_off = a.node_off;
  at.kv_len = a.kv_len;
  at.parent = a.parent;
  at.part_o = reinterpret_cast<float*>(ws + plan->off_po);
  at.part_m = reinterpret_cast<float*>(ws + plan->off_pm);
  at.part_l = reinterpret_cast<float*>(ws + plan->off_pl);
  at.x_out = ws + plan->off_x;
  at.attn_out = a.attn_out;
  at.x_copy = a.x_out;
  at.total_nodes = a.total_nodes;
  at.hidden_size = s.hidden;
  at.n_kv_heads = s.n_kv_heads;
  at.group = plan->group;
  at.kv_cap = a.kv_capacity;
  at.max_nodes = a.max_nodes_in_batch;
  at.batch = a.batch;
  at.pieces = 0;
  at.flat = 0;
  at.scale_log2 = (float)(1.4426950408889634 / sqrt((double)s.head_dim));
  const int rows = a.max_nodes_in_batch * plan->group;  // query rows per KV head
  hipError_t ae;
  int merge_rows_per_blk;
  // One split per sequence: the attention kernel divides by its sums and writes x itself (96
  // sequences of 1-12 nodes over 100-1500 rows: the merge of 624 rows' single partials took 15 us).
  bool direct = false;
  const long long t_max = (long long)a.max_kv_len_in_batch + a.max_nodes_in_batch;
  const int t_tiles = cdiv(t_max, kKvTile);
  const AttnPath path = attn_path(plan->es, s.head_dim, s.n_kv_heads, a.batch, rows, t_tiles);
  const LdsUser user = path == AttnPath::kShared ? kLdsShared : path == AttnPath::kStream ? kLdsStream : kLdsRegister;
  if (!(plan->lds_ready.load(std::memory_order_acquire) & (1u << user))) {
    if (!raise_lds_limits(user, s.dtype, plan->es, s.head_dim)) return RESPEC_ERR_HIP;
    plan->lds_ready.fetch_or(1u << user, std::memory_order_release);
  }
  // splits (or pieces) whose partials the workspace holds
  auto held = [&](int heads) { return plan->part_total / ((size_t)a.batch * heads * at.rows_per_wg); };
  if (path == AttnPath::kShared) {
    const int rg = cdiv(rows, 32);  // 1..4: two key groups
    at.wr = rg;
    at.n_rowblk = 1;
    at.rows_per_wg = 32 * rg;
    const Splits sp = kv_splits(kCUs, a.batch, s.n_kv_heads, t_tiles, 2, held(s.n_kv_heads));
    at.nsplit = sp.n;
    at.chunk = sp.tiles * kKvTile;
    at.rotate = tiles_rotated(s.head_dim, a.batch, a.kv_capacity);
    merge_rows_per_blk = rows;
    ae = launch_tree_attn_shared(s.head_dim, dim3(at.nsplit, s.n_kv_heads, a.batch), at, st, ev ? ev[0] : nullptr);
  } else if (path == AttnPath::kStream) {
    const StreamGeom ge = stream_geom(plan, a.max_nodes_in_batch, a.max_kv_len_in_batch, a.batch);
    at.wr = ge.wr;
    at.n_rowblk = ge.n_rowblk;
    at.rows_per_wg = ge.wr * 32;
    merge_rows_per_blk = at.part_rows = ge.part_rows;
    at.pieces = ge.pieces;
    at.piece_shift = ge.kg == 4 ? 2 : 1;  // a piece holds at least a tile per key group, and two
    at.part_blocks = ge.slices * (ge.pieces - 1) + a.batch;
    at.span = reinterpret_cast<int32_t*>(ws + plan->off_span);
    ae = launch_tree_attn_stream(s.head_dim, ge.kg, dim3(ge.pieces, s.n_kv_heads * ge.n_rowblk, ge.slices), at, st,
                                 ev ? ev[0] : nullptr);
  } else {
    const RowGeom ge = row_geom(rows);
    const int heads = s.n_kv_heads * ge.n_rowblk;
    const int wg_target = kTargetWaves / (ge.threads / 64);
    at.rows_per_wg = ge.rows_per_wg;
    const Splits sp = kv_splits(wg_target, a.batch, heads, t_tiles, ge.wk, held(heads));
    at.nsplit = sp.n;
    at.chunk = sp.tiles * kKvTile;
    // Long ragged batches: each head's KV tiles over every sequence are cut into
    // equal pieces, one workgroup each and one piece per CU, so that the longest
    // sequence does not finish alone (two pieces per CU measured slower on an
    // 8-sequence ragged batch: 158 against 144 us).
    const bool flat = path == AttnPath::kFlat;
    if (flat) {
      at.flat = at.nsplit = clampi(wg_target / heads, 1, (int)std::min(held(heads), (size_t)64));
      at.chunk = 0;
    }
    at.n_rowblk = ge.n_rowblk;
    merge_rows_per_blk = ge.rows_per_wg;
    at.wr = ge.wr;
    at.wk = ge.wk;
    direct = !flat && at.nsplit == 1;
    ae = launch_tree_attn(s.dtype, s.head_dim, ge.nb, dim3(at.nsplit, heads, flat ? 1 : a.batch), ge.threads,
                          row_lds(plan->es, s.head_dim, ge), at, st, ev ? ev[0] : nullptr,
                          ev && direct ? ev[1] : nullptr);
  }
  if (ae != hipSuccess) return RESPEC_ERR_HIP;
  // partials of a row: its sequence's splits, or of a batch that is cut into pieces about its share of them
  const int splits = path == AttnPath::kStream ? min(cdiv(at.pieces, a.batch), max(1, t_tiles >> at.piece_shift))
                     : path == AttnPath::kFlat ? cdiv(at.flat, a.batch)
                                               : at.nsplit;
  if (!direct && launch_attn_merge(s.dtype, s.head_dim, at, merge_rows_per_blk, splits, st, ev ? ev[1] : nullptr) !=
                     hipSuccess)
    return RESPEC_ERR_HIP;

  // ---- LM head ----
  if (need_logits) {
    LmArgs lm;
    lm.x = ws + plan->off_x;
    lm.w = a.lm_head;
    lm.logits = a.logits;
    lm.m_rows = a.total_nodes;
    lm.vocab = s.vocab;
    lm.hidden_size = s.hidden;
    const LmTile tile = lm_tile(s.dtype, a.total_nodes, s.vocab);
    lm.n_mtiles = cdiv(a.total_nodes, lm_tile_rows(tile));
    lm.partials = vocab_pass ? reinterpret_cast<float*>(ws + plan->off_part) : nullptr;
    lm.n_vtiles = plan->n_vtiles;
    if (launch_lmhead(s.dtype, tile, lm, st, ev ? ev[2] : nullptr) != hipSuccess) return RESPEC_ERR_HIP;
  } else if (ev && hipEventRecord(ev[2], st) != hipSuccess) {
    return RESPEC_ERR_HIP;
  }

  // ---- row statistics, predicates, path ----
  if (vocab_pass) {
    VocabArgs v;
    v.logits = a.logits;
    v.partials = reinterpret_cast<const float*>(ws + plan->off_part);
    v.node_off = a.node_off;
    v.kv_len = a.kv_len;
    v.parent = a.parent;
    v.token = a.token;
    v.src = a.src;
    v.seq_counter = cnt;
    v.flag_ws = reinterpret_cast<int32_t*>(ws + plan->off_flag);
    v.max_logit = a.max_logit;
    v.lse = a.lse;
    v.entropy = a.entropy;
    v.argmax = a.argmax;
    v.topk_id = a.topk_id;
    v.topk_logprob = a.topk_logprob;
    v.tok_logprob = a.tok_logprob;
    v.flags = a.flags;
    v.leaf_acc_len = a.leaf_acc_len;
    v.path = a.path;
    v.acc_len = a.acc_len;
    v.bonus = a.bonus;
    v.winner_leaf = a.winner_leaf;
    v.seq_status = a.seq_status;
    v.total_nodes = a.total_nodes;
    v.batch = a.batch;
    v.vocab = s.vocab;
    v.n_vtiles = plan->n_vtiles;
    v.topk_out = s.topk_out;
    v.max_nodes = a.max_nodes_in_batch;
    v.max_depth = s.max_depth;
    v.kv_cap = a.kv_capacity;
    v.max_kv = a.max_kv_len_in_batch;
    v.topk = a.accept.topk;
    v.min_lookahead = a.accept.min_lookahead;
    v.max_relaxed = a.accept.max_relaxed;
    v.tau = a.accept.tau;
    v.stats_only = stats_only;
    v.rank_req = rank ? reinterpret_cast<int32_t*>(ws + plan->off_rank) : nullptr;
    v.tok_rank = rank ? a.tok_rank : nullptr;
    // (the stage's last kernel takes the stop event: the rank pass, else the sampling walk, else this one)
    if (launch_finalize(plan->ko, a.total_nodes + a.batch, v, st, (ev && !stochastic && !rank) ? ev[3] : nullptr) !=
        hipSuccess)
      return RESPEC_ERR_HIP;
    if (stochastic) {
      // speculative-sampling walk, after the row statistics and the tree checks
      StochArgs sa;
      sa.logits = a.logits;
      sa.max_logit = a.max_logit;
      sa.lse = a.lse;
      sa.draft_prob = a.draft_prob;
      sa.uniform = a.uniform;
      sa.node_off = a.node_off;
      sa.parent = a.parent;
      sa.token = a.token;
      sa.src = a.src;
      sa.seq_status = a.seq_status;
      sa.seq_counter = cnt;
      sa.ws_next = reinterpret_cast<int32_t*>(ws + plan->off_stoch);
      sa.ws_sample = sa.ws_next + (size_t)s.max_batch * s.max_nodes;
      sa.flags = a.flags;
      sa.sample = a.sample;
      sa.leaf_acc_len = a.leaf_acc_len;
      sa.path = a.path;
      sa.acc_len = a.acc_len;
      sa.bonus = a.bonus;
      sa.winner_leaf = a.winner_leaf;
      sa.total_nodes = a.total_nodes;
      sa.batch = a.batch;
      sa.vocab = s.vocab;
      sa.max_nodes = a.max_nodes_in_batch;
      sa.max_depth = s.max_depth;
      sa.inv_temp = 1.f / a.accept.temperature;
      sa.unit_temp = a.accept.temperature == 1.f;
      if (launch_stochastic(sa, st, (ev && !rank) ? ev[3] : nullptr) != hipSuccess) return RESPEC_ERR_HIP;
    }
    if (rank) {
      RankArgs ra;
      ra.logits = a.logits;
      ra.token = a.token;
      ra.rank_req = v.rank_req;
      ra.tok_rank = a.tok_rank;
      ra.total_nodes = a.total_nodes;
      ra.vocab = s.vocab;
      if (launch_rank(ra, st, ev ? ev[3] : nullptr) != hipSuccess) return RESPEC_ERR_HIP;
    }
  } else if (ev && hipEventRecord(ev[3], st) != hipSuccess) {
    return RESPEC_ERR_HIP;
  }
  return RESPEC_OK;
}

// ---- static workspace of the allocation-free entry point ----
// The array's name is a host-side stand-in: host code uses the device address
// that hipGetSymbolAddress returns for the current device, never `scratch`.
// The front kScratchCounterBytes hold the completion counters at a fixed place,
// so that plans with different workspace layouts sharing the array never read
// another plan's leftovers as counters; the plan's workspace follows them.
constexpr size_t kScratchBytes = (size_t)RESPEC_NOALLOC_SCRATCH_BYTES;
constexpr size_t kScratchCounterBytes = (size_t)RESPEC_NOALLOC_MAX_BATCH * 4;
static_assert(kScratchCounterBytes % 256 == 0, "the workspace after the counters stays 256-byte aligned");

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

struct ScratchSlot {
  std::once_flag once;
  char* ptr = nullptr;  // device address of `scratch` on this device (null: set-up failed)
};
ScratchSlot g_scratch[kMaxDevices];

// Device address of this device's array; on the first call on a device (with
// that device current) it is looked up and the counters are cleared by a fill
// kernel on `stream` (no memset node, so a captured first call stays correct).
char* scratch_for_current_device(hipStream_t stream) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  ScratchSlot& sl = g_scratch[dev];
  std::call_once(sl.once, [&] {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return;
    if (launch_zero_i32(static_cast<int32_t*>(p), RESPEC_NOALLOC_MAX_BATCH, stream) != hipSuccess) return;
    sl.ptr = static_cast<char*>(p);
  });
  return sl.ptr;
}

}  // namespace

extern "C" {

respec_status respec_verify_step(const respec_verify_plan* plan, const respec_verify_args* args, void* workspace,
                                 void* stream) {
  if (!plan || !args) return RESPEC_ERR_NULL;
  if (!workspace || !aligned(workspace, 256)) return RESPEC_ERR_WORKSPACE;
  char* ws = static_cast<char*>(workspace);
  return step_impl(plan, args, ws, reinterpret_cast<int32_t*>(ws + plan->off_cnt), stream);
}

respec_status respec_verify_step_noalloc(const respec_verify_plan* plan, const respec_verify_args* args,
                                         void* stream) {
  if (!plan || !args) return RESPEC_ERR_NULL;
  if (plan->total > kScratchBytes - kScratchCounterBytes || plan->s.max_batch > RESPEC_NOALLOC_MAX_BATCH)
    return RESPEC_ERR_SCRATCH;
  char* base = scratch_for_current_device(static_cast<hipStream_t>(stream));
  if (!base) return RESPEC_ERR_HIP;
  return step_impl(plan, args, base + kScratchCounterBytes, reinterpret_cast<int32_t*>(base), stream);
}

}  // extern "C"
