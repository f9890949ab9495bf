// Host side of the C ABI declared in include/bacon.h: argument checks,
// workspace carving, layer ordering, launch sequencing and event timing.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/bacon.h"
#include "internal.h"
#include "schedule.h"

using namespace bacon;

namespace {

thread_local std::string g_err;

bacon_status fail(bacon_status s, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

bacon_status hip_fail(hipError_t e, const char *what) {
  return fail(BACON_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Layout {
  size_t ring, vec_b, vec_v, vec_pb, vec_pv, vec_s, hist_b, hist_s, list_bk, list_bp, list_bv,
      list_sk, list_sp, cnt_b, cnt_s, rec_b, rec_s, partials, lse2, lambda, hb, sb, sync, total;
  size_t sync_bytes;
  // distances between the copies that layers in flight take in turn
  size_t vec_stride, hist_b_stride, hist_s_stride, list_stride, cnt_stride, rec_stride, hb_stride, sb_stride,
      part_stride, lse_stride, hist_a_stride;
  size_t vec_a, hist_a, list_a, cnt_a, rec_a;   // head-wise allocation
  int rpad, slots;
  int64_t chunks_cap;
};

bacon_status check_shape(const bacon_shape *s) {
  if (!s) return fail(BACON_ERR_INVALID, "shape is NULL");
  if (s->num_layers < 1) return fail(BACON_ERR_INVALID, "num_layers must be >= 1");
  if (s->num_q_heads < 1 || s->num_kv_heads < 1)
    return fail(BACON_ERR_INVALID, "head counts must be >= 1");
  if (s->num_q_heads % s->num_kv_heads)
    return fail(BACON_ERR_INVALID, "num_q_heads (%d) is not a multiple of num_kv_heads (%d)",
                s->num_q_heads, s->num_kv_heads);
  if (s->window < 1) return fail(BACON_ERR_INVALID, "window must be >= 1");
  if (s->max_batch < 1) return fail(BACON_ERR_INVALID, "max_batch must be >= 1");
  if (s->max_total_tokens < 1) return fail(BACON_ERR_INVALID, "max_total_tokens must be >= 1");
  if (s->dtype != BACON_FP32 && s->dtype != BACON_BF16)
    return fail(BACON_ERR_UNSUPPORTED, "dtype %d is not supported", (int)s->dtype);
  if (s->head_dim != 64 && s->head_dim != 128)
    return fail(BACON_ERR_UNSUPPORTED, "head_dim %d is not supported (64 or 128)", s->head_dim);
  if (s->max_batch > kMaxBatch)
    return fail(BACON_ERR_UNSUPPORTED, "max_batch %d exceeds %d", s->max_batch, kMaxBatch);
  const int64_t rows = (int64_t)(s->num_q_heads / s->num_kv_heads) * s->window;
  if (rows > kMaxRows)
    return fail(BACON_ERR_UNSUPPORTED, "group*window = %lld exceeds %d", (long long)rows, kMaxRows);
  if (s->max_total_tokens > ((int64_t)1 << 31) / 2)
    return fail(BACON_ERR_UNSUPPORTED, "max_total_tokens too large");
  return BACON_OK;
}

bacon_status check_params(const bacon_params *p) {
  if (p->radius < 0 || p->radius > 16) return fail(BACON_ERR_INVALID, "radius must be in [0, 16]");
  if (p->persist_m < 0 || p->persist_m > kMaxRing)
    return fail(BACON_ERR_INVALID, "persist_m must be in [0, %d]", kMaxRing);
  if (!(p->rho > 0.0) || !std::isfinite(p->rho)) return fail(BACON_ERR_INVALID, "rho must be > 0");
  if (!(p->gamma >= 0.f) || !std::isfinite(p->gamma))
    return fail(BACON_ERR_INVALID, "gamma must be >= 0");
  if (!(p->eps >= 0.f) || !std::isfinite(p->eps)) return fail(BACON_ERR_INVALID, "eps must be >= 0");
  if (p->pool_kernel < 1 || p->pool_kernel > 33 || (p->pool_kernel & 1) == 0)
    return fail(BACON_ERR_INVALID, "pool_kernel must be odd and in [1, 33]");
  if (p->use_last_query != 0 && p->use_last_query != 1)
    return fail(BACON_ERR_INVALID, "use_last_query must be 0 or 1");
  if (p->terms & ~7u) return fail(BACON_ERR_INVALID, "terms has unknown bits");
  if (p->pool_mode < BACON_POOL_MEAN_S || p->pool_mode > BACON_POOL_MEAN_B)
    return fail(BACON_ERR_INVALID, "pool_mode must be 0, 1 or 2");
  if (p->head_alloc != BACON_ALLOC_GIVEN && p->head_alloc != BACON_ALLOC_ADAPTIVE)
    return fail(BACON_ERR_INVALID, "head_alloc must be 0 or 1");
  if (!(p->alloc_floor >= 0.f && p->alloc_floor <= 1.f))
    return fail(BACON_ERR_INVALID, "alloc_floor must be in [0, 1]");
  return BACON_OK;
}

Layout layout_of(const bacon_shape *s, const bacon_params *p) {
  Layout L{};
  const int G = s->num_q_heads / s->num_kv_heads;
  L.rpad = ((G * s->window + 31) / 32) * 32;
  const bool adaptive = p->head_alloc == BACON_ALLOC_ADAPTIVE;
  L.slots = history_slots(p->persist_m, adaptive);
  const int tk = 32 * std::min(L.rpad / 32, 4);
  L.chunks_cap = (s->max_total_tokens + tk - 1) / tk + s->max_batch;
  const size_t vec = (size_t)s->num_kv_heads * (size_t)s->max_total_tokens * sizeof(float);
  size_t off = 0;
  L.vec_stride = align256(vec);
  L.ring = off;     off += align256((size_t)L.slots * vec);
  L.vec_b = off;    off += copies_b(true, adaptive) * L.vec_stride;
  L.vec_v = off;    off += kCopies2 * L.vec_stride;
  L.vec_pb = off;   off += kCopies2 * L.vec_stride;
  L.vec_pv = off;   off += kCopies2 * L.vec_stride;
  L.vec_s = off;    off += kCopiesS * L.vec_stride;
  const size_t hist = (size_t)s->max_batch * s->num_kv_heads * kHRow * sizeof(unsigned);
  L.hist_b_stride = align256(hist * kHCopies);
  L.hist_s_stride = align256(hist);
  L.hist_b = off;   off += copies_hist_b(true, adaptive) * L.hist_b_stride;
  // the allocation's histograms (bacon_allocate_heads clears its own copy)
  L.hist_a_stride = align256(hist);
  L.hist_a = off;   off += (adaptive ? kCopiesHistA : 1) * L.hist_a_stride;
  // meeting words of the single-read pass (arrival and done counters per
  // (sequence, KV head) on lines of their own, the error word, the published
  // row normalisers)
  L.sync_bytes = align256((size_t)(kSyncStride * s->max_batch * s->num_kv_heads + 1) * sizeof(unsigned)) +
                 align256((size_t)s->max_batch * s->num_kv_heads * L.rpad * sizeof(unsigned));
  L.sync = off;     off += L.sync_bytes;
  L.hist_s = off;   off += kCopiesS * L.hist_s_stride;
  // the lists of one copy lie one after the other: keys, positions, V for B
  // (3 vectors) and keys, positions for S (2 vectors)
  L.list_bk = off;
  L.list_bp = off + L.vec_stride;
  L.list_bv = off + 2 * L.vec_stride;
  L.list_sk = off + 3 * L.vec_stride;
  L.list_sp = off + 4 * L.vec_stride;
  L.list_stride = 5 * L.vec_stride;
  off += kCopies2 * L.list_stride;
  const int64_t segs_cap = (s->max_total_tokens + kSegLen - 1) / kSegLen + s->max_batch;
  L.cnt_stride = align256((size_t)s->num_kv_heads * segs_cap * sizeof(int));
  L.cnt_b = off;    off += kCopies2 * L.cnt_stride;
  L.cnt_s = off;    off += kCopies2 * L.cnt_stride;
  L.rec_stride = align256((size_t)s->max_batch * s->num_kv_heads * sizeof(int4));
  L.rec_b = off;    off += kCopies2 * L.rec_stride;
  L.rec_s = off;    off += kCopies2 * L.rec_stride;
  L.vec_a = off;    off += (adaptive ? kCopiesA : 1) * L.vec_stride;
  L.list_a = off;   off += (adaptive ? kCopies2 : 1) * L.vec_stride;
  L.cnt_a = off;    off += (adaptive ? kCopies2 : 1) * L.cnt_stride;
  L.rec_a = off;    off += (adaptive ? kCopies2 : 1) * L.rec_stride;
  L.part_stride = align256((size_t)s->num_kv_heads * L.chunks_cap * L.rpad * sizeof(float2));
  L.partials = off; off += kCopies2 * L.part_stride;
  L.lse_stride = align256((size_t)s->max_batch * s->num_kv_heads * L.rpad * sizeof(float));
  L.lse2 = off;     off += kCopies2 * L.lse_stride;
  L.lambda = off;   off += align256((size_t)s->max_batch * s->num_kv_heads * sizeof(float));
  L.hb_stride = align256((size_t)s->max_batch * s->num_kv_heads * sizeof(int2));
  L.hb = off;       off += kCopiesTab * L.hb_stride;
  L.sb_stride = align256((size_t)s->max_batch * sizeof(int4));
  L.sb = off;       off += kCopiesTab * L.sb_stride;
  L.total = off;
  return L;
}

const char *kKernelNames[] = {"window_lse",    "lse_merge",     "window_score", "window_score_calib",
                              "segment_calib", "segment_score", "segment_cand",
                              "final_topk",    "split_calib",   "select_topk",
                              "compact",       "window_lse_kr",
                              "window_score_calib_kr", "window_score_calib_lse_kr",
                              "segment_select", "layer_stages", "window_lse_wide", "window_score_calib_wide",
                              "window_score_calib_lse", "window_score_single", "head_alloc"};
enum KernelId { KI_LSE, KI_MERGE, KI_SCORE, KI_FUSED, KI_SEGCAL, KI_SEGSCORE, KI_SEGCAND, KI_FINAL,
                KI_SPLIT_CALIB, KI_SEL_TOPK, KI_COMPACT, KI_LSE_KR, KI_FUSED_KR, KI_DUAL_KR,
                KI_SEL, KI_MEGA, KI_LSE_WIDE, KI_FUSED_WIDE, KI_DUAL, KI_SINGLE, KI_ALLOC, KI_COUNT };

}  // namespace

struct bacon_ctx {
  bacon_shape shape;
  bacon_params params;
  char *ws;
  size_t ws_bytes;
  Layout L;
  bool prompt = false;
  int next_layer = 0;
  std::vector<int32_t> cu;
  int chunk_stages_override = 0;
  bool kr_off = false;   // key-register passes switched off (streaming passes only)
  int single_mode = -1;      // single-read pass: -1 where it pays, 0 never, 1 wherever it can run
  // largest grid of the wide passes, in 512-key workgroups: on 224 (32 heads of
  // d 64, three sequences) a prompt of seven layers takes 195 us with them and
  // 207 with the key-register passes, on 246 (224 rows, 14/2 heads) 180 either
  // way; the ragged batch's 856 take 4139 with them and 2739 without
  int wide_limit = 256;
  int single_cap = -1;       // single-read workgroups the device holds at once (-1: not yet asked)
  int cus = -1;              // compute units of the device (-1: not yet asked)
  // test instrumentation (bacon_debug_capture): per-layer copies of B, V, lambda
  float *cap_B = nullptr, *cap_V = nullptr, *cap_lambda = nullptr;
  int32_t *alloc_out = nullptr;   // [num_layers, max_batch, Hkv] budgets of the adaptive allocation
  // profiling
  bool prof = false;
  std::vector<hipEvent_t> ev_pool;
  struct Pending { int kid; hipEvent_t a, b; };
  std::vector<Pending> pending;
  size_t ev_next = 0;
  int64_t launches[KI_COUNT] = {};
  double ms[KI_COUNT] = {};
};

namespace {

// The device error word (after the meeting counters of the single-read pass):
// 1 if a meeting ran out, 2 if an allocation failed its check.
unsigned *error_word(bacon_ctx *c) {
  return reinterpret_cast<unsigned *>(c->ws + c->L.sync) +
         (size_t)kSyncStride * c->shape.max_batch * c->shape.num_kv_heads;
}

}  // namespace

namespace {

// Records events around a launch when profiling is on.
template <typename F>
bacon_status timed(bacon_ctx *c, int kid, hipStream_t s, F &&launch) {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (c->prof && c->ev_next + 2 <= c->ev_pool.size()) {
    e0 = c->ev_pool[c->ev_next++];
    e1 = c->ev_pool[c->ev_next++];
    hipEventRecord(e0, s);
  }
  const hipError_t e = launch();
  if (e != hipSuccess) return hip_fail(e, kKernelNames[kid]);
  if (e0) {
    hipEventRecord(e1, s);
    c->pending.push_back({kid, e0, e1});
  }
  return BACON_OK;
}

bacon_status check_batch(const bacon_ctx *c, const bacon_batch *bt) {
  if (!bt) return fail(BACON_ERR_INVALID, "batch is NULL");
  if (bt->batch < 1 || bt->batch > c->shape.max_batch)
    return fail(BACON_ERR_INVALID, "batch size %d outside [1, %d]", bt->batch, c->shape.max_batch);
  if (!bt->cu_seqlens || (!bt->budgets && !bt->head_budgets))
    return fail(BACON_ERR_INVALID, "batch arrays are NULL");
  if (bt->cu_seqlens[0] != 0) return fail(BACON_ERR_INVALID, "cu_seqlens[0] must be 0");
  for (int b = 0; b < bt->batch; ++b) {
    const int64_t n = (int64_t)bt->cu_seqlens[b + 1] - bt->cu_seqlens[b];
    if (n < c->shape.window)
      return fail(BACON_ERR_INVALID, "sequence %d has %lld tokens, fewer than the window %d", b,
                  (long long)n, c->shape.window);
    if (n > kMaxSeqLen)
      return fail(BACON_ERR_UNSUPPORTED, "sequence %d has %lld tokens (max %d)", b, (long long)n,
                  kMaxSeqLen);
    if (bt->head_budgets) {
      for (int h = 0; h < c->shape.num_kv_heads; ++h)
        if (bt->head_budgets[(int64_t)b * c->shape.num_kv_heads + h] < 1)
          return fail(BACON_ERR_INVALID, "budget of sequence %d, KV head %d must be >= 1", b, h);
    } else if (bt->budgets[b] < 1) {
      return fail(BACON_ERR_INVALID, "budget of sequence %d must be >= 1", b);
    }
  }
  if (bt->cu_seqlens[bt->batch] > c->shape.max_total_tokens)
    return fail(BACON_ERR_INVALID, "total tokens %d exceed max_total_tokens %lld",
                bt->cu_seqlens[bt->batch], (long long)c->shape.max_total_tokens);
  return BACON_OK;
}

bacon_status check_prompt_batch(const bacon_ctx *c, const bacon_batch *bt) {
  if (!c->prompt) return fail(BACON_ERR_ORDER, "no prompt begun (call bacon_begin_prompt)");
  // the sequences are fixed for the prompt; the budgets may change from layer
  // to layer (a per-layer budget schedule)
  if (bt->batch + 1 != (int)c->cu.size() ||
      memcmp(bt->cu_seqlens, c->cu.data(), c->cu.size() * sizeof(int32_t)) != 0)
    return fail(BACON_ERR_INVALID, "batch sequences differ from the ones given to bacon_begin_prompt");
  return BACON_OK;
}

bacon_status check_ptr(const void *p, const char *name, size_t align) {
  if (!p) return fail(BACON_ERR_INVALID, "%s is NULL", name);
  if (reinterpret_cast<uintptr_t>(p) % align)
    return fail(BACON_ERR_INVALID, "%s is not %zu-byte aligned", name, align);
  return BACON_OK;
}

#define TRY(x)                     \
  do {                             \
    bacon_status _s = (x);         \
    if (_s != BACON_OK) return _s; \
  } while (0)

// Budget of (sequence b, KV head h), and the largest budget of sequence b's
// heads (its rows per head in the compacted cache, less W).
int batch_head_budget(const bacon_batch *bt, int hkv, int b, int h) {
  return bt->head_budgets ? bt->head_budgets[(int64_t)b * hkv + h] : bt->budgets[b];
}
int batch_seq_rows(const bacon_batch *bt, int hkv, int b) {
  if (!bt->head_budgets) return bt->budgets[b];
  int m = 0;
  for (int h = 0; h < hkv; ++h) m = std::max(m, batch_head_budget(bt, hkv, b, h));
  return m;
}

SeqTable make_table(const bacon_ctx *c, const bacon_batch *bt, int *chunk_out, int force_chunk = 0) {
  SeqTable st{};
  st.batch = bt->batch;
  const bool bf16 = c->shape.dtype == BACON_BF16;
  const int nw = c->L.rpad / 32, tk = stage_keys(nw);
  int64_t stages = 0;
  for (int b = 0; b < bt->batch; ++b) {
    const int n = bt->cu_seqlens[b + 1] - bt->cu_seqlens[b];
    stages += (n + tk - 1) / tk;
  }
  stages *= c->shape.num_kv_heads;
  // one round of workgroups over the 256 CUs at the occupancy LDS and waves allow
  const int lds = pass_lds_bytes(PASS_FUSED, bf16, c->shape.head_dim, c->L.rpad, 4 * tk);
  const int by_lds = std::max(1, (160 * 1024) / std::max(1, lds));
  const int by_waves = std::max(1, 16 / nw);
  const int64_t slots = 256LL * std::min(by_lds, by_waves);
  int per_wg = (int)std::max<int64_t>(1, (stages + slots - 1) / slots);
  if (c->chunk_stages_override > 0) per_wg = c->chunk_stages_override;
  per_wg = std::min(per_wg, kMaxChunk / tk);
  const int chunk = force_chunk > 0 ? force_chunk : tk * per_wg;
  int cb = 0, ib = 0, kb = 0, sb = 0;
  for (int b = 0; b < bt->batch; ++b) {
    const int n = bt->cu_seqlens[b + 1] - bt->cu_seqlens[b];
    const int nseg = (n + kSegLen - 1) / kSegLen;
    st.cu[b] = bt->cu_seqlens[b];
    st.chunk_base[b] = cb;
    st.budget[b] = batch_seq_rows(bt, c->shape.num_kv_heads, b);
    st.idx_base[b] = ib;
    st.kept_base[b] = kb;
    st.seg_base[b] = sb;
    cb += (n + chunk - 1) / chunk;
    for (int h = 0; h < c->shape.num_kv_heads; ++h) ib += batch_head_budget(bt, c->shape.num_kv_heads, b, h);
    kb += st.budget[b] + c->shape.window;
    sb += nseg;
  }
  st.cu[bt->batch] = bt->cu_seqlens[bt->batch];
  st.chunk_base[bt->batch] = cb;
  st.seg_base[bt->batch] = sb;
  st.total_chunks = cb;
  st.total_segs = sb;
  *chunk_out = chunk;
  return st;
}

PassArgs pass_args(const bacon_ctx *c, const SeqTable &st, int chunk, const void *q, const void *k) {
  PassArgs a{};
  const bacon_shape &s = c->shape;
  a.q = q;
  a.k = k;
  a.Hq = s.num_q_heads;
  a.Hkv = s.num_kv_heads;
  a.G = s.num_q_heads / s.num_kv_heads;
  a.W = s.window;
  a.R = a.G * s.window;
  a.Rpad = c->L.rpad;
  a.chunk = chunk;
  a.T = s.max_total_tokens;
  a.c2 = (float)(1.4426950408889634 / std::sqrt((double)s.head_dim));
  if (c->ws) {   // a context over no workspace (the static-scratch call) sets its own
    a.partials = reinterpret_cast<float2 *>(c->ws + c->L.partials);
    a.lse2 = reinterpret_cast<float *>(c->ws + c->L.lse2);
    a.hist_B = reinterpret_cast<unsigned *>(c->ws + c->L.hist_b);
    a.ring = reinterpret_cast<float *>(c->ws + c->L.ring);
    a.vec_B = reinterpret_cast<float *>(c->ws + c->L.vec_b);
  }
  a.radius = c->params.radius;
  a.terms = c->params.terms;
  if (c->ws) {
    a.sync = reinterpret_cast<unsigned *>(c->ws + c->L.sync);
    a.sync_groups = c->shape.max_batch * c->shape.num_kv_heads;
    a.bcast = reinterpret_cast<unsigned *>(
        c->ws + c->L.sync + align256((size_t)(kSyncStride * a.sync_groups + 1) * sizeof(unsigned)));
  }
  (void)st;
  return a;
}

// Per-head budgets of the batch into the workspace table (budget, idx offset
// within the sequence), or NULL with one budget per sequence.  The table rides
// in the arguments of small kernels on the stream, ahead of the select.
bacon_status head_table(bacon_ctx *c, const bacon_batch *bt, hipStream_t s, const int2 **out,
                        int copy = 0) {
  *out = nullptr;
  if (!bt->head_budgets) return BACON_OK;
  const int hkv = c->shape.num_kv_heads;
  int2 *dst = reinterpret_cast<int2 *>(c->ws + c->L.hb + (size_t)copy * c->L.hb_stride);
  HbChunk ch{};
  const int n = bt->batch * hkv;
  int off = 0;
  for (int p = 0; p < n; ++p) {
    if (p % hkv == 0) off = 0;
    const int k = bt->head_budgets[p];
    ch.v[ch.n++] = make_int2(k, off);
    off += k;
    if (ch.n == kHbChunk || p == n - 1) {
      const hipError_t e = launch_set_hb(ch, dst, s);
      if (e != hipSuccess) return hip_fail(e, "budget table");
      ch.base += ch.n;
      ch.n = 0;
    }
  }
  *out = dst;
  return BACON_OK;
}

// The per-sequence budget fields (budget, idx base, kept-row base) of a
// layer's batch into the workspace table of its copy, for the launches
// that hold the jobs of several layers with different budgets.
bacon_status seq_table(bacon_ctx *c, const SeqTable &st, hipStream_t s, const int4 **out, int copy) {
  int2 *dst = reinterpret_cast<int2 *>(c->ws + c->L.sb + (size_t)copy * c->L.sb_stride);
  HbChunk ch{};
  for (int b = 0; b < st.batch; ++b) {
    ch.v[ch.n++] = make_int2(st.budget[b], st.idx_base[b]);
    ch.v[ch.n++] = make_int2(st.kept_base[b], 0);
  }
  const hipError_t e = launch_set_hb(ch, dst, s);
  if (e != hipSuccess) return hip_fail(e, "budget table");
  *out = reinterpret_cast<const int4 *>(dst);
  return BACON_OK;
}

// History slots for layer `layer`: E of layer j lives in slot j % slots, with more
// than m of them, so the previous cnt = min(m, layer) layers are the slots
// wr - cnt .. wr - 1 (mod slots), none of them wr.
void ring_slots(const bacon_ctx *c, int layer, int *wr, int *cnt) {
  *cnt = std::min(c->params.persist_m, layer);
  *wr = layer % c->L.slots;
}

// Compute units of the device.
int device_cus(bacon_ctx *c) {
  if (c->cus < 0) {
    int dev = 0, n = 0;
    c->cus = 256;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
      c->cus = n;
  }
  return c->cus;
}

// Calls that plan the wide passes: the fused calls, the fused calls with the
// normalisers given (no pass 1), bacon_score (no select).
enum WideCall { WIDE_FUSED, WIDE_GIVEN, WIDE_SCORE };

// A batch's grid on the wide passes with s row groups per workgroup.
struct WideGrid {
  double cus;
  int nrt, rpad;
  int chunks;             // of the longest sequence
  double blocks, jobs;    // chunks and workgroups over the KV heads
  double sel;             // select workgroups
};

// Estimates of a plan (the smaller the better).  The prompt call and the layer
// calls must share the row groups, which decide how the normalisers' sums are
// grouped: both return the same bits.
//
// bf16 (us, from traces of 16 to 512 workgroups): a workgroup takes 6 plus 2.2 per
// further chunk and 0.9 per row tile of four waves on a SIMD; a select workgroup 8;
// beyond one round of the CUs a launch takes the sum over the CUs and half a
// workgroup more.  A pass of a layer call counts beside the prompt's launch, more
// beyond 128 rows, where one row group leaves a layer call well behind the
// streaming passes (28/4 heads, 8K tokens, 12 layers: prompt 280 and layer calls
// 742 us with one, 300 and 660 with two; 472 and 629 before).
double wide_cost_bf16(const WideGrid &g, int s, int p) {
  const double t = 6.0 + 2.2 * (p - 1) + p * 0.9 * std::max((double)g.nrt / s, 0.25 * ((g.nrt + s - 1) / s));
  const double n = 2.0 * g.jobs + g.sel, t1 = t - (p - 1) * (t - 3.8) / 2;
  return (n <= g.cus ? std::max(t, 8.0) : (2.0 * g.jobs * t + g.sel * 8.0) / g.cus + 0.5 * t) +
         (g.nrt > 4 ? 1.3 : 0.5) * (g.blocks <= g.cus ? t1 : g.blocks * t1 / g.cus + 0.5 * t1);
}
// fp32: a workgroup takes 4.4, what its waves' key requests take (a 16-byte load
// of a wave touches 32 rows: 0.027 us per load instruction) and 0.0149 d per row tile
// of a SIMD (its matrix instructions); pass 2 1.5 and the merge of the normalisers more
// (d 128, 8 rows, 700 tokens: pass 1 18.5, 12.0 and 7.7 us with one, two and four
// row groups).  A layer of a six-layer prompt call then takes 7.3 + 1.1 (pass 2) in one
// round of the CUs, else 8.3 + 0.97 (K passes over the CUs) + 7.2 (select) + 0.3
// (pass 2), and a layer call 28 more than its passes, both within 6% over 38 shapes
// of 8 to 128 rows and 700 to 13201 tokens.  The product weighs the two calls the
// same: 4.5% off the prompt calls and 6.3% off the layer calls of these shapes (up to
// 1.12 of the streaming passes' time without it).
double wide_cost_fp32(const WideGrid &g, int d, WideCall call, int s, int p) {
  const double unit = d / 8, chunk = 0.027 * (16 / s * std::min(s, g.nrt)) * unit + 0.0149 * d * 4 * g.nrt / s;
  const double more = 1.5 + (call == WIDE_GIVEN ? 0.0 : 0.03 * g.chunks * g.rpad / 256);
  const double first = call == WIDE_GIVEN ? 0.0 : 1.0;
  const double passes = (first * (4.4 + chunk) + 4.4 + chunk + more) * (g.blocks <= g.cus ? 1.0 : g.blocks / g.cus + 0.3);
  if (call == WIDE_SCORE) return passes;
  const double t1 = 4.1 + p * (0.3 + chunk), t2 = t1 + more;
  const double prompt = (1.0 + first) * g.jobs + g.sel <= g.cus
                            ? std::max(16.5, 7.3 + 1.1 * t2)
                            : 8.3 + (0.97 * g.jobs * (first * t1 + t2) + 7.2 * g.sel) / g.cus + 0.3 * t2;
  return prompt * (28.0 + 1.07 * passes);
}
// The same of the streaming passes with fp32's 128 rows: 6.5 and 9.5 (d 128) per
// stage that a CU takes, two passes, the merge, a select launch of 12.  (3344, 3127 and
// 5213 tokens, 32/8 heads, six layers: prompt call 558 and layer calls 666 us, 605 and
// 742 on the wide passes; 13201 tokens: 648 and 760, 599 and 752.)
double stream_cost_fp32(const bacon_ctx *c, const bacon_batch *bt, double cus) {
  const int d = c->shape.head_dim, tk = stage_keys(c->L.rpad / 32);
  double stages = 0;
  for (int b = 0; b < bt->batch; ++b) stages += (bt->cu_seqlens[b + 1] - bt->cu_seqlens[b] + tk - 1) / tk;
  stages *= c->shape.num_kv_heads;
  const double fit = std::max(1, kLdsBytes / pass_lds_bytes(PASS_FUSED, false, d, c->L.rpad, 4 * tk));
  const double each = std::ceil(stages / (cus * fit));   // stages of a workgroup
  const double t = 6.5 + 0.074 * d * each * std::ceil(stages / each / cus);
  return (2 * t + 16.5) * (28.0 + 2 * t + 2.5);
}

// Whether a batch takes the wide passes, with how many row groups per
// workgroup and chunks per workgroup.
bool wide_plan(bacon_ctx *c, const bacon_batch *bt, WideCall call, int *split, int *cpw) {
  const bool bf16 = c->shape.dtype == BACON_BF16;
  const int hkv = c->shape.num_kv_heads, d = c->shape.head_dim;
  WideGrid g{};
  g.cus = device_cus(c);
  g.rpad = c->L.rpad;
  g.nrt = g.rpad / 32;
  // (more than 128 rows of fp32: a layer call of 13404 and 2013 tokens, 14/2 heads,
  // takes 111 us a layer here and 89 with the streaming passes)
  if (!bf16 && g.nrt > 4) return false;
  for (int b = 0; b < bt->batch; ++b)
    g.sel += 1 + 3 * ((bt->cu_seqlens[b + 1] - bt->cu_seqlens[b] + kSegLen - 1) / kSegLen);
  g.sel *= hkv;
  double best = 1e30;
  for (int s = 1; s <= 4; s *= 2) {
    if (!wide_supported(bf16, d, g.rpad, s)) continue;
    for (int p = 1; p <= 2; ++p) {
      g.chunks = 0;
      g.blocks = g.jobs = 0;
      for (int b = 0; b < bt->batch; ++b) {
        const int k = (bt->cu_seqlens[b + 1] - bt->cu_seqlens[b] + wide_keys(s) - 1) / wide_keys(s);
        g.chunks = std::max(g.chunks, k);
        g.blocks += (double)k * hkv;
        g.jobs += (double)((k + p - 1) / p) * hkv;
      }
      if (g.chunks > wide_max_chunks(g.rpad) || g.blocks > (double)c->wide_limit * s) continue;
      const double est = bf16 ? wide_cost_bf16(g, s, p) : wide_cost_fp32(g, d, call, s, p);
      if (est < best) {
        best = est;
        *split = s;
        *cpw = p;
      }
    }
  }
  // (within the estimates' error the wide passes stay)
  if (!bf16 && g.nrt == 4 && call == WIDE_FUSED && 0.95 * best > stream_cost_fp32(c, bt, g.cus)) return false;
  return best < 1e30;
}

// Whether a layer call with the normalisers given is faster on the streaming
// pass 2, whose sums (B and Q given the normalisers) are those of the wide pass
// where no key-register pass covers the shape: 128 rows of fp32 (3634 tokens, 32/8
// heads, d 128, six layers: 288 us against 302; 13201: 471 and 466), and more than
// 128 of bf16 as long as it runs one stage per workgroup and CU (3634 tokens, 28/4
// heads, d 128: 228 and 240; 13201 tokens, d 64: 279 and 232).
bool stream_given(bacon_ctx *c, const bacon_batch *bt) {
  const int nrt = c->L.rpad / 32;
  if (c->shape.dtype != BACON_BF16) return nrt == 4;
  int64_t stages = 0;
  for (int b = 0; b < bt->batch; ++b)
    stages += (bt->cu_seqlens[b + 1] - bt->cu_seqlens[b] + stage_keys(nrt) - 1) / stage_keys(nrt);
  return nrt > 4 && stages * c->shape.num_kv_heads <= device_cus(c);
}

// The wide passes' fields of a's arguments over the chunks of st.
void wide_args(const bacon_ctx *c, PassArgs &a, int split, int cpw, const SeqTable &st) {
  a.wide_split_log = split >> 1;   // 1, 2, 4
  a.wide_cpw_log = cpw >> 1;       // 1, 2
  a.row_log = wide_row_log(c->L.rpad);
  a.w_magic = 65536u / (unsigned)a.W + 1u;
  a.wide_jobs = 0;
  for (int b = 0; b < st.batch; ++b) a.wide_jobs += (st.chunk_base[b + 1] - st.chunk_base[b] + cpw - 1) / cpw;
}

// The head-wise allocation's arguments of a layer, but for B and the sequences'
// budgets.
AllocArgs alloc_args(const bacon_ctx *c, int64_t T, int layer) {
  const Layout &L = c->L;
  const bool ad = c->params.head_alloc == BACON_ALLOC_ADAPTIVE;
  const size_t c2 = ad ? layer % kCopies2 : 0;
  AllocArgs a{};
  a.Hkv = c->shape.num_kv_heads;
  a.W = c->shape.window;
  a.pool_half = c->params.pool_kernel / 2;
  a.T = T;
  a.alpha = c->params.alloc_floor;
  a.vec_A = reinterpret_cast<float *>(c->ws + L.vec_a + (ad ? layer % kCopiesA : 0) * L.vec_stride);
  a.hist_A = reinterpret_cast<unsigned *>(c->ws + L.hist_a + (ad ? layer % kCopiesHistA : 0) * L.hist_a_stride);
  a.list_A = reinterpret_cast<unsigned *>(c->ws + L.list_a + c2 * L.vec_stride);
  a.cnt_A = reinterpret_cast<int *>(c->ws + L.cnt_a + c2 * L.cnt_stride);
  a.rec_A = reinterpret_cast<uint2 *>(c->ws + L.rec_a + c2 * L.rec_stride);
  a.hb = reinterpret_cast<int2 *>(c->ws + L.hb + (size_t)(layer % kCopiesTab) * L.hb_stride);
  a.err = error_word(const_cast<bacon_ctx *>(c));
  return a;
}

int max_len(const bacon_batch *bt);

// Every workgroup of the pass must fit the LDS of one CU; checked before
// anything is enqueued.
bacon_status check_lds(const bacon_ctx *c, int chunk) {
  if (pass_lds_bytes(PASS_FUSED, c->shape.dtype == BACON_BF16, c->shape.head_dim, c->L.rpad, chunk) > kLdsBytes)
    return fail(BACON_ERR_UNSUPPORTED, "pass workgroup needs more LDS than a CU has");
  return BACON_OK;
}
// The split calls' selections hold sequences of up to kMaxSelLen tokens.
bacon_status check_split(const bacon_batch *bt) {
  if (max_len(bt) > kMaxSelLen)
    return fail(BACON_ERR_UNSUPPORTED, "the split calls select sequences of up to %d tokens (%d given); "
                "the fused calls take up to %d", kMaxSelLen, max_len(bt), kMaxSeqLen);
  return BACON_OK;
}

int max_len(const bacon_batch *bt) {
  int m = 0;
  for (int b = 0; b < bt->batch; ++b) m = std::max(m, bt->cu_seqlens[b + 1] - bt->cu_seqlens[b]);
  return m;
}

}  // namespace

extern "C" {

void bacon_default_params(bacon_params *p) {
  if (!p) return;
  p->radius = 5;
  p->persist_m = 4;
  p->rho = 2.0;
  p->gamma = 1.0f;
  p->eps = 1e-12f;
  p->pool_kernel = 7;
  p->pool_mode = BACON_POOL_MEAN_S;
  p->use_last_query = 1;
  p->terms = BACON_TERM_E | BACON_TERM_L | BACON_TERM_T;
  p->head_alloc = BACON_ALLOC_GIVEN;
  p->alloc_floor = 0.2f;
}

size_t bacon_workspace_bytes(const bacon_shape *shape, const bacon_params *params) {
  bacon_params p;
  if (params) p = *params; else bacon_default_params(&p);
  if (check_shape(shape) != BACON_OK || check_params(&p) != BACON_OK) return 0;
  return layout_of(shape, &p).total;
}

bacon_status bacon_init(bacon_ctx **ctx, const bacon_shape *shape, const bacon_params *params,
                        void *d_ws, size_t ws_bytes) {
  if (!ctx) return fail(BACON_ERR_INVALID, "ctx is NULL");
  *ctx = nullptr;
  TRY(check_shape(shape));
  bacon_params p;
  if (params) p = *params; else bacon_default_params(&p);
  TRY(check_params(&p));
  if (!d_ws) return fail(BACON_ERR_WORKSPACE, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(d_ws) % 256)
    return fail(BACON_ERR_WORKSPACE, "workspace is not 256-byte aligned");
  const Layout L = layout_of(shape, &p);
  if (ws_bytes < L.total)
    return fail(BACON_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", ws_bytes, L.total);
  bacon_ctx *c = new bacon_ctx();
  c->shape = *shape;
  c->params = p;
  c->ws = static_cast<char *>(d_ws);
  c->ws_bytes = ws_bytes;
  c->L = L;
  if (const char *e = std::getenv("BACON_CHUNK_STAGES")) c->chunk_stages_override = std::atoi(e);
  if (const char *e = std::getenv("BACON_KEY_REGISTERS")) c->kr_off = std::atoi(e) == 0;
  if (const char *e = std::getenv("BACON_WIDE")) c->wide_limit = std::atoi(e);
  if (const char *e = std::getenv("BACON_SINGLE")) c->single_mode = std::atoi(e) == 0 ? 0 : 1;
  *ctx = c;
  return BACON_OK;
}

bacon_status bacon_free(bacon_ctx *c) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  for (hipEvent_t e : c->ev_pool) hipEventDestroy(e);
  delete c;
  return BACON_OK;
}

bacon_status bacon_begin_prompt(bacon_ctx *c, const bacon_batch *bt, void *stream) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  TRY(check_batch(c, bt));
  c->cu.assign(bt->cu_seqlens, bt->cu_seqlens + bt->batch + 1);

  // layer 0 reads no history; the histograms of the select and of the allocation
  // start at zero (each layer's jobs clear their copy for the layer that takes it
  // next), and so do the meeting counters of the single-read pass.  Only the
  // batch's rows of each copy: 64 sequences of 32 KV heads have 302 MB of copies,
  // 60 us to clear for a prompt of one.
  const Layout &L = c->L;
  const bool adaptive = c->params.head_alloc == BACON_ALLOC_ADAPTIVE;
  const int64_t rows = (int64_t)bt->batch * c->shape.num_kv_heads;
  auto at = [&](size_t off) { return reinterpret_cast<unsigned *>(c->ws + off); };
  ClearArgs z{};
  z.p[0] = at(L.hist_b);
  z.words[0] = rows * kHCopies * kHRow;
  z.stride[0] = (int64_t)(L.hist_b_stride / sizeof(unsigned));
  z.copies[0] = copies_hist_b(true, adaptive);
  z.p[1] = at(L.hist_a);
  z.words[1] = rows * kHRow;
  z.stride[1] = (int64_t)(L.hist_a_stride / sizeof(unsigned));
  z.copies[1] = adaptive ? kCopiesHistA : 0;
  z.p[2] = at(L.sync);
  z.words[2] = (int64_t)(L.sync_bytes / sizeof(unsigned));
  z.copies[2] = 1;
  const hipError_t e = launch_clear(z, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(e, "clear");
  c->prompt = true;
  c->next_layer = 0;
  return BACON_OK;
}

bacon_status bacon_score(bacon_ctx *c, int32_t layer, const bacon_batch *bt, const void *d_q_win,
                         const void *d_k, float *d_lse, float *d_B, float *d_Q, void *stream) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  TRY(check_batch(c, bt));
  if (layer < 0 || layer >= c->shape.num_layers)
    return fail(BACON_ERR_INVALID, "layer %d outside [0, %d)", layer, c->shape.num_layers);
  TRY(check_ptr(d_q_win, "q_win", 16));
  TRY(check_ptr(d_k, "k", 16));
  TRY(check_ptr(d_B, "B", 4));
  TRY(check_ptr(d_Q, "Q", 4));
  if (d_lse) TRY(check_ptr(d_lse, "lse", 4));
  hipStream_t s = static_cast<hipStream_t>(stream);
  int chunk = 0;
  SeqTable st = make_table(c, bt, &chunk);
  TRY(check_lds(c, chunk));
  // small grids take the wide passes (with the streaming passes' sums)
  int split = 1, cpw = 1;
  const bool wide = !c->kr_off && wide_plan(c, bt, WIDE_SCORE, &split, &cpw);
  if (wide) st = make_table(c, bt, &chunk, wide_keys(split));
  PassArgs a = pass_args(c, st, chunk, d_q_win, d_k);
  a.T = bt->cu_seqlens[bt->batch];
  a.lse_user = d_lse;
  a.out_B = d_B;
  a.out_Q = d_Q;
  const bool bf16 = c->shape.dtype == BACON_BF16;
  const bool w32 = c->shape.window == 32;
  if (wide) {
    wide_args(c, a, split, 1, st);
    TRY(timed(c, KI_LSE_WIDE, s, [&] { return launch_wide(PASS_LSE, bf16, c->shape.head_dim, a, st, s); }));
    if (d_lse) TRY(timed(c, KI_MERGE, s, [&] { return launch_lse_merge(a, st, s); }));
    return timed(c, KI_FUSED_WIDE, s, [&] { return launch_wide(PASS_FUSED, bf16, c->shape.head_dim, a, st, s); });
  }
  TRY(timed(c, KI_LSE, s, [&] { return launch_pass(PASS_LSE, bf16, c->shape.head_dim, false, a, st, s); }));
  TRY(timed(c, KI_MERGE, s, [&] { return launch_lse_merge(a, st, s); }));
  return timed(c, KI_SCORE, s, [&] { return launch_pass(PASS_SCORE, bf16, c->shape.head_dim, w32, a, st, s); });
}

bacon_status bacon_calibrate(bacon_ctx *c, int32_t layer, const bacon_batch *bt, const float *d_B,
                             const float *d_Q, float *d_S, float *d_lambda, float *d_E,
                             float *d_V, void *stream) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  TRY(check_batch(c, bt));
  TRY(check_prompt_batch(c, bt));
  if (layer != c->next_layer)
    return fail(BACON_ERR_ORDER, "layer %d given, layer %d expected next", layer, c->next_layer);
  if (layer >= c->shape.num_layers)
    return fail(BACON_ERR_ORDER, "layer %d beyond num_layers %d", layer, c->shape.num_layers);
  TRY(check_ptr(d_B, "B", 4));
  TRY(check_ptr(d_Q, "Q", 4));
  TRY(check_ptr(d_S, "S", 4));
  TRY(check_ptr(d_lambda, "lambda", 4));
  if (d_E) TRY(check_ptr(d_E, "E", 4));
  if (d_V) TRY(check_ptr(d_V, "V", 4));
  hipStream_t s = static_cast<hipStream_t>(stream);
  TRY(check_split(bt));
  int chunk = 0;
  const SeqTable st = make_table(c, bt, &chunk);
  // the [Hkv, T] vectors of the split path use the batch's T as row length;
  // V, the lists and a copy of B take the first copies of the fused pass's, and the B
  // histogram an S histogram (each user clears it first)
  const Layout &L = c->L;
  SplitArgs p{};
  SegArgs &a = p.s;
  a.Hkv = c->shape.num_kv_heads;
  a.W = c->shape.window;
  a.T = bt->cu_seqlens[bt->batch];
  a.radius = c->params.radius;
  a.pool_half = c->params.pool_kernel / 2;
  a.pool_mode = c->params.pool_mode;
  a.rho = c->params.rho;
  a.gamma = c->params.gamma;
  a.eps = c->params.eps;
  a.use_last_query = c->params.use_last_query;
  a.terms = c->params.terms;
  p.in_B = d_B;
  a.vec_B = d_B;
  {
    // outputs over B: the stages after the first read a copy
    const uintptr_t bytes = (uintptr_t)a.Hkv * a.T * sizeof(float), b0 = reinterpret_cast<uintptr_t>(d_B);
    for (const float *o : {d_S, d_E, d_V, d_lambda}) {
      const uintptr_t o0 = reinterpret_cast<uintptr_t>(o);
      if (o && o0 < b0 + bytes && b0 < o0 + bytes) a.vec_B = p.copy_B = reinterpret_cast<float *>(c->ws + L.vec_b);
    }
  }
  a.ring = reinterpret_cast<float *>(c->ws + L.ring);
  a.ring_stride = (int64_t)a.Hkv * a.T;
  a.ring_slots = L.slots;
  ring_slots(c, layer, &a.ring_slot, &a.ring_cnt);
  a.vec_V = reinterpret_cast<float *>(c->ws + L.vec_v);
  a.hist_B = reinterpret_cast<unsigned *>(c->ws + L.hist_s);
  a.listB_key = reinterpret_cast<unsigned *>(c->ws + L.list_bk);
  a.listB_pos = reinterpret_cast<int *>(c->ws + L.list_bp);
  a.listB_v = reinterpret_cast<float *>(c->ws + L.list_bv);
  a.cntB = reinterpret_cast<int *>(c->ws + L.cnt_b);
  a.recB = reinterpret_cast<int4 *>(c->ws + L.rec_b);
  a.lambda_ws = reinterpret_cast<float *>(c->ws + L.lambda);
  a.out_lambda = d_lambda;
  p.in_Q = d_Q;
  p.out_S = d_S;
  p.out_V = d_V;
  p.out_E = d_E;
  TRY(head_table(c, bt, s, &a.hb));
  const hipError_t e = launch_zero(a.hist_B, (int64_t)bt->batch * a.Hkv * kHRow, s);
  if (e != hipSuccess) return hip_fail(e, "clear");
  for (int stage = 0; stage < 3; ++stage)
    TRY(timed(c, KI_SPLIT_CALIB, s, [&] { return launch_split(stage, p, st, s); }));
  c->next_layer = layer + 1;
  return BACON_OK;
}

bacon_status bacon_select_topk(bacon_ctx *c, const bacon_batch *bt, const float *d_S,
                               int32_t *d_idx, void *stream) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  TRY(check_batch(c, bt));
  TRY(check_ptr(d_S, "S", 4));
  TRY(check_ptr(d_idx, "idx", 4));
  hipStream_t s = static_cast<hipStream_t>(stream);
  int chunk = 0;
  const SeqTable st = make_table(c, bt, &chunk);
  TRY(check_split(bt));
  SelArgs a{};
  a.Hkv = c->shape.num_kv_heads;
  a.W = c->shape.window;
  a.T = bt->cu_seqlens[bt->batch];
  a.pool_half = c->params.pool_kernel / 2;
  a.pool_mode = c->params.pool_mode;
  a.in_S = d_S;
  a.idx = d_idx;
  TRY(head_table(c, bt, s, &a.hb));
  return timed(c, KI_SEL_TOPK, s, [&] { return launch_select(a, st, s); });
}

bacon_status bacon_allocate_heads(bacon_ctx *c, const bacon_batch *bt, const float *d_B,
                                  int32_t *d_budgets, void *stream) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  TRY(check_batch(c, bt));
  TRY(check_ptr(d_B, "B", 4));
  TRY(check_ptr(d_budgets, "budgets", 4));
  if (bt->head_budgets)
    return fail(BACON_ERR_INVALID, "the adaptive allocation takes per-sequence budgets, not head_budgets");
  if (c->shape.num_kv_heads > 32)
    return fail(BACON_ERR_UNSUPPORTED, "the adaptive allocation takes at most 32 KV heads");
  hipStream_t s = static_cast<hipStream_t>(stream);
  int chunk = 0;
  const SeqTable st = make_table(c, bt, &chunk);
  AllocArgs a = alloc_args(c, bt->cu_seqlens[bt->batch], 0);
  a.vec_B = d_B;
  a.out = d_budgets;
  // the histogram is zero before the pool job, here and for a prompt's layers
  auto clear = [&] {
    return launch_zero(a.hist_A, (int64_t)(c->L.hist_a_stride / sizeof(unsigned)), s);
  };
  hipError_t e = clear();
  if (e != hipSuccess) return hip_fail(e, "clear");
  for (int stage = 0; stage < 3; ++stage)
    TRY(timed(c, KI_ALLOC, s, [&] { return launch_alloc(stage, a, st, s); }));
  e = clear();
  return e == hipSuccess ? BACON_OK : hip_fail(e, "clear");
}

bacon_status bacon_alloc_output(bacon_ctx *c, int32_t *d_budgets) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  if (d_budgets) TRY(check_ptr(d_budgets, "budgets", 4));
  c->alloc_out = d_budgets;
  return BACON_OK;
}

bacon_status bacon_compact(bacon_ctx *c, const bacon_batch *bt, const void *d_k, const void *d_v,
                           const int32_t *d_idx, void *d_k_out, void *d_v_out, void *stream) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  TRY(check_batch(c, bt));
  TRY(check_ptr(d_k, "k", 16));
  TRY(check_ptr(d_v, "v", 16));
  TRY(check_ptr(d_idx, "idx", 4));
  TRY(check_ptr(d_k_out, "k_out", 16));
  TRY(check_ptr(d_v_out, "v_out", 16));
  hipStream_t s = static_cast<hipStream_t>(stream);
  int chunk = 0;
  const SeqTable st = make_table(c, bt, &chunk);
  CompactArgs a{};
  a.idx = d_idx;
  a.k = d_k;
  a.v = d_v;
  a.k_out = d_k_out;
  a.v_out = d_v_out;
  a.Hkv = c->shape.num_kv_heads;
  a.W = c->shape.window;
  a.row_bytes = c->shape.head_dim * (c->shape.dtype == BACON_BF16 ? 2 : 4);
  TRY(head_table(c, bt, s, &a.hb));
  return timed(c, KI_COMPACT, s, [&] { return launch_compact(a, st, s); });
}

}  // extern "C"

namespace {

// Everything the launches of one layer of the fused pass need.
struct LayerRun {
  int layer = 0;
  bool bf16 = false, w32 = false, kr = false, single = false;
  bool wide = false;       // wide passes (small grids)
  bool adaptive = false;   // head-wise budgets from the adaptive allocation
  int chunk = 0, kmax = 0;
  int parts_alone = 1;     // final workgroups per (sequence, KV head) in a launch of their own
  int parts_mega = 1;      // and beside every other stage
  SeqTable st{};
  PassArgs a{};
  SegArgs g{};
  AllocArgs al{};
  const float *lse = nullptr;   // caller normalisers (pass 1 skipped)
};

// Checks one layer's arguments and builds its launch arguments; enqueues
// nothing.  The layer order is the caller's to check.  Buffers that later
// layers may write while this layer's select is still in flight come in
// copies that the layers take in turn: as few as the schedule needs, so that
// they stay in the caches (histograms four layers old, with the keys of four
// layers read since, cost an fp32 layer call of 36569 tokens 5 us in pass 2's
// atomics), and the first alone in a layer call, which leaves none in use.
bacon_status plan_layer(bacon_ctx *c, int32_t layer, const bacon_batch *bt, const void *d_q_win,
                        const void *d_k, const void *d_v, const float *d_lse, int32_t *d_idx,
                        void *d_k_out, void *d_v_out, LayerRun &r, bool alone) {
  TRY(check_batch(c, bt));
  TRY(check_prompt_batch(c, bt));
  if (layer >= c->shape.num_layers)
    return fail(BACON_ERR_ORDER, "layer %d beyond num_layers %d", layer, c->shape.num_layers);
  TRY(check_ptr(d_q_win, "q_win", 16));
  TRY(check_ptr(d_k, "k", 16));
  TRY(check_ptr(d_v, "v", 16));
  TRY(check_ptr(d_idx, "idx", 4));
  TRY(check_ptr(d_k_out, "k_out", 16));
  TRY(check_ptr(d_v_out, "v_out", 16));
  r.layer = layer;
  r.lse = d_lse;
  r.bf16 = c->shape.dtype == BACON_BF16;
  r.w32 = c->shape.window == 32;
  // key-register passes where they cover the shape, else the streaming passes
  r.kr = !c->kr_off && kr_supported(r.bf16, c->shape.head_dim, c->L.rpad);
  if (r.kr) {
    r.st = make_table(c, bt, &r.chunk, kr_keys(r.bf16, c->shape.head_dim));
  } else {
    r.st = make_table(c, bt, &r.chunk);
    TRY(check_lds(c, r.chunk));
  }
  // One read of K (the single-read pass) when its meeting can complete:
  // workgroups run in grid order, chunk-major with the KV heads innermost,
  // so at most the groups of one sequence are incomplete at a time, and
  // all their chunks must fit on the GPU at once.  It pays where the whole
  // grid is resident at once and fills at least half of the GPU's slots:
  // a grid that runs in rounds stalls at every sequence split across them,
  // and a small one leaves the GPU idle through the meeting, where the two-
  // pass path overlaps two layers in each launch.  With normalisers given by
  // the caller the key-register pass 2 alone already reads K once.
  if (r.kr && !d_lse && c->single_mode != 0) {
    if (c->single_cap < 0) c->single_cap = single_resident_blocks(c->shape.head_dim, c->L.rpad);
    int nmax = 0;
    for (int b = 0; b < bt->batch; ++b) nmax = std::max(nmax, r.st.chunk_base[b + 1] - r.st.chunk_base[b]);
    const int64_t hkv = c->shape.num_kv_heads, grid = (int64_t)r.st.total_chunks * hkv;
    r.single = (int64_t)nmax * hkv <= c->single_cap &&
               (c->single_mode == 1 || (grid <= c->single_cap && 2 * grid >= c->single_cap));
  }
  // small grids take the wide passes
  const bool kr_shape = kr_supported(r.bf16, c->shape.head_dim, c->L.rpad);
  int split = 1, cpw = 1;
  if (!c->kr_off && !r.single) r.wide = wide_plan(c, bt, d_lse ? WIDE_GIVEN : WIDE_FUSED, &split, &cpw);
  if (r.wide && alone && d_lse && !kr_shape && stream_given(c, bt)) r.wide = false;
  if (r.wide) {
    r.kr = false;
    r.st = make_table(c, bt, &r.chunk, wide_keys(split));
  }
  r.kmax = 0;
  for (int b = 0; b < bt->batch; ++b) r.kmax = std::max(r.kmax, batch_seq_rows(bt, c->shape.num_kv_heads, b));
  r.adaptive = c->params.head_alloc == BACON_ALLOC_ADAPTIVE;
  if (r.adaptive) {
    if (bt->head_budgets)
      return fail(BACON_ERR_INVALID, "the adaptive allocation takes per-sequence budgets, not head_budgets");
    if (c->shape.num_kv_heads > 32)
      return fail(BACON_ERR_UNSUPPORTED, "the adaptive allocation takes at most 32 KV heads");
    // a head may take up to all H_kv K_b slots of its sequence, at most its candidates
    for (int b = 0; b < bt->batch; ++b) {
      const int nc = bt->cu_seqlens[b + 1] - bt->cu_seqlens[b] - c->shape.window;
      r.kmax = std::max(r.kmax, (int)std::min<int64_t>(nc, (int64_t)c->shape.num_kv_heads * bt->budgets[b]));
    }
  }
  if (final_lds_bytes(r.kmax, c->shape.window) > (size_t)kLdsBytes)
    return fail(BACON_ERR_UNSUPPORTED, "budget %d needs more LDS than a CU has", r.kmax);
  const int turn = alone ? 0 : layer;
  const size_t c2 = turn % kCopies2, cS = turn % kCopiesS;
  const int64_t T = bt->cu_seqlens[bt->batch];
  PassArgs &a = r.a;
  a = pass_args(c, r.st, r.chunk, d_q_win, d_k);
  a.T = T;
  a.lse_in = d_lse;
  a.hist_B += turn % copies_hist_b(r.wide, r.adaptive) * c->L.hist_b_stride / sizeof(unsigned);
  a.vec_B += turn % copies_b(r.wide, r.adaptive) * c->L.vec_stride / sizeof(float);
  a.partials += c2 * c->L.part_stride / sizeof(float2);
  a.lse2 += c2 * c->L.lse_stride / sizeof(float);
  a.kr_sums = kr_shape;
  wide_args(c, a, split, cpw, r.st);
  int ring_cnt = 0;
  ring_slots(c, layer, &a.ring_write, &ring_cnt);
  a.ring_stride = (int64_t)c->shape.num_kv_heads * T;
  SegArgs &g = r.g;
  g = SegArgs{};
  g.Hkv = c->shape.num_kv_heads;
  g.W = c->shape.window;
  g.T = T;
  g.radius = c->params.radius;
  g.pool_half = c->params.pool_kernel / 2;
  g.pool_mode = c->params.pool_mode;
  g.rho = c->params.rho;
  g.gamma = c->params.gamma;
  g.eps = c->params.eps;
  // B of the single-read pass is formed from probabilities stored in fp16
  // (unit roundoff 2^-11); the passes that keep them in fp32 leave B exact
  g.b_floor = r.single ? 0x1p-11f : 0.f;
  g.use_last_query = c->params.use_last_query;
  g.terms = c->params.terms;
  g.vec_B = a.vec_B;
  g.ring = a.ring;
  g.ring_stride = a.ring_stride;
  g.ring_slots = c->L.slots;
  g.ring_slot = a.ring_write;
  g.ring_cnt = ring_cnt;
  g.vec_V = reinterpret_cast<float *>(c->ws + c->L.vec_v + c2 * c->L.vec_stride);
  g.vec_pB = reinterpret_cast<float *>(c->ws + c->L.vec_pb + c2 * c->L.vec_stride);
  g.vec_pV = reinterpret_cast<float *>(c->ws + c->L.vec_pv + c2 * c->L.vec_stride);
  g.vec_S = reinterpret_cast<unsigned *>(c->ws + c->L.vec_s + cS * c->L.vec_stride);
  g.hist_B = a.hist_B;
  g.hist_S = reinterpret_cast<unsigned *>(c->ws + c->L.hist_s + cS * c->L.hist_s_stride);
  char *lists = c->ws + c2 * c->L.list_stride;
  g.listB_key = reinterpret_cast<unsigned *>(lists + c->L.list_bk);
  g.listB_pos = reinterpret_cast<int *>(lists + c->L.list_bp);
  g.listB_v = reinterpret_cast<float *>(lists + c->L.list_bv);
  g.listS_key = reinterpret_cast<unsigned *>(lists + c->L.list_sk);
  g.listS_pos = reinterpret_cast<int *>(lists + c->L.list_sp);
  g.cntB = reinterpret_cast<int *>(c->ws + c->L.cnt_b + c2 * c->L.cnt_stride);
  g.cntS = reinterpret_cast<int *>(c->ws + c->L.cnt_s + c2 * c->L.cnt_stride);
  g.recB = reinterpret_cast<int4 *>(c->ws + c->L.rec_b + c2 * c->L.rec_stride);
  g.recS = reinterpret_cast<int4 *>(c->ws + c->L.rec_s + c2 * c->L.rec_stride);
  g.lambda_ws = reinterpret_cast<float *>(c->ws + c->L.lambda);
  g.idx = d_idx;
  g.k = d_k;
  g.v = d_v;
  g.k_out = d_k_out;
  g.v_out = d_v_out;
  g.row_bytes = c->shape.head_dim * (r.bf16 ? 2 : 4);
  g.flat_heads = r.adaptive;
  if (r.adaptive) {
    r.al = alloc_args(c, T, turn);
    r.al.vec_B = a.vec_B;
    r.al.out = c->alloc_out ? c->alloc_out + (size_t)layer * c->shape.max_batch * c->shape.num_kv_heads : nullptr;
    g.hist_A = r.al.hist_A;
    g.hb = r.al.hb;
  }
  // final workgroups per (sequence, KV head): up to eight.  Beside the other
  // jobs of a prompt call's select launch, no more than keep the launch to
  // the rounds over the GPU that one part per head needs (two 1024-thread
  // workgroups per CU): a batch whose other jobs fill it would take more
  // rounds with every part.
  {
    const int hkv = c->shape.num_kv_heads, heads = std::max(1, bt->batch * hkv), cus = device_cus(c);
    // calibration, scores and candidate lists (and the allocation's jobs)
    const int others = (r.adaptive ? 5 : 3) * r.st.total_segs * hkv;
    auto rounds = [&](int p) { return (others + p * heads + 2 * cus - 1) / (2 * cus); };
    int p = std::max(1, std::min(8, cus / heads));
    r.parts_alone = p;
    auto rounds_mega = [&](int q) {
      return (others + 2 * r.a.wide_jobs * hkv + q * heads + cus - 1) / cus;
    };
    int pm = p;
    while (pm > 1 && rounds_mega(pm) > rounds_mega(1)) --pm;
    r.parts_mega = pm;
    while (p > 1 && rounds(p) > rounds(1)) --p;
    g.parts = p;
  }
  return BACON_OK;
}

// The K passes of a layer.  lse_merged: its pass 1 ran with the previous
// layer's pass 2 and its normalisers are merged.  next (NULL or the next
// layer's pass 1 arguments): that pass 1 runs in this layer's pass-2 launch
// (bf16 keys; fp32 keys: in a launch right after it).
bacon_status stage_pass(bacon_ctx *c, const LayerRun &r, bool lse_merged, const PassArgs *next,
                        hipStream_t s) {
  const int d = c->shape.head_dim;
  if (r.single)
    return timed(c, KI_SINGLE, s, [&] { return launch_single(d, r.w32, r.a, r.st, s); });
  if (r.wide) {
    // a chunk per workgroup: nothing else shares the launch
    PassArgs a = r.a;
    a.wide_cpw_log = 0;
    a.wide_jobs = r.st.total_chunks;
    if (!r.lse) TRY(timed(c, KI_LSE_WIDE, s, [&] { return launch_wide(PASS_LSE, r.bf16, d, a, r.st, s); }));
    return timed(c, KI_FUSED_WIDE, s, [&] { return launch_wide(PASS_FUSED, r.bf16, d, a, r.st, s); });
  }
  if (r.kr) {
    if (!r.lse && !lse_merged) {
      TRY(timed(c, KI_LSE_KR, s, [&] { return launch_krpass(PASS_LSE, r.bf16, d, false, r.a, r.st, s); }));
      TRY(timed(c, KI_MERGE, s, [&] { return launch_lse_merge(r.a, r.st, s); }));
    }
    if (next)
      return timed(c, KI_DUAL_KR, s, [&] { return launch_krdual(r.bf16, d, r.w32, r.a, *next, r.st, s); });
    return timed(c, KI_FUSED_KR, s, [&] { return launch_krpass(PASS_FUSED, r.bf16, d, r.w32, r.a, r.st, s); });
  }
  if (!r.lse && !lse_merged) {
    TRY(timed(c, KI_LSE, s, [&] { return launch_pass(PASS_LSE, r.bf16, d, false, r.a, r.st, s); }));
    TRY(timed(c, KI_MERGE, s, [&] { return launch_lse_merge(r.a, r.st, s); }));
  }
  if (next && r.bf16)
    return timed(c, KI_DUAL, s, [&] { return launch_pass_dual(r.bf16, d, r.w32, r.a, *next, r.st, s); });
  TRY(timed(c, KI_FUSED, s, [&] { return launch_pass(PASS_FUSED, r.bf16, d, r.w32, r.a, r.st, s); }));
  if (next)   // fp32 keys: the next layer's pass 1 in a launch of its own
    return timed(c, KI_LSE, s, [&] { return launch_pass(PASS_LSE, r.bf16, d, false, *next, r.st, s); });
  return BACON_OK;
}

// Head-wise budgets of r's layer from its window score (adaptive allocation
// only), before its calibration reads them.
bacon_status stage_alloc(bacon_ctx *c, const LayerRun &r, hipStream_t s) {
  if (!r.adaptive) return BACON_OK;
  for (int stage = 0; stage < 3; ++stage)
    TRY(timed(c, KI_ALLOC, s, [&] { return launch_alloc(stage, r.al, r.st, s); }));
  return BACON_OK;
}

// The layers of the stages that one launch holds (NULL: none): passes 1 and 2,
// the allocation's three jobs, the four select jobs.
struct Stages {
  const LayerRun *p1 = nullptr, *p2 = nullptr, *pool = nullptr, *list = nullptr, *pick = nullptr,
                 *cal = nullptr, *score = nullptr, *cand = nullptr, *fin = nullptr;
  const PassArgs *merge = nullptr;    // the next layer's row normalisers
  int count() const {
    int n = merge != nullptr;
    for (const LayerRun *r : {p1, p2, pool, list, pick, cal, score, cand, fin}) n += r != nullptr;
    return n;
  }
  const LayerRun *any() const {
    for (const LayerRun *r : {p1, p2, pool, list, pick, cal, score, cand, fin})
      if (r) return r;
    return nullptr;
  }
  // f: storage for the final job's arguments with `parts` workgroups per head
  SelJobs jobs(SegArgs &f, int parts) const {
    SelJobs j;
    j.cal = cal ? &cal->g : nullptr;
    j.score = score ? &score->g : nullptr;
    j.cand = cand ? &cand->g : nullptr;
    j.merge = merge;
    j.pool = pool ? &pool->al : nullptr;
    j.list = list ? &list->al : nullptr;
    j.pick = pick ? &pick->al : nullptr;
    if (fin) {
      f = fin->g;
      f.parts = parts;
      j.fin = &f;
      j.fin_budget = fin->kmax;
    }
    return j;
  }
};

// One select launch: the jobs of the given layers and the next layer's row
// normalisers (the layers share the sequences, so any of their tables serves;
// the budgets come with each layer's own arguments).
bacon_status stage_select(bacon_ctx *c, const Stages &g, hipStream_t s) {
  const int njobs = g.count();
  const LayerRun *any = g.any();
  if (!any) return BACON_OK;
  SegArgs f;
  const SelJobs j = g.jobs(f, g.fin ? (njobs == 1 ? g.fin->parts_alone : g.fin->g.parts) : 0);
  const int kid = njobs > 1 || !(g.cal || g.score || g.cand || g.fin) ? KI_SEL
                  : g.cal ? KI_SEGCAL : g.score ? KI_SEGSCORE : g.cand ? KI_SEGCAND : KI_FINAL;
  return timed(c, kid, s, [&] { return launch_sel(j, any->st, s); });
}

// One launch with any of the stages, each of its own layer.
bacon_status stage_mega(bacon_ctx *c, const Stages &g, hipStream_t s) {
  const LayerRun *any = g.any();
  if (!any) return BACON_OK;
  SegArgs f;
  const SelJobs j = g.jobs(f, g.fin ? g.fin->parts_mega : 0);
  return timed(c, KI_MEGA, s, [&] {
    return launch_mega(any->bf16, c->shape.head_dim, j, g.p2 ? &g.p2->a : nullptr, g.p1 ? &g.p1->a : nullptr,
                       any->st, s);
  });
}

// Test instrumentation: once r's layer has its lambda (after its score
// stage), copies B, V and lambda into the capture buffers, before a later
// launch overwrites them.
bacon_status stage_capture(bacon_ctx *c, const LayerRun &r, const bacon_batch *bt, hipStream_t s) {
  if (!c->cap_B) return BACON_OK;
  const size_t vec = (size_t)c->shape.num_kv_heads * (size_t)bt->cu_seqlens[bt->batch];
  const size_t sc = (size_t)bt->batch * c->shape.num_kv_heads;
  hipError_t e = hipMemcpyAsync(c->cap_B + (size_t)r.layer * vec, r.g.vec_B, vec * sizeof(float),
                                hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(c->cap_V + (size_t)r.layer * vec, r.g.vec_V, vec * sizeof(float),
                       hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(c->cap_lambda + (size_t)r.layer * sc, r.g.lambda_ws, sc * sizeof(float),
                       hipMemcpyDeviceToDevice, s);
  return e == hipSuccess ? BACON_OK : hip_fail(e, "capture");
}

// The fused pass of one layer; d_lse (caller normalisers) skips pass 1.
bacon_status compress(bacon_ctx *c, int32_t layer, const bacon_batch *bt, const void *d_q_win,
                      const void *d_k, const void *d_v, const float *d_lse, int32_t *d_idx,
                      void *d_k_out, void *d_v_out, void *stream) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  if (layer != c->next_layer)
    return fail(BACON_ERR_ORDER, "layer %d given, layer %d expected next", layer, c->next_layer);
  LayerRun r;
  TRY(plan_layer(c, layer, bt, d_q_win, d_k, d_v, d_lse, d_idx, d_k_out, d_v_out, r, true));
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (!r.adaptive) TRY(head_table(c, bt, s, &r.g.hb, layer % kCopiesTab));
  TRY(stage_pass(c, r, false, nullptr, s));
  TRY(stage_alloc(c, r, s));
  Stages cal, score, cand, fin;
  cal.cal = score.score = cand.cand = fin.fin = &r;
  TRY(stage_select(c, cal, s));
  TRY(stage_select(c, score, s));
  TRY(stage_capture(c, r, bt, s));
  TRY(stage_select(c, cand, s));
  TRY(stage_select(c, fin, s));
  c->next_layer = layer + 1;
  return BACON_OK;
}

}  // namespace

extern "C" {

bacon_status bacon_compress_layer(bacon_ctx *c, int32_t layer, const bacon_batch *bt,
                                  const void *d_q_win, const void *d_k, const void *d_v,
                                  int32_t *d_idx, void *d_k_out, void *d_v_out, void *stream) {
  return compress(c, layer, bt, d_q_win, d_k, d_v, nullptr, d_idx, d_k_out, d_v_out, stream);
}

bacon_status bacon_compress_layer_lse(bacon_ctx *c, int32_t layer, const bacon_batch *bt,
                                      const void *d_q_win, const void *d_k, const void *d_v,
                                      const float *d_lse, int32_t *d_idx, void *d_k_out,
                                      void *d_v_out, void *stream) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  TRY(check_ptr(d_lse, "lse", 4));
  return compress(c, layer, bt, d_q_win, d_k, d_v, d_lse, d_idx, d_k_out, d_v_out, stream);
}

bacon_status bacon_compress_prompt(bacon_ctx *c, const bacon_batch *bt, int32_t first_layer,
                                   int32_t num_layers, const void *const *d_q_win,
                                   const void *const *d_k, const void *const *d_v,
                                   const float *const *d_lse, int32_t *const *d_idx,
                                   void *const *d_k_out, void *const *d_v_out,
                                   const bacon_batch *const *layer_batch, void *stream) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  if (num_layers < 1) return fail(BACON_ERR_INVALID, "num_layers %d must be >= 1", num_layers);
  if (!d_q_win || !d_k || !d_v || !d_idx || !d_k_out || !d_v_out)
    return fail(BACON_ERR_INVALID, "a per-layer pointer array is NULL");
  if (first_layer != c->next_layer)
    return fail(BACON_ERR_ORDER, "layer %d given, layer %d expected next", first_layer, c->next_layer);
  if ((int64_t)first_layer + num_layers > c->shape.num_layers)
    return fail(BACON_ERR_ORDER, "layers %d..%d beyond num_layers %d", first_layer,
                first_layer + num_layers - 1, c->shape.num_layers);
  // every layer's arguments are checked before the first launch
  for (int i = 0; i < num_layers; ++i) {
    TRY(check_ptr(d_q_win[i], "q_win", 16));
    TRY(check_ptr(d_k[i], "k", 16));
    TRY(check_ptr(d_v[i], "v", 16));
    TRY(check_ptr(d_idx[i], "idx", 4));
    TRY(check_ptr(d_k_out[i], "k_out", 16));
    TRY(check_ptr(d_v_out[i], "v_out", 16));
    if (d_lse) TRY(check_ptr(d_lse[i], "lse", 4));
  }
  // every layer is planned (and checked) before the first launch; a layer
  // takes its own batch (budgets) when layer_batch is given
  auto lbt = [&](int i) { return layer_batch ? layer_batch[i] : bt; };
  if (layer_batch)
    for (int i = 0; i < num_layers; ++i)
      if (!layer_batch[i]) return fail(BACON_ERR_INVALID, "layer_batch[%d] is NULL", i);
  std::vector<LayerRun> runs(num_layers);
  for (int i = 0; i < num_layers; ++i)
    TRY(plan_layer(c, first_layer + i, lbt(i), d_q_win[i], d_k[i], d_v[i],
                   d_lse ? d_lse[i] : nullptr, d_idx[i], d_k_out[i], d_v_out[i], runs[i], false));
  hipStream_t s = static_cast<hipStream_t>(stream);
  // Layers in flight at once.  Small grids: one launch per layer holds pass 1
  // of layer i, pass 2 of layer i - 1 (which merges the normalisers), and the
  // stages that follow, each of the layer before.  Others: the select launch
  // that follows layer i's K passes holds its calibration, the scores of layer
  // i - 1, the candidate lists of i - 2 and the final job of i - 3, and layer
  // i + 1's pass 1 runs in the launch of layer i's pass 2.  The adaptive
  // allocation's three jobs come between pass 2 and the calibration.  The last
  // launches have no K pass.
  auto at = [&](int i) -> const LayerRun * { return i >= 0 && i < num_layers ? &runs[i] : nullptr; };
  const bool wide = runs[0].wide, adaptive = runs[0].adaptive;   // (the layers share the sequences)
  const Lags lag = stage_lags(wide, runs[0].lse != nullptr, adaptive);
  bool merged = false;
  for (int i = 0; i < num_layers + lag.fin; ++i) {
    Stages g;
    if (i < num_layers) {
      LayerRun &r = runs[i];
      if (layer_batch) TRY(seq_table(c, r.st, s, &r.g.sb, r.layer % kCopiesTab));
      if (adaptive) r.al.sb = r.g.sb;
      else TRY(head_table(c, lbt(i), s, &r.g.hb, r.layer % kCopiesTab));
      c->next_layer = r.layer + 1;
      if (!wide) {
        // the next layer's pass 1 rides in this layer's pass-2 launch, unless the
        // next layer reads K once (single-read pass) or has its normalisers given
        if (!r.lse && !r.single && i + 1 < num_layers && !runs[i + 1].single) g.merge = &runs[i + 1].a;
        TRY(stage_pass(c, r, merged, g.merge, s));
        merged = g.merge != nullptr;
      }
    }
    if (wide) {
      if (!runs[0].lse) g.p1 = at(i - lag.p1);
      g.p2 = at(i - lag.p2);
    }
    if (adaptive) {
      g.pool = at(i - lag.pool);
      g.list = at(i - lag.list);
      g.pick = at(i - lag.pick);
    }
    g.cal = at(i - lag.cal);
    g.score = at(i - lag.score);
    g.cand = at(i - lag.cand);
    g.fin = at(i - lag.fin);
    TRY(wide ? stage_mega(c, g, s) : stage_select(c, g, s));
    if (g.score) TRY(stage_capture(c, *g.score, lbt(i - lag.score), s));
  }
  return BACON_OK;
}

}  // extern "C"

namespace {

// The window-row normalisers of one layer: pass 1 and the merge.  With
// scratch NULL the per-chunk partials and merged normalisers go to the
// context's workspace; otherwise to scratch (scratch_bytes long), which is
// checked before anything is enqueued.
bacon_status window_lse(bacon_ctx *c, const bacon_batch *bt, const void *d_q_win, const void *d_k,
                        float *d_lse, void *stream, char *scratch, size_t scratch_bytes,
                        bool lookup_scratch) {
  TRY(check_batch(c, bt));
  TRY(check_ptr(d_q_win, "q_win", 16));
  TRY(check_ptr(d_k, "k", 16));
  TRY(check_ptr(d_lse, "lse", 4));
  hipStream_t s = static_cast<hipStream_t>(stream);
  const bool bf16 = c->shape.dtype == BACON_BF16;
  int chunk = 0;
  SeqTable st{};
  const bool kr = !c->kr_off && kr_supported(bf16, c->shape.head_dim, c->L.rpad);
  if (kr) {
    st = make_table(c, bt, &chunk, kr_keys(bf16, c->shape.head_dim));
  } else {
    st = make_table(c, bt, &chunk);
    TRY(check_lds(c, chunk));
  }
  PassArgs a = pass_args(c, st, chunk, d_q_win, d_k);
  a.T = bt->cu_seqlens[bt->batch];
  a.lse_user = d_lse;
  if (lookup_scratch) {
    // partials [Hkv, chunks, Rpad] float2, then the merged normalisers [B, Hkv, Rpad]
    const size_t part = align256((size_t)c->shape.num_kv_heads * st.total_chunks * c->L.rpad * sizeof(float2));
    const size_t need = part + align256((size_t)bt->batch * c->shape.num_kv_heads * c->L.rpad * sizeof(float));
    if (need > scratch_bytes)
      return fail(BACON_ERR_WORKSPACE, "the batch needs %zu bytes of scratch; the static scratch holds %zu",
                  need, scratch_bytes);
    void *p = nullptr;
    const hipError_t e = static_scratch(&p);
    if (e != hipSuccess) return hip_fail(e, "static scratch");
    scratch = static_cast<char *>(p);
    a.partials = reinterpret_cast<float2 *>(scratch);
    a.lse2 = reinterpret_cast<float *>(scratch + part);
  }
  if (kr) {
    TRY(timed(c, KI_LSE_KR, s, [&] { return launch_krpass(PASS_LSE, bf16, c->shape.head_dim, false, a, st, s); }));
  } else {
    TRY(timed(c, KI_LSE, s, [&] { return launch_pass(PASS_LSE, bf16, c->shape.head_dim, false, a, st, s); }));
  }
  TRY(timed(c, KI_MERGE, s, [&] { return launch_lse_merge(a, st, s); }));
  return BACON_OK;
}

}  // namespace

extern "C" {

bacon_status bacon_window_lse(bacon_ctx *c, const bacon_batch *bt, const void *d_q_win,
                              const void *d_k, float *d_lse, void *stream) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  return window_lse(c, bt, d_q_win, d_k, d_lse, stream, nullptr, 0, false);
}

bacon_status bacon_window_lse_static(const bacon_shape *shape, const bacon_batch *bt,
                                     const void *d_q_win, const void *d_k, float *d_lse,
                                     void *stream) {
  // a context on the stack, over no workspace: nothing is allocated
  TRY(check_shape(shape));
  bacon_ctx c;
  c.shape = *shape;
  bacon_default_params(&c.params);
  c.L = layout_of(shape, &c.params);
  c.ws = nullptr;
  c.ws_bytes = 0;
  return window_lse(&c, bt, d_q_win, d_k, d_lse, stream, nullptr, kStaticScratchBytes, true);
}

int32_t bacon_debug_device_errors(bacon_ctx *c) {
  if (!c || !c->ws) return -1;
  unsigned v = 0;
  const size_t off = c->L.sync + (size_t)kSyncStride * c->shape.max_batch * c->shape.num_kv_heads * sizeof(unsigned);
  if (hipDeviceSynchronize() != hipSuccess ||
      hipMemcpy(&v, c->ws + off, sizeof(v), hipMemcpyDeviceToHost) != hipSuccess)
    return -1;
  return (int32_t)v;
}

bacon_status bacon_debug_capture(bacon_ctx *c, float *d_B, float *d_V, float *d_lambda) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  const int set = (d_B != nullptr) + (d_V != nullptr) + (d_lambda != nullptr);
  if (set != 0 && set != 3) return fail(BACON_ERR_INVALID, "give all three capture buffers or none");
  if (set) {
    TRY(check_ptr(d_B, "B", 4));
    TRY(check_ptr(d_V, "V", 4));
    TRY(check_ptr(d_lambda, "lambda", 4));
  }
  c->cap_B = d_B;
  c->cap_V = d_V;
  c->cap_lambda = d_lambda;
  return BACON_OK;
}

int64_t bacon_idx_count(const bacon_batch *bt, int32_t num_kv_heads) {
  if (!bt || (!bt->budgets && !bt->head_budgets) || bt->batch < 1 || num_kv_heads < 1) return 0;
  int64_t n = 0;
  for (int b = 0; b < bt->batch; ++b)
    for (int h = 0; h < num_kv_heads; ++h) n += batch_head_budget(bt, num_kv_heads, b, h);
  return n;
}

int64_t bacon_kept_rows(const bacon_batch *bt, int32_t num_kv_heads, int32_t window) {
  if (!bt || (!bt->budgets && !bt->head_budgets) || bt->batch < 1 || num_kv_heads < 1) return 0;
  int64_t n = 0;
  for (int b = 0; b < bt->batch; ++b) n += batch_seq_rows(bt, num_kv_heads, b) + window;
  return n;
}

bacon_status bacon_profile_enable(bacon_ctx *c, int32_t enable) {
  if (!c) return fail(BACON_ERR_INVALID, "ctx is NULL");
  if (enable && c->ev_pool.empty()) {
    c->ev_pool.resize(16384);
    for (auto &e : c->ev_pool) {
      // timing-only events: no system-scope cache write-back when recorded
      const hipError_t r = hipEventCreateWithFlags(&e, hipEventDisableSystemFence);
      if (r != hipSuccess) return hip_fail(r, "hipEventCreate");
    }
  }
  c->prof = enable != 0;
  return BACON_OK;
}

int32_t bacon_profile_read(bacon_ctx *c, bacon_kernel_time *out, int32_t max) {
  if (!c) return -1;
  for (const auto &p : c->pending) {
    float ms = 0.f;
    if (hipEventSynchronize(p.b) == hipSuccess && hipEventElapsedTime(&ms, p.a, p.b) == hipSuccess) {
      c->ms[p.kid] += ms;
      c->launches[p.kid] += 1;
    }
  }
  c->pending.clear();
  c->ev_next = 0;
  int n = 0;
  for (int k = 0; k < KI_COUNT && n < max; ++k) {
    if (!c->launches[k]) continue;
    if (out) {
      std::snprintf(out[n].name, sizeof out[n].name, "%s", kKernelNames[k]);
      out[n].launches = c->launches[k];
      out[n].total_ms = c->ms[k];
    }
    ++n;
  }
  return n;
}

const char *bacon_status_string(bacon_status s) {
  switch (s) {
    case BACON_OK: return "ok";
    case BACON_ERR_INVALID: return "invalid argument";
    case BACON_ERR_UNSUPPORTED: return "unsupported";
    case BACON_ERR_ORDER: return "layer out of order";
    case BACON_ERR_WORKSPACE: return "workspace too small";
    case BACON_ERR_HIP: return "HIP error";
  }
  return "unknown status";
}

const char *bacon_last_error(void) { return g_err.c_str(); }

}  // extern "C"
