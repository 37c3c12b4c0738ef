// C ABI of libprsgd: host-side driver of Algorithm 1 (and the epochs of Algorithms 2 and 3).
// Only argument checking, buffer carving and kernel sequencing live here; every arithmetic
// step of the method runs in the kernels.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <memory>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "prsgd_aux.h"
#include "prsgd_internal.h"

using namespace prsgd;

namespace prsgd {
const char* kernel_kind_name(int kind) {
  static const char* names[KK_COUNT] = {"gather",  "gemm_fwd", "softmax_xent", "gemm_dx",   "gemm_dw",
                                        "sgd_update", "average", "mean",       "broadcast", "lsq_steps",
                                        "mlp2_epoch", "gemm_bwd", "restart_mean", "step_mean", "gemm_bwd_first", "refresh_shadow"};
  return (kind >= 0 && kind < KK_COUNT) ? names[kind] : "?";
}
}  // namespace prsgd

namespace {

constexpr size_t kAlign = 256;
size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

thread_local char g_init_error[256] = "";

struct Carve {
  size_t xb = 0, yb = 0, idx = 0, xb2 = 0, yb2 = 0, idx2 = 0, logits = 0, losses = 0, row_loss = 0, part = 0, sync = 0, shadow = 0, grads = 0, mean = 0, mean_shadow = 0, steps = 0, vel = 0, exchange = 0;
  size_t h[PRSGD_MAX_DIMS] = {0}, delta[PRSGD_MAX_DIMS] = {0};
  size_t total = 0;
  bool spare_part = false;    // the exchange of the epoch kernel keeps one set of partial logits where that is enough
};

bool build_layout(const prsgd_config* c, Layout* lo, char* err, size_t errn) {
  auto fail = [&](const char* msg) { snprintf(err, errn, "%s", msg); return false; };
  if (c == nullptr) return fail("config is null");
  if (c->n_workers < 1 || c->n_workers > 65535) return fail("n_workers out of range");
  if (c->batch < 1 || c->batch > kMaxBatch) return fail("batch out of range (1..4096)");
  if (c->rows_per_worker < 1 || c->rows_per_worker > (1LL << 31) ||
      (c->rows_per_worker & (c->rows_per_worker - 1)) != 0)
    return fail("rows_per_worker must be a power of two");
  if (!(c->lr == c->lr)) return fail("lr is NaN");
  if (!(c->momentum >= 0.0f && c->momentum < 1.0f)) return fail("momentum must be in [0, 1)");
  if (c->momentum_restart < PRSGD_MOM_KEEP || c->momentum_restart > PRSGD_MOM_RESET)
    return fail("unknown momentum_restart");
  memset(lo, 0, sizeof(*lo));
  if (c->model == PRSGD_LSQ) {
    if (c->n_dims != 1) return fail("least squares takes n_dims == 1");
    if (c->dims[0] < 1 || c->dims[0] > kMaxLsqDim) return fail("least-squares dimension out of range");
    lo->n_layers = 0;
    lo->d[0] = c->dims[0];
    lo->ld[0] = c->dims[0];
    lo->m = c->dims[0];
    lo->m_pad = (long)align_up((size_t)c->dims[0], 64);
    return true;
  }
  if (c->model != PRSGD_MLP) return fail("unknown model");
  if (c->n_dims < 2 || c->n_dims > PRSGD_MAX_DIMS) return fail("an MLP takes 2..16 dims");
  if (c->activation != PRSGD_TANH && c->activation != PRSGD_RELU) return fail("unknown activation");
  if (c->gemm_dtype != PRSGD_F32 && c->gemm_dtype != PRSGD_BF16) return fail("unknown gemm_dtype");
  lo->n_layers = c->n_dims - 1;
  long off = 0, m = 0;
  for (int l = 0; l < c->n_dims; ++l) {
    if (c->dims[l] < 1 || c->dims[l] > (1 << 20)) return fail("layer width out of range");
    lo->d[l] = c->dims[l];
    // rows of 8 elements; wide layers (>= 512) are padded to whole 64-column tiles so that the
    // whole-tile kernels apply to them (the padding columns hold zeros and stay zero)
    lo->ld[l] = (int)align_up((size_t)c->dims[l], (l > 0 && c->dims[l] >= 512) ? 64 : 8);
  }
  for (int l = 1; l < c->n_dims; ++l) {
    lo->w_off[l - 1] = off;
    off = (long)align_up((size_t)off + (size_t)lo->d[l - 1] * lo->ld[l], 64);
    lo->b_off[l - 1] = off;
    off = (long)align_up((size_t)off + (size_t)lo->ld[l], 64);
    m += (long)lo->d[l - 1] * lo->d[l] + lo->d[l];
  }
  lo->m = m;
  lo->m_pad = off;
  return true;
}

// Momentum (v <- mu v + G, x <- x - gamma v) is fused into the one-pass backward kernel of the
// bf16 configurations and into the epoch kernel of the one-hidden-layer fp32 MLPs; elsewhere the
// gradients go to HBM and an elementwise kernel applies it.
bool bwd_fused_config(const prsgd_config& c) {
  return c.model == PRSGD_MLP && c.gemm_dtype == PRSGD_BF16 && c.fused_update &&
         prsgd::bwd_fused_supported(c.batch);
}
// shapes the epoch kernel may take (whether it does is decided at init, on the device)
bool epoch_candidate(const prsgd_config& c) {
  return c.model == PRSGD_MLP && c.gemm_dtype == PRSGD_F32 && c.n_dims == 3 && c.fused_update &&
         prsgd::fused2_shape(c.n_workers, c.dims[0], c.dims[1], c.dims[2], c.batch, c.momentum != 0.0f);
}
prsgd_config effective_config(const prsgd_config* c) {
  prsgd_config e = *c;
  if (e.momentum != 0.0f && !bwd_fused_config(e) && !epoch_candidate(e)) e.fused_update = 0;
  return e;
}

// Replica sets from here on are streamed (non-temporal weight loads and stores).  An iteration rewrites the
// whole set, so that past most of the 256 MB last-level cache a line is gone before it is needed again.
// Replicas of 3072-1024-1024-10 at interval 16, per iteration, cached and streamed: 10 (161 MiB) 107 and 110 us, 11 119
// and 119 us, 12 (193 MiB) 138 and 126 us, 16 149 and 146 us (with momentum 262 and 258 us), 32 288 and 279 us.
constexpr size_t kStreamingBytes = (size_t)192 << 20;

// Which launches of a configuration are streamed.
struct Streamed {
  bool rows;          // drawn rows of the shards
  bool steps;         // local steps: they rewrite the replica set
  bool step_mean;     // a step on the node average: the average is all it rewrites, and the next iteration reads
                      // it again (16 x (3072-1024-1024-10) at interval 1, an average of 17 MB: 78 us per iteration, 84
                      // streamed; 2 x (4096-4096-4096-4096-1000), 218 MB: 302 us, 295 streamed)
  bool mean;          // the average written apart: with up to four workers it writes 6 bytes for the next iteration
                      // to every 16 or fewer that it reads, and streamed reads lose (2 x (4096-4096-4096-10), 257 MiB at
                      // interval 2: 239 us per iteration, 251 streamed; 8 x (2048-2048-2048-10), as large: 167 us, 156
                      // streamed)
  bool average;       // the average written to every replica, which the next iteration reads: pays from well past
                      // the cache on (fp32 at interval 4, 28 x (1024-1024-1024-10), 226 MiB: 191 us, 194 streamed; 2 x
                      // (4096-4096-4096-10), 257 MiB: 262 and 277 us; 12 x (2048-2048-2048-10), 386 MiB: 341 and 332 us)
};
// Shards from here on: a drawn row is gone from the last-level cache before it is drawn again, and in passing made room there (8 workers of
// 4096-4096-4096-4096-1000, shards of 1 GB, 15850 -> 15805 us per 16 iterations, 16 of 3072-1024-1024-10 4470 -> 4410 per 32).
constexpr size_t kStreamingRowBytes = (size_t)256 << 20;
constexpr size_t kStreamingMeanFewBytes = (size_t)1 << 30, kStreamingAverageBytes = (size_t)384 << 20;
Streamed streamed_uses(const prsgd_config& c, const Layout& lo) {
  const size_t average = (size_t)lo.m_pad * sizeof(float), set = average * (size_t)c.n_workers;
  Streamed u;
  u.steps = set >= kStreamingBytes;
  u.step_mean = average >= kStreamingBytes;
  u.mean = set >= (c.n_workers > 4 ? kStreamingBytes : kStreamingMeanFewBytes);
  u.average = set >= kStreamingAverageBytes;
  u.rows = u.steps && (size_t)c.n_workers * (size_t)c.rows_per_worker * (size_t)lo.d[0] * sizeof(float) >= kStreamingRowBytes;
  return u;
}

// `scratch`: PRSGD_SCRATCH_RUNS, or without what a configuration can do without: what keeps restarts inside a launch (they are
// launches of their own then), and what the epoch kernel exchanges (local steps are the chain of per-layer launches then).
void build_carve(const prsgd_config* c_in, const Layout& lo, int scratch, Carve* cv) {
  const prsgd_config eff = effective_config(c_in);
  const prsgd_config* c = &eff;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, kAlign); return o; };
  const size_t n = (size_t)c->n_workers, b = (size_t)c->batch;
  const bool bf16 = c->model == PRSGD_MLP && c->gemm_dtype == PRSGD_BF16;
  const size_t es = bf16 ? 2 : 4;
  cv->idx = take(n * b * 4);
  cv->losses = take(n * 4);
  cv->steps = take(n * 4);
  cv->mean = take((size_t)lo.m_pad * 4 + (c->model == PRSGD_LSQ ? kAlign : 0));   // least squares: abort flag behind it
  if (c->momentum != 0.0f) cv->vel = take(n * (size_t)lo.m_pad * 4);
  if (scratch >= PRSGD_SCRATCH_RUNS && c->model == PRSGD_LSQ && lsq_restarts_in_launch(c->n_workers, lo.d[0], c->batch)) {
    cv->sync = take(4);
    cv->exchange = take(lsq_exchange_bytes(c->n_workers, lo.d[0]));
  }
  if (c->model == PRSGD_MLP) {
    const int L = lo.n_layers;
    cv->yb = take(n * b * 4);
    cv->row_loss = take(n * b * 4);
    cv->xb = take(n * b * lo.ld[0] * es);
    // second set: the next iteration's minibatch is gathered while the current one is in use
    cv->xb2 = take(n * b * lo.ld[0] * es);
    cv->yb2 = take(n * b * 4);
    cv->idx2 = take(n * b * 4);
    for (int l = 1; l < L; ++l) {
      cv->h[l] = take(n * b * lo.ld[l] * es);
      cv->delta[l] = take(n * b * lo.ld[l] * es);
    }
    cv->delta[L] = take(n * b * lo.ld[L] * es);
    cv->logits = take((size_t)kMaxLogitSplits * n * b * lo.ld[L] * 4);   // room for split partial sums
    if (bf16) {
      cv->shadow = take(n * (size_t)lo.m_pad * 2);
      cv->mean_shadow = take((size_t)lo.m_pad * 2);
    }
    if (scratch >= PRSGD_SCRATCH_EPOCHS && epoch_candidate(*c)) {
      // epoch kernel: partial logits, numbers of the exchanges, abort flag; for restarts inside a launch flags behind
      // them, and the slices on their way
      const size_t members = n * (((size_t)lo.d[1] + 15) / 16);
      const size_t exchange = scratch < PRSGD_SCRATCH_RUNS ? 0 : fused2_exchange_floats(c->n_workers, lo.d[0], lo.d[1], lo.d[2]);
      const size_t flags = exchange == 0 ? 0 : 16 * (size_t)fused2_flag_stride((int)(members < 4096 ? members : 4096));
      cv->part = take(fused2_part_slots(c->n_workers, lo.d[1], lo.d[2], c->batch, scratch < PRSGD_SCRATCH_RUNS) * 8);
      cv->spare_part = scratch < PRSGD_SCRATCH_RUNS;
      cv->sync = take((n + 1) * 128 + flags);
      if (exchange != 0) cv->exchange = take(exchange * 4);
    }
    // un-fused update; also the fallback of a momentum run whose epoch kernel does not fit the device
    if (!c->fused_update || (c->momentum != 0.0f && !bwd_fused_config(*c)))
      cv->grads = take(n * (size_t)lo.m_pad * 4);
  }
  cv->total = off;
}
// The most scratch that prsgd_init_static has room for (PRSGD_SCRATCH_LAYERS also where even that is too much).
int static_scratch(const prsgd_config* cfg, const Layout& lo, Carve* cv) {
  for (int scratch = PRSGD_SCRATCH_RUNS;; --scratch) {
    *cv = Carve();
    build_carve(cfg, lo, scratch, cv);
    if (cv->total <= PRSGD_STATIC_WORKSPACE_BYTES || scratch == PRSGD_SCRATCH_LAYERS) return scratch;
  }
}

struct EventPair { hipEvent_t a, b; int kind; };

}  // namespace

struct prsgd_ctx {
  prsgd_config cfg;
  Layout lo;
  Carve cv;
  bool bf16;
  bool use_fused2;      // one-hidden-layer fp32 MLP: whole epochs in one launch
  // contexts whose launches have workgroups that wait for each other: the list of all of them, and what the rules of
  // launches beside each other need of this one
  bool enlisted;
  prsgd_ctx* next_waiting;
  int wait_dev, wait_team;     // device, workgroups per worker
  long wait_places;            // workgroups that an XCD of it holds, one per compute unit
  hipEvent_t wait_event;       // behind its newest launch (nullptr: none recorded), and that launch's place among all
  uint64_t wait_seq;
  bool ran_pinned;             // launches of it, maybe still under way, had teams pinned because its stream was the only one
  int64_t n_whole, n_followed; // launches with restarts inside; launches of other streams that this one's stream waited for
  bool restarts_in_launch;   // whole runs in one launch: its workgroups exchange the points at a restart
  Fused2Plan f2;
  Streamed streamed;    // launches whose weight traffic is marked non-temporal
  bool lazy_restart;    // a restart only writes the node average; the next local iteration
                        // reads it as every worker's starting point (no broadcast)
  bool at_mean;         // the replicas are stale: every worker's current point is the vector `mean`
  bool poisoned;        // the epoch kernel gave up a team barrier: the replicas are inconsistent
                        // until the caller restores them (prsgd_write_params)
  unsigned char restored[65536 / 8];   // bit i: worker i written since the abort
  size_t n_restored;
  unsigned int spin_limit;      // polls of the epoch kernel's team barrier before it gives up
  hipStream_t stream;
  const float* features;
  const void* targets;
  float* params;
  char* ws;
  int64_t t;
  // two minibatch buffer sets (layer-wise MLP path): batch_t[k] is the iteration whose draw set k
  // holds for ALL workers (-1: none), batch_cur the set of the last local iteration
  int64_t batch_t[2];
  int batch_cur;
  // first hidden activation computed ahead by the first layer's backward kernel: valid for
  // iteration h1_t on batch set h1_batch while the replicas are untouched (-1: none)
  int64_t h1_t;
  int h1_batch;
  bool recorded;      // calls were recorded into a graph, whose replays move the points and rewrite the minibatch sets unseen by the host
  bool restart_fusion;  // prsgd_run: take an epoch's last iteration and the restart as one pass
  bool first_fusion;    // let the first layer's backward kernel run the next forward product
  bool shadow1_stale;   // that kernel skipped the bf16 shadow of W_1 (nothing reads it while the
                        // chain of ahead-computed activations holds): refresh before any other reader
  float lr;
  char err[256];
  // profiling
  bool profiling;
  std::vector<EventPair> pool;
  size_t pool_used;
  double prof_ms[KK_COUNT];
  int64_t prof_n[KK_COUNT];
  // scratch host buffer for padded <-> dense parameter conversion
  float* host_pad;                    // [m_pad + 1]
  std::vector<float> host_pad_heap;   // owns it, unless the context lives in static storage
  int static_slot;                    // >= 0: context, workspace and host_pad are the per-device
                                      // static ones of prsgd_init_static

  template <typename T> T* at(size_t off) const { return reinterpret_cast<T*>(ws + off); }
  void* xb(int k) const { return at<void>(k ? cv.xb2 : cv.xb); }
  int32_t* yb(int k) const { return at<int32_t>(k ? cv.yb2 : cv.yb); }
  int32_t* idx(int k) const { return at<int32_t>(k ? cv.idx2 : cv.idx); }
  uint16_t* shadow() const { return bf16 ? at<uint16_t>(cv.shadow) : nullptr; }
  float* mean() const { return at<float>(cv.mean); }
  float* velocity() const { return cfg.momentum != 0.0f ? at<float>(cv.vel) : nullptr; }
  uint16_t* mean_shadow() const { return bf16 ? at<uint16_t>(cv.mean_shadow) : nullptr; }
  // where a worker's current point is read from, and the stride between workers
  const float* src() const { return at_mean ? mean() : params; }
  long src_stride() const { return at_mean ? 0 : lo.m_pad; }
  // configurations whose first local iteration can start from the shared node average
  bool can_start_from_mean() const {
    return cfg.model == PRSGD_LSQ || use_fused2 ||
           (bf16 && cfg.fused_update && prsgd::bwd_fused_supported(cfg.batch));
  }
  // local steps are launches of single layers
  bool layered() const { return cfg.model == PRSGD_MLP && !use_fused2; }
  // set by a launch whose workgroups gave up waiting for each other (nullptr: no such launches)
  unsigned int* abort_flag() const {
    if (use_fused2) return at<unsigned int>(cv.sync) + (size_t)cfg.n_workers * 32;
    if (cfg.model == PRSGD_LSQ && restarts_in_launch) return reinterpret_cast<unsigned int*>(mean() + lo.m_pad);
    return nullptr;
  }
  float* grads() const { return cfg.fused_update ? nullptr : at<float>(cv.grads); }
};

namespace {

int set_err(prsgd_ctx* ctx, int code, const char* fmt, const char* detail = "") {
  if (ctx != nullptr) snprintf(ctx->err, sizeof(ctx->err), fmt, detail);
  else snprintf(g_init_error, sizeof(g_init_error), fmt, detail);
  return code;
}
int hip_fail(prsgd_ctx* ctx, hipError_t e, const char* what) {
  char buf[200];
  snprintf(buf, sizeof(buf), "%s: %s", what, hipGetErrorString(e));
  return set_err(ctx, PRSGD_EHIP, "%s", buf);
}

// Drains finished event pairs into the per-kind totals.
int profile_flush(prsgd_ctx* ctx) {
  if (ctx->pool_used == 0) return PRSGD_OK;
  hipError_t e = hipStreamSynchronize(ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "hipStreamSynchronize");
  for (size_t i = 0; i < ctx->pool_used; ++i) {
    float ms = 0.0f;
    e = hipEventElapsedTime(&ms, ctx->pool[i].a, ctx->pool[i].b);
    if (e != hipSuccess) return hip_fail(ctx, e, "hipEventElapsedTime");
    ctx->prof_ms[ctx->pool[i].kind] += ms;
    ctx->prof_n[ctx->pool[i].kind] += 1;
  }
  ctx->pool_used = 0;
  return PRSGD_OK;
}

// Brackets one kernel launch with an event pair while profiling is on.
struct Timed {
  prsgd_ctx* ctx;
  EventPair* ep = nullptr;
  Timed(prsgd_ctx* c, int kind) : ctx(c) {
    if (!c->profiling) return;
    if (c->pool_used == c->pool.size() && profile_flush(c) != PRSGD_OK) return;
    ep = &c->pool[c->pool_used++];
    ep->kind = kind;
    (void)hipEventRecord(ep->a, c->stream);
  }
  ~Timed() {
    if (ep != nullptr) (void)hipEventRecord(ep->b, ctx->stream);
  }
};

#define LAUNCH(ctx, kind, call)                                        \
  do {                                                                 \
    hipError_t e_;                                                     \
    {                                                                  \
      Timed timed_(ctx, kind);                                         \
      e_ = (call);                                                     \
    }                                                                  \
    if (e_ != hipSuccess) return hip_fail(ctx, e_, kernel_kind_name(kind)); \
  } while (0)

int materialize(prsgd_ctx* ctx);
void strike_waiting(prsgd_ctx* ctx);
bool is_capturing(hipStream_t stream, bool unknown = true);

// bf16 shadow of W_1 of every replica from its fp32 master (after first-layer kernels that skipped it)
int refresh_first_shadow(prsgd_ctx* ctx) {
  const Layout& lo = ctx->lo;
  const long count = (long)lo.d[0] * lo.ld[1];
  for (int i = 0; i < ctx->cfg.n_workers; ++i) {
    const size_t off = (size_t)i * lo.m_pad + lo.w_off[0];
    LAUNCH(ctx, KK_REFRESH, launch_refresh_shadow(ctx->params + off, ctx->shadow() + off, count, ctx->stream));
  }
  ctx->shadow1_stale = false;
  return PRSGD_OK;
}

// Weight-gradient products of one backward pass.  They wait for each other and share a launch: they
// read H and D of their layers, which stay as they are until the next iteration, and write W_l after
// the backward-data product that needs its old value.
struct DwQueue {
  prsgd_ctx* ctx;
  GemmArgs ps[kMaxGemmSet];
  int n = 0, n_groups = 0, kind = 0;
  explicit DwQueue(prsgd_ctx* c) : ctx(c) {}
  int flush() {
    if (n == 0) return PRSGD_OK;
    const int count = n;
    n = 0;
    LAUNCH(ctx, kind, launch_gemm_dw(ps, count, n_groups, ctx->bf16, ctx->stream));
    return PRSGD_OK;
  }
  int add(const GemmArgs& p, int groups, int k) {
    if (n == kMaxGemmSet) {
      const int rc = flush();
      if (rc != PRSGD_OK) return rc;
    }
    ps[n++] = p;
    n_groups = groups;
    kind = k;
    return PRSGD_OK;
  }
};

// Workers that take an iteration (Algorithm 3), and those for which it may prepare the next one.  By falling step counts, the
// workers that go on are the first of those that take the present step, so that a launch has workgroups for them only.  With a
// workgroup of every worker that ended at once for the others, workers of unlike speed also left XCDs idle: one to four steps of
// worker i after i mod 4 had their last step on two of eight (two epochs of 16 workers of
// 3072-1024-1024-10, 64 rows: 1250 -> 1010 us, with the first layer fused for those that go on).
struct Active {
  const int* order = nullptr;   // device: workers by falling step counts (nullptr: every worker, in its own place)
  int now = 0;                  // order[0 .. now) take this iteration
  const int* next_order = nullptr;
  int next = 0;                 // next_order[0 .. next) also take the following one, whose minibatch is drawn ahead
  int idx_set = -1;             // batch set whose row numbers a masked draw writes: the last ones of every worker stand together
};

// One local iteration of every (active) MLP worker: gradient observation + eq. (3).
// fuse_average: this iteration is followed by a restart, and both are taken together,
//   (1/N) sum_i (x_i - gamma G_i) = ybar - (gamma / N) sum_i G_i,   ybar = (1/N) sum_i x_i   (eq. 2-3).
// The backward pass contracts over the stacked minibatches of all workers and writes only the new
// ybar; the replicas are not rewritten and the context ends "at the mean".  With every worker
// already at ybar (I = 1) it is one mini-batch SGD step with the N B samples of all workers (first
// footnote of Section 1).
// The workers that go on have the minibatch of the next iteration drawn, and its first activation computed where that pays.
int mlp_step(prsgd_ctx* ctx, int64_t t, const Active& active, bool fuse_average = false) {
  const prsgd_config& c = ctx->cfg;
  const Layout& lo = ctx->lo;
  const Carve& cv = ctx->cv;
  const int* order = active.order;
  const int N = active.now, B = c.batch, L = lo.n_layers;
  const bool bf16 = ctx->bf16;
  hipStream_t s = ctx->stream;

  // The minibatch of iteration t: already there when the previous iteration's loss-head launch
  // drew it (below); otherwise gathered now.  prsgd_local_steps_hetero forgets masked draws at the end of an epoch.
  auto batch_args = [&](int k, int64_t tt, const int* workers, int n) {
    GatherArgs a = gather_args(ctx->features, reinterpret_cast<const int32_t*>(ctx->targets), ctx->xb(k), ctx->yb(k),
                               ctx->idx(workers != nullptr && active.idx_set >= 0 ? active.idx_set : k), B, lo.d[0], lo.ld[0],
                               (long)c.rows_per_worker, c.seed, tt, workers, n);
    a.once = ctx->streamed.rows ? 1 : 0;
    return a;
  };
  int bk = ctx->batch_t[0] == t ? 0 : ctx->batch_t[1] == t ? 1 : -1;
  if (bk < 0) {
    bk = ctx->batch_cur;
    ctx->batch_t[bk] = -1;
    LAUNCH(ctx, KK_GATHER, launch_gather(batch_args(bk, t, order, N), bf16, s));
    ctx->batch_t[bk] = t;
  }
  ctx->batch_cur = bk;

  GemmArgs base;
  memset(&base, 0, sizeof(base));
  base.act = c.activation;
  base.lr = ctx->lr;
  base.params = ctx->params;
  base.grads = ctx->grads();
  base.shadow = ctx->shadow();
  base.p_gs = lo.m_pad;
  base.order = order;
  base.streaming = ctx->streamed.steps ? 1 : 0;

  auto act_in = [&](int l) -> const void* {   // H_l as stored (l = 0: the gathered batch)
    return l == 0 ? ctx->xb(bk) : ctx->at<void>(cv.h[l]);
  };
  const bool fused_bwd = bf16 && c.fused_update && bwd_fused_supported(B);
  // Right after a restart every worker starts from the shared node average (stride 0); only
  // the fused backward kernel writes complete replicas from it, so every other path first
  // broadcasts the average.  A masked worker (Algorithm 3) would keep a stale replica.
  if (ctx->at_mean && (!fused_bwd || order != nullptr)) {
    const int rc = materialize(ctx);
    if (rc != PRSGD_OK) return rc;
  }
  const bool from_mean = ctx->at_mean;
  const long w_gs = from_mean ? 0 : lo.m_pad;
  // The matrix products read weights from the bf16 shadow (bf16 mode) or the fp32 master.
  const void* wsrc = bf16 ? (const void*)(from_mean ? ctx->mean_shadow() : ctx->shadow())
                          : (const void*)ctx->params;
  base.src = ctx->src();
  base.src_gs = ctx->src_stride();

  // forward.  H_1 may already be there: the previous iteration's first-layer backward kernel computes
  // it from the weights it writes, for this iteration's minibatch
  const bool h1_ready = fused_bwd && !from_mean && L >= 2 && ctx->h1_t == t && ctx->h1_batch == bk;
  ctx->h1_t = -1;
  if (!h1_ready && ctx->shadow1_stale && !from_mean) {
    const int rc = refresh_first_shadow(ctx);
    if (rc != PRSGD_OK) return rc;
  }
  int logit_parts = 1;
  const long logit_part_stride = (long)c.n_workers * B * lo.ld[L];
  // a narrow logits layer is multiplied inside the loss-head launch
  const bool narrow_head = softmax_narrow_applies(lo.d[L], lo.ld[L], lo.d[L - 1], bf16);
  for (int l = 1; l <= L; ++l) {
    if (l == 1 && h1_ready) continue;
    if (l == L && narrow_head) continue;
    GemmArgs p = base;
    p.a = act_in(l - 1); p.a_gs = (long)B * lo.ld[l - 1]; p.lda = lo.ld[l - 1];
    p.b = bf16 ? (const void*)(reinterpret_cast<const uint16_t*>(wsrc) + lo.w_off[l - 1])
               : (const void*)(reinterpret_cast<const float*>(wsrc) + lo.w_off[l - 1]);
    p.b_gs = w_gs; p.ldb = lo.ld[l];
    p.M = B; p.N = lo.d[l]; p.Kc = lo.d[l - 1];
    p.b_off = lo.b_off[l - 1];
    p.out_gs = (long)B * lo.ld[l]; p.ldo = lo.ld[l]; p.out_cols = lo.ld[l];
    if (l < L) { p.epi = EPI_FWD_HIDDEN; p.out = ctx->at<void>(cv.h[l]); }
    else {
      p.epi = EPI_FWD_LOGITS; p.out = ctx->at<void>(cv.logits);
      logit_parts = gemm_logit_splits(p, N, bf16);
      p.k_splits = logit_parts; p.split_stride = logit_part_stride;
    }
    LAUNCH(ctx, KK_FWD, launch_gemm_fwd(p, N, bf16, s));
  }

  auto bwd_args = [&](int l) {
    BwdArgs q;
    memset(&q, 0, sizeof(q));
    q.h = reinterpret_cast<const uint16_t*>(act_in(l - 1)); q.h_gs = (long)B * lo.ld[l - 1]; q.ldh = lo.ld[l - 1];
    q.d = ctx->at<uint16_t>(cv.delta[l]); q.d_gs = (long)B * lo.ld[l]; q.ldd = lo.ld[l];
    q.params = ctx->params; q.shadow = ctx->shadow(); q.p_gs = lo.m_pad;
    q.src = ctx->src(); q.src_gs = ctx->src_stride();
    q.w_off = lo.w_off[l - 1]; q.b_off = lo.b_off[l - 1]; q.ldw = lo.ld[l];
    if (l > 1) { q.dx = ctx->at<uint16_t>(cv.delta[l - 1]); q.dx_gs = (long)B * lo.ld[l - 1]; q.lddx = lo.ld[l - 1]; }
    q.B = B; q.K = lo.d[l - 1]; q.Nn = lo.d[l];
    q.n_groups = N; q.act = c.activation; q.streaming = ctx->streamed.steps ? 1 : 0;
    q.lr = ctx->lr;
    q.vel = ctx->velocity(); q.mu = c.momentum;
    q.order = order;
    return q;
  };
  // the first layer's pass that also runs the next forward product, for the workers that go on
  const bool prefetch = active.next > 0;
  auto first_args = [&]() {
    BwdArgs q = bwd_args(1);
    q.x_next = reinterpret_cast<const uint16_t*>(ctx->xb(bk ^ 1)); q.x_gs = (long)B * lo.ld[0]; q.ldx = lo.ld[0];
    q.h_next = ctx->at<uint16_t>(cv.h[1]); q.hn_gs = (long)B * lo.ld[1]; q.ldhn = lo.ld[1];
    q.order = active.next_order;
    q.n_groups = active.next;
    return q;
  };
  const bool first_fused = fused_bwd && !fuse_average && L >= 2 && ctx->first_fusion && prefetch && bwd_first_fwd_applies(first_args());
  int n_apart = 0, widest_apart = 0;
  for (int l = L; fused_bwd && l >= (first_fused ? 2 : 1); --l) {
    if (!bwd_products_apart(bwd_args(l))) continue;
    ++n_apart;
    if (lo.d[l] > widest_apart) widest_apart = lo.d[l];
  }
  const bool take_apart = bwd_apart_pays(n_apart, widest_apart, B);
  // A narrow head takes the last layer's delta one layer down as well, where that is a product of its own and faster so.  With up
  // to 16 classes it stays one where the layers' products are apart, because test_backward_launches_of_ragged_layers counts the
  // backward launches of such nets; it is not the faster way (300-253-10, eight workers, 64 rows 15.6 us per iteration apart and 14.1
  // in the head; 16 workers, 128 rows 20.1 and 18.8).
  const bool head_delta = narrow_head && L > 1 &&
                          softmax_narrow_delta_pays(lo.ld[L], lo.d[L - 1], softmax_narrow_blocks(N, B), bf16) &&
                          (fuse_average || !fused_bwd || (lo.d[L] > 16 && take_apart && bwd_products_apart(bwd_args(L))));

  // the loss-head launch also draws the minibatch of iteration t + 1 into the other buffer set
  GatherArgs next_batch = batch_args(bk ^ 1, t + 1, active.next_order, active.next);
  if (prefetch) ctx->batch_t[bk ^ 1] = -1;
  HeadDelta below;
  memset(&below, 0, sizeof(below));
  if (head_delta) {
    below.out = ctx->at<void>(cv.delta[L - 1]); below.gs = (long)B * lo.ld[L - 1]; below.ld = lo.ld[L - 1];
    below.act = c.activation;
  }
  if (narrow_head)
    LAUNCH(ctx, KK_LOSS,
           launch_softmax_xent_narrow(act_in(L - 1), (long)B * lo.ld[L - 1], lo.ld[L - 1], lo.d[L - 1],
                                      bf16 ? (const void*)(reinterpret_cast<const uint16_t*>(wsrc) + lo.w_off[L - 1])
                                           : (const void*)(reinterpret_cast<const float*>(wsrc) + lo.w_off[L - 1]),
                                      w_gs, ctx->src() + lo.b_off[L - 1], ctx->src_stride(), ctx->yb(bk),
                                      ctx->at<void>(cv.delta[L]), ctx->at<float>(cv.row_loss), N, B, lo.d[L],
                                      lo.ld[L], bf16, order, prefetch ? &next_batch : nullptr,
                                      head_delta ? &below : nullptr, s));
  else
  LAUNCH(ctx, KK_LOSS,
         launch_softmax_xent(ctx->at<float>(cv.logits), logit_parts, logit_part_stride,
                             logit_parts > 1 ? ctx->src() + lo.b_off[L - 1] : nullptr, ctx->src_stride(),
                             ctx->yb(bk),
                             ctx->at<void>(cv.delta[L]), ctx->at<float>(cv.row_loss), N, B, lo.d[L],
                             lo.ld[L], bf16, order, prefetch ? &next_batch : nullptr, s));
  if (prefetch) ctx->batch_t[bk ^ 1] = t + 1;

  // products of layer l: D_{l-1} = (D_l W_l^T) phi'(H_{l-1}) and dW_l = H_{l-1}^T D_l
  auto dx_args = [&](int l) {
    GemmArgs p = base;
    p.a = ctx->at<void>(cv.delta[l]); p.a_gs = (long)B * lo.ld[l]; p.lda = lo.ld[l];
    p.b = bf16 ? (const void*)(reinterpret_cast<const uint16_t*>(wsrc) + lo.w_off[l - 1])
               : (const void*)(reinterpret_cast<const float*>(wsrc) + lo.w_off[l - 1]);
    p.b_gs = w_gs; p.ldb = lo.ld[l];
    p.M = B; p.N = lo.d[l - 1]; p.Kc = lo.d[l];
    p.epi = EPI_DX;
    p.out = ctx->at<void>(cv.delta[l - 1]); p.out_gs = (long)B * lo.ld[l - 1];
    p.ldo = lo.ld[l - 1]; p.out_cols = lo.ld[l - 1];
    p.aux = act_in(l - 1); p.aux_gs = (long)B * lo.ld[l - 1]; p.ldaux = lo.ld[l - 1];
    return p;
  };
  auto dw_args = [&](int l) {
    GemmArgs p = base;
    p.a = act_in(l - 1); p.a_gs = (long)B * lo.ld[l - 1]; p.lda = lo.ld[l - 1];
    p.b = ctx->at<void>(cv.delta[l]); p.b_gs = (long)B * lo.ld[l]; p.ldb = lo.ld[l];
    p.M = lo.d[l - 1]; p.N = lo.d[l]; p.Kc = B;
    p.w_off = lo.w_off[l - 1]; p.b_off = lo.b_off[l - 1]; p.ldw = lo.ld[l];
    return p;
  };
  DwQueue dw(ctx);

  if (fuse_average) {
    // The workers' points differ (the last iteration of an epoch with I >= 2, or the first
    // iteration of a run): ybar is first taken from the points as they are (the restart kernel),
    // then moved by the averaged gradient; the points themselves are not rewritten.
    if (!from_mean)
      LAUNCH(ctx, KK_RESTART_MEAN,
             launch_mean(ctx->params, ctx->mean(), ctx->mean_shadow(), lo.m_pad, N, ctx->streamed.mean, s));
    // eq. (3) and eq. (2) in one pass over ybar, layer by layer from the top: D_{l-1} needs the
    // weights the forward pass used (the bf16 image of ybar, or of every worker's own point), and
    // when that is ybar it runs before layer l's pass changes it
    for (int l = L; l >= 1; --l) {
      if (l > 1 && !(l == L && head_delta)) LAUNCH(ctx, KK_DX, launch_gemm_dx(dx_args(l), N, true, s));
      // all minibatches stacked: sum_i dW_i = [H_1; ..; H_N]^T [D_1; ..; D_N], one contraction of N B
      // rows, and ybar <- ybar - (gamma / N) sum_i dW_i (likewise the bias from the column sums)
      GemmArgs p = dw_args(l);
      p.a_gs = 0; p.b_gs = 0;
      p.Kc = N * B;
      p.epi = EPI_DW_FUSED;
      p.lr = ctx->lr / (float)N;
      p.params = ctx->mean(); p.shadow = ctx->mean_shadow(); p.p_gs = 0;
      p.src = ctx->mean(); p.src_gs = 0;
      p.streaming = ctx->streamed.step_mean ? 1 : 0;
      const int rc = dw.add(p, 1, KK_STEP_MEAN);
      if (rc != PRSGD_OK) return rc;
    }
    const int rc = dw.flush();
    if (rc != PRSGD_OK) return rc;
    ctx->at_mean = true;             // every worker's point is the new ybar; the replicas are stale
    return PRSGD_OK;
  }

  // backward.  bf16 operands with the fused update: one kernel per layer does the weight
  // gradient, eq. (3) and the delta of the layer below in a single pass over W_l.
  bool first_shadow_left = false;
  for (int l = L; fused_bwd && l >= 1; --l) {
    if (l == 1 && first_fused) {
      const int rc = dw.flush();            // H_1 is rewritten: layer 2's weight gradient still reads it
      if (rc != PRSGD_OK) return rc;
      LAUNCH(ctx, KK_BWD_FIRST, launch_bwd_first_fwd(first_args(), s));
      ctx->shadow1_stale = first_shadow_left = true;     // not written: it has no reader while H_1 comes from here
      ctx->h1_t = t + 1;
      ctx->h1_batch = bk ^ 1;
      if (N == active.next) continue;
      BwdArgs q = bwd_args(1);
      q.order = active.next_order + active.next;         // the workers that are done
      q.n_groups = N - active.next;
      LAUNCH(ctx, KK_BWD, launch_bwd_fused(q, s));
      continue;
    }
    const BwdArgs q = bwd_args(l);
    if (take_apart && bwd_products_apart(q)) {
      if (l > 1 && !(l == L && head_delta)) LAUNCH(ctx, KK_BWD, launch_gemm_dx(dx_args(l), N, true, s));
      GemmArgs p = dw_args(l);
      p.epi = EPI_DW_FUSED;
      p.vel = ctx->velocity(); p.mu = c.momentum;
      const int rc = dw.add(p, N, KK_BWD);
      if (rc != PRSGD_OK) return rc;
      continue;
    }
    LAUNCH(ctx, KK_BWD, launch_bwd_fused(q, s));
  }
  // otherwise: D_{l-1} needs the pre-update W_l, so it runs before layer l's weight kernel
  for (int l = L; !fused_bwd && l >= 1; --l) {
    if (l > 1 && !(l == L && head_delta)) LAUNCH(ctx, KK_DX, launch_gemm_dx(dx_args(l), N, bf16, s));
    GemmArgs p = dw_args(l);
    p.epi = c.fused_update ? EPI_DW_FUSED : EPI_DW_GRAD;
    const int rc = dw.add(p, N, KK_DW);
    if (rc != PRSGD_OK) return rc;
  }
  {
    const int rc = dw.flush();
    if (rc != PRSGD_OK) return rc;
  }
  // every other backward pass of layer 1 writes the shadows of the replicas it steps: those of all workers, or of those
  // whose first activation was there, which had been left
  if (fused_bwd && (order == nullptr || h1_ready) && !first_shadow_left) ctx->shadow1_stale = false;

  if (!c.fused_update) {
    if (ctx->velocity() != nullptr)
      LAUNCH(ctx, KK_UPDATE, launch_momentum_update(ctx->params, ctx->velocity(), ctx->grads(), ctx->shadow(),
                                                    (size_t)N * lo.m_pad, ctx->lr, c.momentum, s));
    else if (order == nullptr)
      LAUNCH(ctx, KK_UPDATE, launch_update(ctx->params, ctx->grads(), ctx->shadow(),
                                           (size_t)N * lo.m_pad, ctx->lr, s));
    else
      LAUNCH(ctx, KK_UPDATE, launch_update_workers(ctx->params, ctx->grads(), ctx->shadow(), lo.m_pad, order, N, ctx->lr, s));
  }
  ctx->at_mean = false;            // every parameter of every replica has been rewritten
  return PRSGD_OK;
}

// An iteration of every worker, and one behind it.  `last` one of a call: nothing is prepared behind it if the context has been recorded.
Active every_worker(const prsgd_ctx* ctx, bool last) {
  Active a;
  a.now = ctx->cfg.n_workers;
  a.next = last && ctx->recorded ? 0 : a.now;
  return a;
}

// Around every call that enqueues steps or restarts.  A graph that holds such calls takes the recorded launches again, with their buffers
// and iteration numbers, as often as it is replayed and between whatever calls, and the host learns nothing of it.  So from its first
// recording on a context hands no more than the points from one call to the next, in the replicas and with their shadows: a call's
// first step draws its own minibatch and computes its own first activation, its last one prepares nothing, and a restart at its end is
// broadcast.  (Without this a replayed step multiplied what the steps after the recording had drawn and computed ahead.)
// `steps`: up to the one whose row numbers stay the newest; they end in set 0, as those of every replay do.
void begin_call(prsgd_ctx* ctx, int64_t steps) {
  if (!ctx->recorded) ctx->recorded = is_capturing(ctx->stream, false);
  if (!ctx->recorded) return;
  ctx->batch_t[0] = ctx->batch_t[1] = -1;
  ctx->h1_t = -1;
  if (steps > 0 && ctx->layered()) ctx->batch_cur = (int)((steps - 1) & 1);
}
int end_call(prsgd_ctx* ctx) { return ctx->recorded ? materialize(ctx) : PRSGD_OK; }

Fused2Args fused2_args(prsgd_ctx* ctx, int k, const int* worker_steps) {
  const prsgd_config& c = ctx->cfg;
  const Layout& lo = ctx->lo;
  Fused2Args a;
  memset(&a, 0, sizeof(a));
  a.features = ctx->features;
  a.labels = reinterpret_cast<const int32_t*>(ctx->targets);
  a.params = ctx->params;
  a.src = ctx->src();
  a.src_stride = ctx->src_stride();
  a.m_pad = lo.m_pad;
  a.w1_off = lo.w_off[0]; a.b1_off = lo.b_off[0]; a.w2_off = lo.w_off[1]; a.b2_off = lo.b_off[1];
  a.ld1 = lo.ld[1]; a.ld2 = lo.ld[2];
  a.n_workers = c.n_workers;
  a.d0 = lo.d[0]; a.d1 = lo.d[1]; a.d2 = lo.d[2];
  a.batch = c.batch;
  a.rows = (long)c.rows_per_worker;
  a.log2n = 0;
  while ((1LL << a.log2n) < c.rows_per_worker) ++a.log2n;
  a.act = c.activation;
  a.lr = ctx->lr;
  a.seed = c.seed;
  a.t0 = (uint64_t)ctx->t;
  a.k = k;
  a.worker_steps = worker_steps;
  a.part = ctx->at<unsigned long long>(ctx->cv.part);
  a.spare_part = ctx->cv.spare_part;
  a.exchange = ctx->at<float>(ctx->cv.exchange);
  a.sync = ctx->at<unsigned int>(ctx->cv.sync);
  a.spin_limit = ctx->spin_limit;
  a.row_loss = ctx->at<float>(ctx->cv.row_loss);
  a.idx = ctx->at<int32_t>(ctx->cv.idx);
  a.vel = ctx->velocity();
  a.mu = c.momentum;
  return a;
}

LsqArgs lsq_args(prsgd_ctx* ctx, int k) {
  const prsgd_config& c = ctx->cfg;
  LsqArgs a;
  memset(&a, 0, sizeof(a));
  a.features = ctx->features;
  a.targets = reinterpret_cast<const float*>(ctx->targets);
  a.src = ctx->src(); a.src_stride = ctx->src_stride();
  a.params = ctx->params; a.m_pad = ctx->lo.m_pad;
  a.velocity = ctx->velocity(); a.mu = c.momentum;
  a.losses = ctx->at<float>(ctx->cv.losses); a.idx = ctx->at<int32_t>(ctx->cv.idx);
  a.n_workers = c.n_workers; a.d = ctx->lo.d[0]; a.rows = (long)c.rows_per_worker; a.batch = c.batch;
  a.lr = ctx->lr; a.seed = c.seed; a.t0 = (uint64_t)ctx->t; a.k = k;
  return a;
}

constexpr const char* kPoisonedMsg =
    "the epoch kernel gave up waiting for a team member (was other work running on the device?); "
    "the replicas are inconsistent: restore them with prsgd_write_params (and prsgd_set_iteration)";

// Calls that enqueue work refuse to run on replicas an aborted epoch launch left inconsistent.
int check_poisoned(prsgd_ctx* ctx) {
  return ctx->poisoned ? set_err(ctx, PRSGD_ESTATE, "%s", kPoisonedMsg) : PRSGD_OK;
}

// The epoch kernel's bounded team barrier raises a flag instead of hanging.  Called wherever the
// stream is synchronised anyway: reads the flag (4 bytes); if it is set, clears it, marks the
// context poisoned and switches every later local step to the per-layer kernel chain, which needs
// no co-resident workgroups.
int workgroups_gave_up(prsgd_ctx* ctx) {
  const unsigned int zero = 0;
  hipError_t e = hipMemcpyAsync(ctx->abort_flag(), &zero, sizeof(zero), hipMemcpyHostToDevice, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "abort-flag reset");
  if (ctx->use_fused2 && ctx->cfg.momentum != 0.0f) ctx->cfg.fused_update = 0;   // the chain applies momentum elementwise
  ctx->use_fused2 = false;
  ctx->restarts_in_launch = false;
  strike_waiting(ctx);                      // no launch of it waits any more
  ctx->poisoned = true;
  ctx->at_mean = false;
  ctx->n_restored = 0;
  memset(ctx->restored, 0, sizeof(ctx->restored));
  return set_err(ctx, PRSGD_ESTATE, "%s", kPoisonedMsg);
}
int check_gave_up(prsgd_ctx* ctx) {
  if (ctx->poisoned) return set_err(ctx, PRSGD_ESTATE, "%s", kPoisonedMsg);
  unsigned int* flag_dev = ctx->abort_flag();
  if (flag_dev == nullptr) return PRSGD_OK;
  unsigned int flag = 0;
  hipError_t e = hipMemcpyAsync(&flag, flag_dev, sizeof(flag), hipMemcpyDeviceToHost, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "abort-flag read");
  return flag == 0 ? PRSGD_OK : workgroups_gave_up(ctx);
}

// Writes the node average into every replica (and the bf16 shadow) if the last restart left the
// replicas stale.
int materialize(prsgd_ctx* ctx) {
  ctx->h1_t = -1;
  if (!ctx->at_mean) return PRSGD_OK;
  ctx->shadow1_stale = false;               // the broadcast rewrites every shadow
  LAUNCH(ctx, KK_BROADCAST, launch_broadcast(ctx->mean(), ctx->params, ctx->shadow(), ctx->lo.m_pad,
                                             ctx->cfg.n_workers, ctx->stream));
  ctx->at_mean = false;
  return PRSGD_OK;
}

int pad_from_dense(const prsgd_ctx* ctx, const float* dense, float* padded) {
  const Layout& lo = ctx->lo;
  memset(padded, 0, sizeof(float) * (size_t)lo.m_pad);
  if (lo.n_layers == 0) { memcpy(padded, dense, sizeof(float) * (size_t)lo.m); return 0; }
  size_t src = 0;
  for (int l = 1; l <= lo.n_layers; ++l) {
    for (int r = 0; r < lo.d[l - 1]; ++r) {
      memcpy(padded + lo.w_off[l - 1] + (size_t)r * lo.ld[l], dense + src, sizeof(float) * lo.d[l]);
      src += lo.d[l];
    }
    memcpy(padded + lo.b_off[l - 1], dense + src, sizeof(float) * lo.d[l]);
    src += lo.d[l];
  }
  return 0;
}
void dense_from_pad(const prsgd_ctx* ctx, const float* padded, float* dense) {
  const Layout& lo = ctx->lo;
  if (lo.n_layers == 0) { memcpy(dense, padded, sizeof(float) * (size_t)lo.m); return; }
  size_t dst = 0;
  for (int l = 1; l <= lo.n_layers; ++l) {
    for (int r = 0; r < lo.d[l - 1]; ++r) {
      memcpy(dense + dst, padded + lo.w_off[l - 1] + (size_t)r * lo.ld[l], sizeof(float) * lo.d[l]);
      dst += lo.d[l];
    }
    memcpy(dense + dst, padded + lo.b_off[l - 1], sizeof(float) * lo.d[l]);
    dst += lo.d[l];
  }
}

}  // namespace

extern "C" {

size_t prsgd_param_count(const prsgd_config* cfg) {
  Layout lo;
  char err[128];
  return build_layout(cfg, &lo, err, sizeof(err)) ? (size_t)lo.m : 0;
}
size_t prsgd_param_stride(const prsgd_config* cfg) {
  Layout lo;
  char err[128];
  return build_layout(cfg, &lo, err, sizeof(err)) ? (size_t)lo.m_pad : 0;
}
size_t prsgd_workspace_bytes(const prsgd_config* cfg) {
  Layout lo;
  char err[128];
  if (!build_layout(cfg, &lo, err, sizeof(err))) return 0;
  Carve cv;
  build_carve(cfg, lo, PRSGD_SCRATCH_RUNS, &cv);
  return cv.total;
}

}  // extern "C"

namespace {

// Workspace of prsgd_init_static: one array per device, held until the process ends.  In host
// code the array's name is only a handle for hipGetSymbolAddress; kernels and memsets get the
// device address resolved once per device below.
constexpr size_t kStaticBytes = PRSGD_STATIC_WORKSPACE_BYTES;
constexpr int kMaxStaticDevices = 8;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

struct StaticSlot {
  void* ws_dev = nullptr;             // device address of `scratch` on this device
  bool in_use = false;
  alignas(prsgd_ctx) unsigned char ctx_mem[sizeof(prsgd_ctx)];
};
StaticSlot g_static[kMaxStaticDevices];
float g_static_pad[kMaxStaticDevices][kStaticBytes / sizeof(float)];   // host staging, per device
std::mutex g_static_mutex;

// Contexts whose launches have workgroups that wait for each other, on any device.  Such a launch ends only while all that it
// waits for can be resident.  Launches of one stream follow each other; those of other streams may run beside them, and
// several half-resident grids would wait for each other until they give up.  So launches that may be under way together
// have to fit the device together, XCD by XCD, with a compute unit per workgroup (LDS and registers mostly leave no
// room for a second one):
//   - the only stream of its device: nothing runs beside it, any grid that its plan has accepted goes out;
//   - several streams that fit together: likewise, but teams are spread over the XCDs (pinned, the few workers of several
//     contexts would meet on the first XCDs: five times 2 x (784-256-10), 160 workgroups, would need 80 places on XCD 0);
//   - several that do not: a launch follows the oldest launches of other streams until those left fit beside it (stream
//     events), and restarts are launches of their own, so that a stream holds the device for an epoch at a time.
// A stream that is being captured takes no part: its launches run when the graph is launched, beside anything.
prsgd_ctx* g_waiting = nullptr;      // list of such contexts
uint64_t g_waiting_seq = 0;          // launches recorded so far
std::mutex g_waiting_mutex;

bool is_capturing(hipStream_t stream, bool unknown) {
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &capture) == hipSuccess) return capture != hipStreamCaptureStatusNone;
  (void)hipGetLastError();           // the default stream while another one is being captured
  return unknown;
}
// The rules below, with g_waiting_mutex held.  A stream is stood for by the first of its contexts in the list.
bool stands_for_stream(const prsgd_ctx* c) {
  for (const prsgd_ctx* o = g_waiting; o != c; o = o->next_waiting)
    if (o->wait_dev == c->wait_dev && o->stream == c->stream) return false;
  return true;
}
// Workgroups on the fullest XCD of the largest launch in this context's stream: from now on, or (`past`) so far.
long stream_demand(const prsgd_ctx* c, bool past) {
  long most = 0;
  for (const prsgd_ctx* o = g_waiting; o != nullptr; o = o->next_waiting)
    if (o->wait_dev == c->wait_dev && o->stream == c->stream) {
      const long need = xcd_workgroups(o->cfg.n_workers, o->wait_team, past && o->ran_pinned);
      if (need > most) most = need;
    }
  return most;
}
// Newest recorded launch of this context's stream (nullptr: none).
const prsgd_ctx* stream_newest(const prsgd_ctx* c) {
  const prsgd_ctx* newest = nullptr;
  for (const prsgd_ctx* o = g_waiting; o != nullptr; o = o->next_waiting)
    if (o->wait_dev == c->wait_dev && o->stream == c->stream && o->wait_seq != 0 &&
        (newest == nullptr || o->wait_seq > newest->wait_seq))
      newest = o;
  return newest;
}
int waiting_regime(long n_streams, long demand, long xcd_places) {
  return n_streams <= 1 ? PRSGD_WAIT_ALONE : demand <= xcd_places ? PRSGD_WAIT_TOGETHER : PRSGD_WAIT_CROWDED;
}
int waiting_regime_of(const prsgd_ctx* ctx) {
  long n_streams = 0, demand = 0;
  for (const prsgd_ctx* o = g_waiting; o != nullptr; o = o->next_waiting)
    if (o->wait_dev == ctx->wait_dev && stands_for_stream(o)) {
      ++n_streams;
      demand += stream_demand(o, false);
    }
  return waiting_regime(n_streams, demand, ctx->wait_places);
}
// Everything enqueued so far in the context's stream counts as its newest launch.
hipError_t record_waiting(prsgd_ctx* ctx) {
  if (ctx->wait_event == nullptr) {
    const hipError_t e = hipEventCreateWithFlags(&ctx->wait_event, hipEventDisableTiming);
    if (e != hipSuccess) return e;
  }
  ctx->wait_seq = ++g_waiting_seq;
  return hipEventRecord(ctx->wait_event, ctx->stream);
}
hipError_t follow(prsgd_ctx* ctx, const prsgd_ctx* newest) {
  ++ctx->n_followed;
  return hipStreamWaitEvent(ctx->stream, newest->wait_event, 0);
}
// Lets the context's stream wait for the oldest launches of other streams until those left fit beside its own.
hipError_t follow_others(prsgd_ctx* ctx) {
  long total = xcd_workgroups(ctx->cfg.n_workers, ctx->wait_team, false);
  for (const prsgd_ctx* o = g_waiting; o != nullptr; o = o->next_waiting)
    if (o->wait_dev == ctx->wait_dev && o->stream != ctx->stream && stands_for_stream(o) && stream_newest(o) != nullptr)
      total += stream_demand(o, false);
  uint64_t followed = 0;
  while (total > ctx->wait_places) {
    const prsgd_ctx* oldest = nullptr;
    for (const prsgd_ctx* o = g_waiting; o != nullptr; o = o->next_waiting) {
      if (o->wait_dev != ctx->wait_dev || o->stream == ctx->stream || !stands_for_stream(o)) continue;
      const prsgd_ctx* newest = stream_newest(o);
      if (newest != nullptr && newest->wait_seq > followed && (oldest == nullptr || newest->wait_seq < oldest->wait_seq))
        oldest = newest;
    }
    if (oldest == nullptr) return hipSuccess;
    const hipError_t e = follow(ctx, oldest);
    if (e != hipSuccess) return e;
    followed = oldest->wait_seq;
    total -= stream_demand(oldest, false);
  }
  return hipSuccess;
}

// Around one launch whose workgroups wait for each other.
struct WaitingLaunch {
  prsgd_ctx* ctx;
  std::lock_guard<std::mutex> lock;
  int regime;
  bool capturing;
  explicit WaitingLaunch(prsgd_ctx* c)
      : ctx(c), lock(g_waiting_mutex), regime(waiting_regime_of(c)), capturing(is_capturing(c->stream)) {}
  bool may_wait_as_whole() const { return !capturing && regime != PRSGD_WAIT_CROWDED; }
  bool pinned() const {
    if (ctx->cfg.n_workers % 8 == 0) return true;          // as many workgroups per XCD as spread
    if (regime != PRSGD_WAIT_ALONE || capturing || !ctx->f2.pinned_fits) return false;
    return ctx->ran_pinned = true;
  }
  hipError_t before() {
    if (capturing || regime != PRSGD_WAIT_CROWDED) return hipSuccess;
    return follow_others(ctx);
  }
  hipError_t after() { return capturing || regime != PRSGD_WAIT_CROWDED ? hipSuccess : record_waiting(ctx); }
};

// A context joins the list.  Launches under way were ordered without it.  Its own follow those of a stream that had its teams
// pinned, unless all that has been launched so far leaves them room; if the streams do not fit together any more, they follow
// others until those left do.
hipError_t enlist_waiting(prsgd_ctx* ctx, int team) {
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  ctx->wait_dev = dev;
  ctx->wait_places = cus / 8;
  ctx->wait_team = team;
  std::lock_guard<std::mutex> lock(g_waiting_mutex);
  ctx->next_waiting = g_waiting;
  g_waiting = ctx;
  ctx->enlisted = true;
  if (waiting_regime_of(ctx) == PRSGD_WAIT_ALONE) return hipSuccess;
  long total = xcd_workgroups(ctx->cfg.n_workers, team, false);
  bool past_pinned = false;
  for (const prsgd_ctx* o = g_waiting; o != nullptr; o = o->next_waiting) {
    if (o->wait_dev != dev || o->stream == ctx->stream) continue;
    past_pinned |= o->ran_pinned;
    if (stands_for_stream(o)) total += stream_demand(o, true);
  }
  const bool crowded = waiting_regime_of(ctx) == PRSGD_WAIT_CROWDED;
  past_pinned &= total > ctx->wait_places;
  if (!crowded && !past_pinned) return hipSuccess;
  for (prsgd_ctx* o = g_waiting; o != nullptr; o = o->next_waiting) {
    if (o->wait_dev != dev || o->stream == ctx->stream || is_capturing(o->stream)) continue;
    const bool pinned = past_pinned && o->ran_pinned;
    if (!pinned && !(crowded && stands_for_stream(o))) continue;
    e = record_waiting(o);
    if (e == hipSuccess && pinned) e = follow(ctx, o);
    if (e != hipSuccess) return e;
  }
  return crowded ? follow_others(ctx) : hipSuccess;
}
void strike_waiting(prsgd_ctx* ctx) {
  if (!ctx->enlisted) return;
  std::lock_guard<std::mutex> lock(g_waiting_mutex);
  for (prsgd_ctx** at = &g_waiting; *at != nullptr; at = &(*at)->next_waiting)
    if (*at == ctx) {
      *at = ctx->next_waiting;
      break;
    }
  ctx->enlisted = false;
  if (ctx->wait_event != nullptr) (void)hipEventDestroy(ctx->wait_event);
  ctx->wait_event = nullptr;
}

// k iterations of every worker in one launch of the epoch kernel.
int launch_epoch(prsgd_ctx* ctx, int k, const int* worker_steps) {
  WaitingLaunch waiting(ctx);
  hipError_t e = waiting.before();
  if (e != hipSuccess) return hip_fail(ctx, e, "order of launches that wait");
  LAUNCH(ctx, KK_FUSED2, launch_fused2(ctx->f2, fused2_args(ctx, k, worker_steps), waiting.pinned(), ctx->stream));
  e = waiting.after();
  return e == hipSuccess ? PRSGD_OK : hip_fail(ctx, e, "order of launches that wait");
}

void release_ctx(prsgd_ctx* ctx) {
  strike_waiting(ctx);
  if (ctx->static_slot < 0) { delete ctx; return; }
  const int slot = ctx->static_slot;
  ctx->~prsgd_ctx();
  std::lock_guard<std::mutex> lock(g_static_mutex);
  g_static[slot].in_use = false;
}

// Shared body of prsgd_init and prsgd_init_static.  static_slot < 0: the context goes on the heap
// and `workspace_dev` is the caller's; otherwise context, staging buffer and workspace are the
// slot's static ones and nothing is allocated.
int init_common(const prsgd_config* cfg, const float* x0_host, const void* features_dev,
                const void* targets_dev, void* params_dev, void* workspace_dev, void* hip_stream,
                int static_slot, prsgd_ctx** out_ctx) {
  Layout lo;
  char err[128];
  if (!build_layout(cfg, &lo, err, sizeof(err))) return set_err(nullptr, PRSGD_EINVAL, "%s", err);
  if (x0_host == nullptr || features_dev == nullptr || targets_dev == nullptr || params_dev == nullptr ||
      workspace_dev == nullptr)
    return set_err(nullptr, PRSGD_EINVAL, "null buffer");
  if (((uintptr_t)params_dev % kAlign) != 0 || ((uintptr_t)workspace_dev % kAlign) != 0)
    return set_err(nullptr, PRSGD_EINVAL, "params_dev and workspace_dev must be 256-byte aligned");
  if (((uintptr_t)features_dev % 16) != 0 || ((uintptr_t)targets_dev % 4) != 0)
    return set_err(nullptr, PRSGD_EINVAL, "features_dev must be 16-byte and targets_dev 4-byte aligned");

  prsgd_ctx* ctx;
  if (static_slot < 0) {
    ctx = new (std::nothrow) prsgd_ctx();
    if (ctx == nullptr) return set_err(nullptr, PRSGD_ENOMEM, "out of host memory");
  } else {
    // claim the device's slot; from here on every failure path gives it back (release_ctx)
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (g_static[static_slot].in_use)
      return set_err(nullptr, PRSGD_ESTATE, "prsgd_init_static: the device's static workspace already "
                                            "serves a live context; destroy it first");
    g_static[static_slot].in_use = true;
    ctx = new (g_static[static_slot].ctx_mem) prsgd_ctx();
  }
  ctx->static_slot = static_slot;
  ctx->cfg = effective_config(cfg);
  ctx->lo = lo;
  if (static_slot >= 0) (void)static_scratch(cfg, lo, &ctx->cv);
  else build_carve(cfg, lo, PRSGD_SCRATCH_RUNS, &ctx->cv);
  ctx->bf16 = cfg->model == PRSGD_MLP && cfg->gemm_dtype == PRSGD_BF16;
  ctx->streamed = streamed_uses(*cfg, lo);
  ctx->stream = reinterpret_cast<hipStream_t>(hip_stream);
  ctx->use_fused2 = ctx->cv.part != 0 && ctx->cv.sync != 0 &&
                    fused2_plan(cfg->n_workers, lo.d[0], lo.d[1], lo.d[2], cfg->batch,
                                cfg->momentum != 0.0f, &ctx->f2);
  if (cfg->momentum != 0.0f && !bwd_fused_config(ctx->cfg) && !ctx->use_fused2) ctx->cfg.fused_update = 0;
  ctx->restarts_in_launch = ctx->cv.exchange != 0 && (cfg->model == PRSGD_LSQ || ctx->use_fused2);
  ctx->enlisted = false;
  ctx->next_waiting = nullptr;
  ctx->wait_event = nullptr;
  ctx->wait_seq = 0;
  ctx->ran_pinned = false;
  ctx->n_whole = ctx->n_followed = 0;
  ctx->features = reinterpret_cast<const float*>(features_dev);
  ctx->targets = targets_dev;
  ctx->params = reinterpret_cast<float*>(params_dev);
  ctx->ws = reinterpret_cast<char*>(workspace_dev);
  ctx->t = 0;
  ctx->batch_t[0] = ctx->batch_t[1] = -1;
  ctx->batch_cur = 0;
  ctx->h1_t = -1;
  ctx->h1_batch = 0;
  ctx->recorded = false;
  ctx->first_fusion = true;
  ctx->restart_fusion = true;
  ctx->shadow1_stale = false;
  ctx->lazy_restart = true;
  ctx->at_mean = false;
  ctx->poisoned = false;
  ctx->n_restored = 0;
  memset(ctx->restored, 0, sizeof(ctx->restored));
  ctx->spin_limit = kFused2SpinLimit;
  ctx->lr = cfg->lr;
  ctx->err[0] = 0;
  ctx->profiling = false;
  ctx->pool_used = 0;
  memset(ctx->prof_ms, 0, sizeof(ctx->prof_ms));
  memset(ctx->prof_n, 0, sizeof(ctx->prof_n));
  if (static_slot >= 0) {
    ctx->host_pad = g_static_pad[static_slot];       // m_pad + 1 floats fit: the workspace holds more
  } else {
    try {
      ctx->host_pad_heap.resize((size_t)lo.m_pad + 1);
    } catch (...) {
      release_ctx(ctx);
      return set_err(nullptr, PRSGD_ENOMEM, "out of host memory");
    }
    ctx->host_pad = ctx->host_pad_heap.data();
  }

  // Zero the workspace once: padding columns of every activation buffer must read as zero, and
  // the numbers of the epoch kernel's exchanges and its abort flag start at zero (the static workspace keeps
  // what the previous context left in it).
  hipError_t e = hipMemsetAsync(ctx->ws, 0, ctx->cv.total, ctx->stream);
  if (e == hipSuccess) {
    pad_from_dense(ctx, x0_host, ctx->host_pad);
    e = hipMemcpyAsync(ctx->at<float>(ctx->cv.mean), ctx->host_pad, sizeof(float) * (size_t)lo.m_pad,
                       hipMemcpyHostToDevice, ctx->stream);
  }
  if (e == hipSuccess)
    e = launch_broadcast(ctx->at<float>(ctx->cv.mean), ctx->params, ctx->shadow(), lo.m_pad,
                         cfg->n_workers, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e == hipSuccess && (ctx->use_fused2 || ctx->restarts_in_launch))
    e = enlist_waiting(ctx, ctx->use_fused2 ? ctx->f2.P : 1);
  if (e != hipSuccess) {
    hip_fail(nullptr, e, "prsgd_init");
    release_ctx(ctx);
    return PRSGD_EHIP;
  }
  *out_ctx = ctx;
  return PRSGD_OK;
}

}  // namespace

extern "C" {

int prsgd_init(const prsgd_config* cfg, const float* x0_host, const void* features_dev,
               const void* targets_dev, void* params_dev, void* workspace_dev, void* hip_stream,
               prsgd_ctx** out_ctx) {
  if (out_ctx == nullptr) return set_err(nullptr, PRSGD_EINVAL, "out_ctx is null");
  *out_ctx = nullptr;
  return init_common(cfg, x0_host, features_dev, targets_dev, params_dev, workspace_dev, hip_stream, -1,
                     out_ctx);
}

int prsgd_init_static(const prsgd_config* cfg, const float* x0_host, const void* features_dev,
                      const void* targets_dev, void* params_dev, void* hip_stream, prsgd_ctx** out_ctx) {
  if (out_ctx == nullptr) return set_err(nullptr, PRSGD_EINVAL, "out_ctx is null");
  *out_ctx = nullptr;
  Layout lo;
  char err[128];
  if (!build_layout(cfg, &lo, err, sizeof(err))) return set_err(nullptr, PRSGD_EINVAL, "%s", err);
  Carve cv;
  (void)static_scratch(cfg, lo, &cv);
  if (cv.total > kStaticBytes) {
    char msg[200];
    snprintf(msg, sizeof(msg), "prsgd_init_static: this configuration needs %zu bytes of workspace, the "
             "static workspace holds %zu; use prsgd_init", cv.total, kStaticBytes);
    return set_err(nullptr, PRSGD_EINVAL, "%s", msg);
  }
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(nullptr, e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxStaticDevices)
    return set_err(nullptr, PRSGD_EINVAL, "prsgd_init_static: device index beyond the static slots");
  void* ws = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_static_mutex);
    StaticSlot& slot = g_static[dev];
    if (slot.ws_dev == nullptr) {                  // once per device, with that device current
      void* ptr = nullptr;
      e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
      if (e != hipSuccess || ptr == nullptr)
        return hip_fail(nullptr, e != hipSuccess ? e : hipErrorInvalidSymbol, "hipGetSymbolAddress");
      slot.ws_dev = ptr;
    }
    ws = slot.ws_dev;
  }
  return init_common(cfg, x0_host, features_dev, targets_dev, params_dev, ws, hip_stream, dev, out_ctx);
}

}  // extern "C"

namespace {

// The workers by falling step counts, equal ones in their order: a counting sort over the bytes in which the counts differ.  Two arrays of
// n, the result in the first.
void order_by_steps(const int32_t* steps, int n, int32_t k_min, int32_t k_max, int32_t* order, int32_t* spare) {
  const uint32_t spread = (uint32_t)(k_max - k_min);
  int32_t *from = order, *to = spare;
  for (int i = 0; i < n; ++i) from[i] = i;
  for (int shift = 0; shift < 32 && (spread >> shift) != 0; shift += 8) {
    int place[257] = {};
    auto digit = [&](int32_t i) { return ((uint32_t)(k_max - steps[i]) >> shift) & 255u; };
    for (int i = 0; i < n; ++i) ++place[digit(from[i]) + 1];
    for (int d = 0; d < 256; ++d) place[d + 1] += place[d];
    for (int i = 0; i < n; ++i) to[place[digit(from[i])]++] = from[i];
    std::swap(from, to);
  }
  if (from != order) memcpy(order, from, (size_t)n * sizeof(*order));
}

// k local steps; `last`: nothing of the call comes behind them
int local_steps(prsgd_ctx* ctx, int32_t k, bool last) {
  if (check_poisoned(ctx) != PRSGD_OK) return PRSGD_ESTATE;
  const prsgd_config& c = ctx->cfg;
  if (c.model == PRSGD_LSQ) {
    if (k == 0) return PRSGD_OK;
    LAUNCH(ctx, KK_LSQ, launch_lsq_steps(lsq_args(ctx, k), ctx->stream));
    ctx->at_mean = false;
    ctx->t += k;
    return PRSGD_OK;
  }
  if (ctx->use_fused2) {
    if (k > 0) {
      const int rc = launch_epoch(ctx, k, nullptr);
      if (rc != PRSGD_OK) return rc;
      ctx->at_mean = false;
    }
    ctx->t += k;
    return PRSGD_OK;
  }
  for (int32_t s = 0; s < k; ++s) {
    const int rc = mlp_step(ctx, ctx->t + 1, every_worker(ctx, last && s + 1 == k));
    if (rc != PRSGD_OK) return rc;
    ctx->t += 1;
  }
  return PRSGD_OK;
}

int average(prsgd_ctx* ctx) {
  if (check_poisoned(ctx) != PRSGD_OK) return PRSGD_ESTATE;
  if (ctx->at_mean) return PRSGD_OK;        // all workers already sit at their node average
  ctx->h1_t = -1;                           // an activation computed ahead belongs to the old points
  if (ctx->velocity() != nullptr && ctx->cfg.momentum_restart != PRSGD_MOM_KEEP) {
    // the paper leaves the momentum buffers at a restart open: average them like the points,
    // or start every epoch without momentum
    if (ctx->cfg.momentum_restart == PRSGD_MOM_AVERAGE)
      LAUNCH(ctx, KK_AVERAGE, launch_average(ctx->velocity(), nullptr, ctx->lo.m_pad, ctx->cfg.n_workers,
                                             ctx->streamed.average, ctx->stream));
    else
      LAUNCH(ctx, KK_UPDATE, launch_fill_zero(ctx->velocity(), (size_t)ctx->cfg.n_workers * ctx->lo.m_pad,
                                              ctx->stream));
  }
  if (ctx->lazy_restart && ctx->can_start_from_mean()) {
    // eq. (2) without the broadcast: ybar is written once; the next local iteration reads it as
    // every worker's starting point and writes the replicas  x_i = ybar - gamma G_i  itself
    LAUNCH(ctx, KK_RESTART_MEAN,
           launch_mean(ctx->params, ctx->mean(), ctx->mean_shadow(), ctx->lo.m_pad, ctx->cfg.n_workers,
                       ctx->streamed.mean, ctx->stream));
    ctx->at_mean = true;
    return PRSGD_OK;
  }
  LAUNCH(ctx, KK_AVERAGE,
         launch_average(ctx->params, ctx->shadow(), ctx->lo.m_pad, ctx->cfg.n_workers, ctx->streamed.average,
                        ctx->stream));
  ctx->shadow1_stale = false;               // the averaging kernel rewrites every shadow
  return PRSGD_OK;
}

}  // namespace

extern "C" {

int prsgd_local_steps(prsgd_ctx* ctx, int32_t k) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (k < 0) return set_err(ctx, PRSGD_EINVAL, "k must be >= 0");
  begin_call(ctx, k);
  const int rc = local_steps(ctx, k, true);
  return rc != PRSGD_OK ? rc : end_call(ctx);
}

int prsgd_local_steps_hetero(prsgd_ctx* ctx, const int32_t* steps_host) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (steps_host == nullptr) return set_err(ctx, PRSGD_EINVAL, "steps_host is null");
  if (ctx->cfg.momentum != 0.0f)
    return set_err(ctx, PRSGD_EINVAL, "heterogeneous epochs are not defined with momentum");
  if (check_poisoned(ctx) != PRSGD_OK) return PRSGD_ESTATE;
  const prsgd_config& c = ctx->cfg;
  int32_t k_max = 0, k_min = steps_host[0];
  for (int i = 0; i < c.n_workers; ++i) {
    if (steps_host[i] < 0) return set_err(ctx, PRSGD_EINVAL, "worker step counts must be >= 0");
    if (steps_host[i] > k_max) k_max = steps_host[i];
    if (steps_host[i] < k_min) k_min = steps_host[i];
  }
  // a graph takes whole epochs of every worker only: its replays would keep the step counts of the recording
  if (is_capturing(ctx->stream)) return hip_fail(ctx, hipErrorStreamCaptureUnsupported, "worker step counts");
  // a worker that takes no step must still hold the restart point: broadcast it first.  Layer by layer the
  // steps that every worker takes run unmasked, and the first of them starts from the average itself
  // (16 workers of 3072-1024-1024-10, one to four steps: broadcast 67 us, first step 72 + 22 us for layer 1
  // with private weights; 1594 -> 1338 us for two epochs).
  const bool layers = ctx->layered();
  begin_call(ctx, k_min > 1 ? k_min : 1);         // masked steps leave their rows beside those of the last step of all workers
  if (!layers || k_min == 0) {
    const int mrc = materialize(ctx);
    if (mrc != PRSGD_OK) return mrc;
  }
  // the step counts, or (layer by layer) the workers by falling step counts
  int* steps_dev = ctx->at<int>(ctx->cv.steps);
  std::unique_ptr<int32_t[]> order;
  if (layers) {
    order.reset(new (std::nothrow) int32_t[2 * (size_t)c.n_workers]);
    if (order == nullptr) return set_err(ctx, PRSGD_ENOMEM, "out of host memory");
    order_by_steps(steps_host, c.n_workers, k_min, k_max, order.get(), order.get() + c.n_workers);
  }
  const hipError_t e = launch_store_ints(steps_dev, layers ? order.get() : steps_host, c.n_workers, layers ? c.n_workers - 1 : k_max,
                                         ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "worker step counts");
  if (c.model == PRSGD_LSQ) {
    LsqArgs a = lsq_args(ctx, k_max);
    a.worker_steps = steps_dev;
    LAUNCH(ctx, KK_LSQ, launch_lsq_steps(a, ctx->stream));
    ctx->t += k_max;
    return PRSGD_OK;
  }
  if (ctx->use_fused2) {
    if (k_max > 0) {
      const int rc = launch_epoch(ctx, k_max, steps_dev);
      if (rc != PRSGD_OK) return rc;
    }
    ctx->t += k_max;
    return PRSGD_OK;
  }
  int taking = c.n_workers;
  auto workers_at = [&](int32_t s) {              // that take step s (from 0); s never falls
    while (taking > 0 && steps_host[order[taking - 1]] <= s) --taking;
    return taking;
  };
  int rc = PRSGD_OK, idx_set = -1;
  if (k_min == 0 && k_max > 0) ctx->batch_t[0] = ctx->batch_t[1] = -1;   // drawn for workers that take no step as well
  for (int32_t s = 0; s < k_max && rc == PRSGD_OK; ++s) {
    Active a = every_worker(ctx, s + 1 == k_max);
    if (s >= k_min) {
      a.order = steps_dev;
      a.now = workers_at(s);
    }
    if (s + 1 >= k_min && k_min != k_max) {
      a.next_order = steps_dev;
      a.next = workers_at(s + 1);
      // masked draws write the row numbers beside those that the workers that are done drew last
      if (idx_set < 0) idx_set = ctx->batch_t[0] == ctx->t + 1 ? 0 : ctx->batch_t[1] == ctx->t + 1 ? 1 : ctx->batch_cur;
      a.idx_set = idx_set;
    }
    rc = mlp_step(ctx, ctx->t + 1, a);
    if (rc == PRSGD_OK) ctx->t += 1;
  }
  if (k_min != k_max) {                           // a masked draw is not reused
    ctx->batch_t[0] = ctx->batch_t[1] = -1;
    if (idx_set >= 0) ctx->batch_cur = idx_set;
  }
  return rc;
}

int prsgd_average(prsgd_ctx* ctx) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  begin_call(ctx, 0);
  const int rc = average(ctx);
  return rc != PRSGD_OK ? rc : end_call(ctx);
}

int prsgd_set_lazy_restart(prsgd_ctx* ctx, int32_t on) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (!on) {
    begin_call(ctx, 0);
    const int rc = materialize(ctx);
    if (rc != PRSGD_OK) return rc;
  }
  ctx->lazy_restart = on != 0;
  return PRSGD_OK;
}

int prsgd_run(prsgd_ctx* ctx, int64_t iterations, int32_t interval) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (iterations < 0 || interval < 1) return set_err(ctx, PRSGD_EINVAL, "iterations >= 0, interval >= 1");
  int64_t left = iterations;
  begin_call(ctx, iterations);
  // Restarts that need no launch of their own: the whole run, up to a restart at its end, is one launch (least squares, 4
  // workers of 64 floats, 256 iterations with a restart after every eighth: 530 us with two launches per epoch, 200 us).
  // Per-kernel timing keeps them apart, as launches of their own.
  while (ctx->restarts_in_launch && ctx->lazy_restart && !ctx->profiling &&
         (ctx->velocity() == nullptr || ctx->cfg.momentum_restart == PRSGD_MOM_KEEP)) {
    constexpr int64_t kLongest = 1 << 20;
    const int k = (int)(left < kLongest ? left : kLongest);
    if (k <= interval - (ctx->t % interval)) break;
    if (check_poisoned(ctx) != PRSGD_OK) return PRSGD_ESTATE;
    {
      WaitingLaunch waiting(ctx);
      if (!waiting.may_wait_as_whole()) break;
      if (ctx->use_fused2) {
        Fused2Args a = fused2_args(ctx, k, nullptr);
        a.interval = interval;
        LAUNCH(ctx, KK_FUSED2, launch_fused2(ctx->f2, a, waiting.pinned(), ctx->stream));
      } else {
        LsqArgs a = lsq_args(ctx, k);
        a.interval = interval;
        a.sync = ctx->at<unsigned int>(ctx->cv.sync);
        a.abort_flag = ctx->abort_flag();
        a.exchange = ctx->at<unsigned long long>(ctx->cv.exchange);
        a.spin_limit = ctx->spin_limit;
        LAUNCH(ctx, KK_LSQ, launch_lsq_steps(a, ctx->stream));
      }
      ++ctx->n_whole;
    }
    ctx->at_mean = false;
    ctx->t += k;
    left -= k;
    if (ctx->t % interval == 0) {
      const int rc = average(ctx);
      if (rc != PRSGD_OK) return rc;
    }
  }
  // Plain SGD on bf16 operands with the deferred broadcast: the iteration that completes an epoch
  // and the restart after it are one pass that writes only ybar (with I = 1: every iteration)
  const bool can_fuse = ctx->cfg.model == PRSGD_MLP && ctx->bf16 && ctx->cfg.fused_update &&
                        ctx->cfg.momentum == 0.0f && ctx->lazy_restart && !ctx->use_fused2 &&
                        ctx->restart_fusion && bwd_fused_supported(ctx->cfg.batch);
  while (left > 0) {
    if (can_fuse && interval - (ctx->t % interval) <= left) {
      const int64_t k_epoch = interval - (ctx->t % interval);
      if (k_epoch > 1) {
        const int rc = local_steps(ctx, (int32_t)(k_epoch - 1), false);
        if (rc != PRSGD_OK) return rc;
      }
      if (check_poisoned(ctx) != PRSGD_OK) return PRSGD_ESTATE;
      const int rc = mlp_step(ctx, ctx->t + 1, every_worker(ctx, k_epoch == left), true);
      if (rc != PRSGD_OK) return rc;
      ctx->t += 1;
      left -= k_epoch;
      continue;
    }
    int64_t k = interval - (ctx->t % interval);      // steps until the next multiple of I
    if (k > left) k = left;
    int rc = local_steps(ctx, (int32_t)k, k == left);
    if (rc != PRSGD_OK) return rc;
    left -= k;
    if (ctx->t % interval == 0) {
      rc = average(ctx);
      if (rc != PRSGD_OK) return rc;
    }
  }
  return end_call(ctx);
}

int prsgd_read_params(prsgd_ctx* ctx, int32_t worker, float* out_host, size_t m) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (out_host == nullptr) return set_err(ctx, PRSGD_EINVAL, "out_host is null");
  if (m != (size_t)ctx->lo.m) return set_err(ctx, PRSGD_EINVAL, "m does not match the parameter count");
  if (worker < -1 || worker >= ctx->cfg.n_workers) return set_err(ctx, PRSGD_EINVAL, "worker out of range");
  // the average of a least-squares context comes with the abort flag that stands behind it: one copy
  const bool with_flag = ctx->lo.n_layers == 0 && ctx->abort_flag() != nullptr && !ctx->poisoned &&
                         (ctx->at_mean || worker < 0);
  if (!with_flag) {
    const int arc = check_gave_up(ctx);
    if (arc != PRSGD_OK) return arc;
  }
  const float* src;
  if (ctx->at_mean) {
    src = ctx->mean();                      // every worker's point, and their average
  } else if (worker < 0) {
    LAUNCH(ctx, KK_MEAN, launch_mean(ctx->params, ctx->mean(), nullptr, ctx->lo.m_pad,
                                     ctx->cfg.n_workers, true, ctx->stream));
    src = ctx->mean();
  } else {
    src = ctx->params + (size_t)worker * ctx->lo.m_pad;
  }
  hipError_t e = hipMemcpyAsync(ctx->host_pad, src, sizeof(float) * (size_t)(ctx->lo.m_pad + (with_flag ? 1 : 0)),
                                hipMemcpyDeviceToHost, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "prsgd_read_params");
  if (with_flag) {
    unsigned int flag = 0;
    memcpy(&flag, ctx->host_pad + ctx->lo.m_pad, sizeof(flag));
    if (flag != 0) return workgroups_gave_up(ctx);
  }
  dense_from_pad(ctx, ctx->host_pad, out_host);
  return PRSGD_OK;
}

int prsgd_write_params(prsgd_ctx* ctx, int32_t worker, const float* in_host, size_t m) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (in_host == nullptr) return set_err(ctx, PRSGD_EINVAL, "in_host is null");
  if (m != (size_t)ctx->lo.m) return set_err(ctx, PRSGD_EINVAL, "m does not match the parameter count");
  if (worker < -1 || worker >= ctx->cfg.n_workers) return set_err(ctx, PRSGD_EINVAL, "worker out of range");
  if (worker >= 0) {                        // the other replicas must hold their restart point
    const int mrc = materialize(ctx);
    if (mrc != PRSGD_OK) return mrc;
  }
  if (ctx->poisoned) {                      // an aborted epoch launch: usable again once every
    if (worker < 0) {                       // replica has been rewritten
      ctx->poisoned = false;
    } else if (!((ctx->restored[worker >> 3] >> (worker & 7)) & 1)) {
      ctx->restored[worker >> 3] |= (unsigned char)(1u << (worker & 7));
      if (++ctx->n_restored == (size_t)ctx->cfg.n_workers) ctx->poisoned = false;
    }
  }
  ctx->at_mean = false;
  ctx->h1_t = -1;
  pad_from_dense(ctx, in_host, ctx->host_pad);
  const size_t bytes = sizeof(float) * (size_t)ctx->lo.m_pad;
  hipError_t e;
  if (worker < 0) {
    e = hipMemcpyAsync(ctx->at<float>(ctx->cv.mean), ctx->host_pad, bytes, hipMemcpyHostToDevice,
                       ctx->stream);
    if (e == hipSuccess)
      e = launch_broadcast(ctx->at<float>(ctx->cv.mean), ctx->params, ctx->shadow(), ctx->lo.m_pad,
                           ctx->cfg.n_workers, ctx->stream);
    ctx->shadow1_stale = false;
  } else {
    float* dst = ctx->params + (size_t)worker * ctx->lo.m_pad;
    e = hipMemcpyAsync(dst, ctx->host_pad, bytes, hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess && ctx->bf16)
      e = launch_refresh_shadow(dst, ctx->shadow() + (size_t)worker * ctx->lo.m_pad, ctx->lo.m_pad,
                                ctx->stream);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "prsgd_write_params");
  return PRSGD_OK;
}

int prsgd_read_velocity(prsgd_ctx* ctx, int32_t worker, float* out_host, size_t m) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (out_host == nullptr) return set_err(ctx, PRSGD_EINVAL, "out_host is null");
  if (m != (size_t)ctx->lo.m) return set_err(ctx, PRSGD_EINVAL, "m does not match the parameter count");
  if (worker < 0 || worker >= ctx->cfg.n_workers) return set_err(ctx, PRSGD_EINVAL, "worker out of range");
  if (ctx->velocity() == nullptr) return set_err(ctx, PRSGD_ESTATE, "the context has no momentum buffers");
  const int arc = check_gave_up(ctx);
  if (arc != PRSGD_OK) return arc;
  hipError_t e = hipMemcpyAsync(ctx->host_pad, ctx->velocity() + (size_t)worker * ctx->lo.m_pad,
                                sizeof(float) * (size_t)ctx->lo.m_pad, hipMemcpyDeviceToHost, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "prsgd_read_velocity");
  dense_from_pad(ctx, ctx->host_pad, out_host);
  return PRSGD_OK;
}

int prsgd_write_velocity(prsgd_ctx* ctx, int32_t worker, const float* in_host, size_t m) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (in_host == nullptr) return set_err(ctx, PRSGD_EINVAL, "in_host is null");
  if (m != (size_t)ctx->lo.m) return set_err(ctx, PRSGD_EINVAL, "m does not match the parameter count");
  if (worker < 0 || worker >= ctx->cfg.n_workers) return set_err(ctx, PRSGD_EINVAL, "worker out of range");
  if (ctx->velocity() == nullptr) return set_err(ctx, PRSGD_ESTATE, "the context has no momentum buffers");
  pad_from_dense(ctx, in_host, ctx->host_pad);
  hipError_t e = hipMemcpyAsync(ctx->velocity() + (size_t)worker * ctx->lo.m_pad, ctx->host_pad,
                                sizeof(float) * (size_t)ctx->lo.m_pad, hipMemcpyHostToDevice, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "prsgd_write_velocity");
  return PRSGD_OK;
}

int prsgd_read_loss(prsgd_ctx* ctx, float* out_host) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (out_host == nullptr) return set_err(ctx, PRSGD_EINVAL, "out_host is null");
  const int arc = check_gave_up(ctx);
  if (arc != PRSGD_OK) return arc;
  hipError_t e = hipSuccess;
  if (ctx->cfg.model == PRSGD_MLP)
    e = launch_loss_mean(ctx->at<float>(ctx->cv.row_loss), ctx->at<float>(ctx->cv.losses),
                         ctx->cfg.n_workers, ctx->cfg.batch, ctx->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(out_host, ctx->at<float>(ctx->cv.losses), sizeof(float) * ctx->cfg.n_workers,
                                hipMemcpyDeviceToHost, ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "prsgd_read_loss");
  return PRSGD_OK;
}

int prsgd_read_indices(prsgd_ctx* ctx, int32_t* out_host) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (out_host == nullptr) return set_err(ctx, PRSGD_EINVAL, "out_host is null");
  const int arc = check_gave_up(ctx);
  if (arc != PRSGD_OK) return arc;
  const size_t bytes = sizeof(int32_t) * (size_t)ctx->cfg.n_workers * ctx->cfg.batch;
  // the layer-wise MLP path alternates between two buffer sets; the others only use the first
  hipError_t e = hipMemcpyAsync(out_host, ctx->idx(ctx->batch_cur), bytes, hipMemcpyDeviceToHost,
                                ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "prsgd_read_indices");
  return PRSGD_OK;
}

int prsgd_sample_indices(uint64_t seed, int32_t n_workers, int32_t batch, int64_t rows_per_worker,
                         int64_t t_first, int32_t n_steps, int32_t* out_dev, void* hip_stream) {
  if (out_dev == nullptr || n_workers < 1 || batch < 1 || n_steps < 0 || t_first < 0 ||
      rows_per_worker < 1 || rows_per_worker > (1LL << 31) ||
      (rows_per_worker & (rows_per_worker - 1)) != 0)
    return set_err(nullptr, PRSGD_EINVAL, "prsgd_sample_indices: bad argument");
  hipError_t e = launch_sample_indices(seed, n_workers, batch, (long)rows_per_worker, t_first, n_steps,
                                       out_dev, reinterpret_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return hip_fail(nullptr, e, "prsgd_sample_indices");
  return PRSGD_OK;
}

int prsgd_sgd_update(float* x_dev, const float* g_dev, uint16_t* shadow_dev, size_t count, float lr,
                     void* hip_stream) {
  if (x_dev == nullptr || g_dev == nullptr) return set_err(nullptr, PRSGD_EINVAL, "null buffer");
  if (((uintptr_t)x_dev % 16) != 0 || ((uintptr_t)g_dev % 16) != 0 || ((uintptr_t)shadow_dev % 8) != 0)
    return set_err(nullptr, PRSGD_EINVAL, "prsgd_sgd_update: misaligned buffer");
  hipError_t e = launch_update(x_dev, g_dev, shadow_dev, count, lr, reinterpret_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return hip_fail(nullptr, e, "prsgd_sgd_update");
  return PRSGD_OK;
}

int prsgd_copy_bytes(void* dst_dev, const void* src_dev, size_t bytes, void* hip_stream) {
  if (dst_dev == nullptr || src_dev == nullptr || (bytes % 16) != 0 || ((uintptr_t)dst_dev % 16) != 0 ||
      ((uintptr_t)src_dev % 16) != 0)
    return set_err(nullptr, PRSGD_EINVAL, "prsgd_copy_bytes: bad argument");
  hipError_t e = launch_copy(dst_dev, src_dev, bytes, reinterpret_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return hip_fail(nullptr, e, "prsgd_copy_bytes");
  return PRSGD_OK;
}

int prsgd_product_tile(int32_t rows, int32_t cols, int32_t n_workers, int32_t gemm_dtype, int32_t* out) {
  if (rows < 1 || cols < 1 || n_workers < 1 || (gemm_dtype != PRSGD_F32 && gemm_dtype != PRSGD_BF16) ||
      out == nullptr)
    return set_err(nullptr, PRSGD_EINVAL, "prsgd_product_tile: bad argument");
  int tile_rows = 0, tile_cols = 0;
  size_t lds = 0;
  gemm_rows_shape(rows, cols, n_workers, gemm_dtype == PRSGD_BF16, &tile_rows, &tile_cols, &lds);
  out[0] = tile_rows;
  out[1] = tile_cols;
  out[2] = (int32_t)lds;
  return PRSGD_OK;
}

int prsgd_streamed_uses(const prsgd_config* cfg) {
  Layout lo;
  char err[128];
  if (!build_layout(cfg, &lo, err, sizeof(err))) return set_err(nullptr, PRSGD_EINVAL, "%s", err);
  const Streamed u = streamed_uses(*cfg, lo);
  return (u.steps ? PRSGD_STREAM_STEPS : 0) | (u.step_mean ? PRSGD_STREAM_STEP_MEAN : 0) |
         (u.mean ? PRSGD_STREAM_MEAN : 0) | (u.average ? PRSGD_STREAM_AVERAGE : 0) | (u.rows ? PRSGD_STREAM_ROWS : 0);
}

int prsgd_static_scratch(const prsgd_config* cfg) {
  Layout lo;
  char err[128];
  if (!build_layout(cfg, &lo, err, sizeof(err))) return set_err(nullptr, PRSGD_EINVAL, "%s", err);
  Carve cv;
  const int scratch = static_scratch(cfg, lo, &cv);
  return cv.total <= kStaticBytes ? scratch : set_err(nullptr, PRSGD_EINVAL, "beyond the static workspace");
}

int prsgd_waiting_regime(const int32_t* n_workers, const int32_t* team, int32_t n_streams, int32_t compute_units) {
  if (n_workers == nullptr || team == nullptr || n_streams < 1 || compute_units < 8)
    return set_err(nullptr, PRSGD_EINVAL, "prsgd_waiting_regime: bad argument");
  long demand = 0;
  for (int k = 0; k < n_streams; ++k) demand += xcd_workgroups(n_workers[k], team[k], false);
  return waiting_regime(n_streams, demand, compute_units / 8);
}

int prsgd_waiting_launches(const prsgd_ctx* ctx, int64_t* out) {
  if (ctx == nullptr || out == nullptr) return PRSGD_EINVAL;
  out[0] = ctx->n_whole;
  out[1] = ctx->n_followed;
  return PRSGD_OK;
}

int prsgd_status(prsgd_ctx* ctx) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  const int arc = check_gave_up(ctx);
  if (arc != PRSGD_OK) return arc;
  const hipError_t e = hipStreamSynchronize(ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "prsgd_status");
  return PRSGD_OK;
}

int prsgd_set_restart_fusion(prsgd_ctx* ctx, int32_t on) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  ctx->restart_fusion = on != 0;
  return PRSGD_OK;
}

int prsgd_set_first_layer_fusion(prsgd_ctx* ctx, int32_t on) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  ctx->first_fusion = on != 0;
  ctx->h1_t = -1;
  return PRSGD_OK;
}

int prsgd_set_epoch_wait_limit(prsgd_ctx* ctx, uint32_t polls) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  ctx->spin_limit = polls;
  return PRSGD_OK;
}

int prsgd_time_varying_schedule(int32_t n_epochs, int32_t n_workers, int32_t* lengths_host,
                                float* rates_host) {
  if (n_epochs < 0 || n_workers < 1 || (n_epochs > 0 && (lengths_host == nullptr || rates_host == nullptr)))
    return set_err(nullptr, PRSGD_EINVAL, "prsgd_time_varying_schedule: bad argument");
  // K^s = ceil(s^(1/3) / N) is the smallest integer k with (k N)^3 >= s: integer arithmetic, so
  // that perfect cubes land exactly.  k N only ever grows with s.
  unsigned __int128 kn = (unsigned __int128)n_workers;      // current k N
  int32_t k = 1;
  for (int32_t s = 1; s <= n_epochs; ++s) {
    while (kn * kn * kn < (unsigned __int128)s) { kn += (unsigned __int128)n_workers; ++k; }
    lengths_host[s - 1] = k;
    const double c = cbrt((double)s);
    rates_host[s - 1] = (float)((double)n_workers / (c * c));
  }
  return PRSGD_OK;
}

int prsgd_set_lr(prsgd_ctx* ctx, float lr) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (!(lr == lr)) return set_err(ctx, PRSGD_EINVAL, "lr is NaN");
  ctx->lr = lr;
  return PRSGD_OK;
}
int prsgd_set_iteration(prsgd_ctx* ctx, int64_t t) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (t < 0) return set_err(ctx, PRSGD_EINVAL, "t must be >= 0");
  ctx->t = t;
  return PRSGD_OK;
}
int64_t prsgd_iteration(const prsgd_ctx* ctx) { return ctx == nullptr ? -1 : ctx->t; }

int prsgd_profile_enable(prsgd_ctx* ctx, int32_t on) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (on && ctx->pool.empty()) {
    constexpr size_t kPairs = 2048;
    try {
      ctx->pool.reserve(kPairs);
    } catch (...) {
      return set_err(ctx, PRSGD_ENOMEM, "out of host memory");
    }
    for (size_t i = 0; i < kPairs; ++i) {
      EventPair ep;
      hipError_t e = hipEventCreate(&ep.a);
      if (e == hipSuccess) {
        e = hipEventCreate(&ep.b);
        if (e != hipSuccess) (void)hipEventDestroy(ep.a);
      }
      if (e != hipSuccess) return hip_fail(ctx, e, "hipEventCreate");
      ep.kind = 0;
      ctx->pool.push_back(ep);
    }
  }
  if (!on) {
    const int rc = profile_flush(ctx);
    if (rc != PRSGD_OK) return rc;
  }
  ctx->profiling = on != 0;
  return PRSGD_OK;
}

int prsgd_profile_read(prsgd_ctx* ctx, prsgd_kernel_stat* out, int32_t max) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  if (out == nullptr || max < 0) return set_err(ctx, PRSGD_EINVAL, "bad output buffer");
  const int rc = profile_flush(ctx);
  if (rc != PRSGD_OK) return rc;
  int n = 0;
  for (int k = 0; k < KK_COUNT; ++k) {
    if (ctx->prof_n[k] == 0) continue;
    if (n < max) {
      memset(&out[n], 0, sizeof(out[n]));
      snprintf(out[n].name, sizeof(out[n].name), "%s", kernel_kind_name(k));
      out[n].launches = ctx->prof_n[k];
      out[n].total_ms = ctx->prof_ms[k];
    }
    ++n;
  }
  memset(ctx->prof_ms, 0, sizeof(ctx->prof_ms));
  memset(ctx->prof_n, 0, sizeof(ctx->prof_n));
  return n;
}

int prsgd_destroy(prsgd_ctx* ctx) {
  if (ctx == nullptr) return PRSGD_EINVAL;
  hipError_t e = hipStreamSynchronize(ctx->stream);
  for (auto& ep : ctx->pool) {
    (void)hipEventDestroy(ep.a);
    (void)hipEventDestroy(ep.b);
  }
  release_ctx(ctx);
  return e == hipSuccess ? PRSGD_OK : PRSGD_EHIP;
}

const char* prsgd_last_error(const prsgd_ctx* ctx) { return ctx != nullptr ? ctx->err : g_init_error; }

}  // extern "C"
