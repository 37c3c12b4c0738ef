// Least-squares workers: k consecutive local iterations of
//   x_i <- x_i - gamma * (1/B) A_b^T (A_b x_i - y_b)             (Algorithm 1, eq. 3)
// in ONE launch.  Workers never exchange anything inside an epoch (paragraph below
// Algorithm 1), so one workgroup per worker keeps x_i on chip for the whole call and only the
// sampled rows travel from HBM.
#include <atomic>
#include <type_traits>

#include "prsgd_internal.h"

namespace prsgd {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kMaxStagedFloats = 8192;   // minibatch floats the staged kernel keeps in LDS
constexpr int kMaxStagedBatch = 512;     // its targets travel in two registers per thread and stage

static int ilog2_rows(long n) {
  int l = 0;
  while ((1L << l) < n) ++l;
  return l;
}

__global__ __launch_bounds__(kThreads) void lsq_steps_kernel(LsqArgs p) {
  const float *features = p.features, *targets = p.targets, *src = p.src;
  float *params = p.params, *velocity = p.velocity, *losses = p.losses;
  int32_t* idx = p.idx;
  const int d = p.d, log2n = p.log2n, batch = p.batch, k = p.k;
  const int* worker_steps = p.worker_steps;
  const long src_stride = p.src_stride, m_pad = p.m_pad, rows = p.rows;
  const float mu = p.mu, lr = p.lr;
  const uint64_t seed = p.seed, t0 = p.t0;
  extern __shared__ float lds[];
  float* x = lds;                                   // [d]
  float* vel = lds + d;                             // [d] momentum buffer (unused when mu == 0)
  float* res = vel + d;                             // [batch] residuals a_j . x - y_j
  int32_t* row = reinterpret_cast<int32_t*>(res + batch);   // [batch]

  const int i = blockIdx.x;
  const int my_k = worker_steps != nullptr ? min(worker_steps[i], k) : k;
  if (my_k <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* feat_i = features + (size_t)i * rows * d;
  const float* targ_i = targets + (size_t)i * rows;
  float* x_glob = params + (size_t)i * m_pad;
  const float inv_b = 1.0f / (float)batch;

  const float* x_start = src + (size_t)i * src_stride;     // the replica, or the shared node average
  float* v_glob = velocity != nullptr ? velocity + (size_t)i * m_pad : nullptr;
  for (int c = tid; c < d; c += kThreads) {
    x[c] = x_start[c];
    vel[c] = v_glob != nullptr ? v_glob[c] : 0.0f;
  }
  float loss = 0.0f;

  for (int s = 1; s <= my_k; ++s) {
    const uint64_t t = t0 + (uint64_t)s;
    for (int j = tid; j < batch; j += kThreads) row[j] = sample_row(seed, (uint32_t)i, t, (uint32_t)j, log2n);
    __syncthreads();
    // residuals: one wavefront per sampled row, lanes stride over the features
    for (int j = wave; j < batch; j += kThreads / kWave) {
      const float* a = feat_i + (size_t)row[j] * d;
      float dot = 0.0f;
      for (int c = lane; c < d; c += kWave) dot = fmaf(a[c], x[c], dot);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) dot += __shfl_xor(dot, o);
      if (lane == 0) res[j] = dot - targ_i[row[j]];
    }
    __syncthreads();
    // gradient column c and update; rows summed in slot order
    for (int c = tid; c < d; c += kThreads) {
      float gc = 0.0f;
      for (int j = 0; j < batch; ++j) gc = fmaf(feat_i[(size_t)row[j] * d + c], res[j], gc);
      if (v_glob != nullptr) {                      // v <- mu v + G,  x <- x - gamma v
        const float vc = fmaf(mu, vel[c], gc * inv_b);
        vel[c] = vc;
        x[c] = fmaf(-lr, vc, x[c]);
      } else {
        x[c] = fmaf(-lr, gc * inv_b, x[c]);
      }
    }
    if (s == my_k && tid == 0) {
      float sq = 0.0f;
      for (int j = 0; j < batch; ++j) sq = fmaf(res[j], res[j], sq);
      loss = 0.5f * sq * inv_b;
    }
    if (s == my_k)
      for (int j = tid; j < batch; j += kThreads) idx[(size_t)i * batch + j] = row[j];
    __syncthreads();
  }
  for (int c = tid; c < d; c += kThreads) {
    x_glob[c] = x[c];
    if (v_glob != nullptr) v_glob[c] = vel[c];
  }
  if (tid == 0) losses[i] = loss;
}

// Sum over the 64 lanes of a wavefront, returned in every lane: butterflies inside each row of
// 16 lanes on the data-parallel-primitive path (no LDS round trips), then the four row sums.
__device__ inline float wave_sum(float v) {
  auto dpp = [](float f, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(f), decltype(ctrl)::value, 0xF, 0xF, true));
  };
  v += dpp(v, std::integral_constant<int, 0xB1>());    // quad_perm [1,0,3,2]
  v += dpp(v, std::integral_constant<int, 0x4E>());    // quad_perm [2,3,0,1]
  v += dpp(v, std::integral_constant<int, 0x141>());   // row_half_mirror
  v += dpp(v, std::integral_constant<int, 0x140>());   // row_mirror
  const int iv = __float_as_int(v);
  return (__int_as_float(__builtin_amdgcn_readlane(iv, 0)) + __int_as_float(__builtin_amdgcn_readlane(iv, 16))) +
         (__int_as_float(__builtin_amdgcn_readlane(iv, 32)) + __int_as_float(__builtin_amdgcn_readlane(iv, 48)));
}

// Staged variant for larger minibatches of at most kMaxStagedFloats floats (d a multiple of 4): the
// sampled rows pass through LDS (two buffers, so an iteration costs two workgroup barriers),
// and because the index stream is a pure function of (seed, worker, t, slot) the rows of
// iteration s + D are requested D iterations early and wait in registers: no iteration stalls
// on HBM latency.  The rows themselves are drawn D iterations at a time, two blocks ahead.
// PFV = 16-byte vectors per thread and minibatch, D = prefetch depth in iterations.
template <int PFV, int D>
__global__ __launch_bounds__(kThreads) void lsq_steps_staged_kernel(LsqArgs p) {
  const float *features = p.features, *targets = p.targets, *src = p.src;
  float *params = p.params, *velocity = p.velocity, *losses = p.losses;
  int32_t* idx = p.idx;
  const int d = p.d, log2n = p.log2n, batch = p.batch, k = p.k;
  const int* worker_steps = p.worker_steps;
  const long src_stride = p.src_stride, m_pad = p.m_pad, rows = p.rows;
  const float mu = p.mu, lr = p.lr;
  const uint64_t seed = p.seed, t0 = p.t0;
  constexpr int YV = (kMaxStagedBatch + kThreads - 1) / kThreads;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int bd = batch * d;
  float* A = lds;                                   // [2][batch][d] rows of the current / next iteration
  float* x = A + 2 * (size_t)bd;                    // [d]
  float* vel = x + d;                               // [d]
  float* res = vel + d;                             // [batch]
  float* ys = res + batch;                          // [2][batch] targets
  int32_t* row = reinterpret_cast<int32_t*>(ys + 2 * batch);   // [3][D][batch]: block b of D iterations at slot b % 3

  const int i = blockIdx.x;
  const int my_k = worker_steps != nullptr ? min(worker_steps[i], k) : k;
  if (my_k <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* feat_i = features + (size_t)i * rows * d;
  const float* targ_i = targets + (size_t)i * rows;
  float* x_glob = params + (size_t)i * m_pad;
  const float inv_b = 1.0f / (float)batch;
  const int d4 = d >> 2, nvec = batch * d4;

  const float* x_start = src + (size_t)i * src_stride;
  float* v_glob = velocity != nullptr ? velocity + (size_t)i * m_pad : nullptr;
  for (int c = tid; c < d; c += kThreads) {
    x[c] = x_start[c];
    vel[c] = v_glob != nullptr ? v_glob[c] : 0.0f;
  }
  // rows of block b: iterations b*D + 1 ... b*D + D of this call
  auto draw_block = [&](int b) {
    int32_t* r = row + (size_t)(b % 3) * D * batch;
    for (int e = tid; e < D * batch; e += kThreads) {
      const int u = e / batch, j = e - u * batch;
      r[e] = sample_row(seed, (uint32_t)i, t0 + (uint64_t)(b * D + 1 + u), (uint32_t)j, log2n);
    }
  };
  f32x4_t pre[D][PFV];
  float ypre[D][YV];
  auto issue = [&](int b, int u) {                  // request the minibatch of iteration b*D + 1 + u
    const int32_t* r = row + ((size_t)(b % 3) * D + u) * batch;
#pragma unroll
    for (int v = 0; v < PFV; ++v) {
      const int e = tid + kThreads * v;
      const int ec = e < nvec ? e : 0;
      const int j = ec / d4, c4 = ec - j * d4;
      pre[u][v] = *reinterpret_cast<const f32x4_t*>(feat_i + (size_t)r[j] * d + 4 * c4);
    }
#pragma unroll
    for (int v = 0; v < YV; ++v) {
      const int j = tid + kThreads * v;
      ypre[u][v] = targ_i[r[j < batch ? j : 0]];
    }
  };
  auto land = [&](int u, float* Ab, float* yb) {    // registers -> LDS
#pragma unroll
    for (int v = 0; v < PFV; ++v) {
      const int e = tid + kThreads * v;
      if (e < nvec) *reinterpret_cast<f32x4_t*>(Ab + 4 * (size_t)e) = pre[u][v];
    }
#pragma unroll
    for (int v = 0; v < YV; ++v) {
      const int j = tid + kThreads * v;
      if (j < batch) yb[j] = ypre[u][v];
    }
  };

  draw_block(0);
  draw_block(1);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < D; ++u)
    if (1 + u <= my_k) issue(0, u);
  constexpr int RW = 4;                             // rows in flight per wavefront

  for (int b = 0; b * D < my_k; ++b) {
    draw_block(b + 2);                              // read from the next block on: barriers in between
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int s = b * D + 1 + u;
      if (s <= my_k) {                              // uniform over the workgroup
        float* Ab = A + (size_t)(s & 1) * bd;
        float* yb = ys + (size_t)(s & 1) * batch;
        land(u, Ab, yb);
        if (s + D <= my_k) issue(b + 1, u);         // nothing is requested past the last iteration
        __syncthreads();
        // residuals: RW rows per wavefront at a time, lanes stride over the features
        for (int j0 = wave * RW; j0 < batch; j0 += (kThreads / kWave) * RW) {
          float dot[RW];
#pragma unroll
          for (int q = 0; q < RW; ++q) dot[q] = 0.0f;
          for (int c = lane; c < d; c += kWave) {
            const float xc = x[c];
#pragma unroll
            for (int q = 0; q < RW; ++q)
              dot[q] = fmaf(Ab[(size_t)min(j0 + q, batch - 1) * d + c], xc, dot[q]);
          }
#pragma unroll
          for (int q = 0; q < RW; ++q) {
            const float t = wave_sum(dot[q]);
            if (lane == q && j0 + q < batch) res[j0 + q] = t - yb[j0 + q];
          }
        }
        __syncthreads();
        // gradient column c and update; rows summed in slot order
        for (int c = tid; c < d; c += kThreads) {
          float gc = 0.0f;
#pragma unroll 8
          for (int j = 0; j < batch; ++j) gc = fmaf(Ab[(size_t)j * d + c], res[j], gc);
          if (v_glob != nullptr) {
            const float vc = fmaf(mu, vel[c], gc * inv_b);
            vel[c] = vc;
            x[c] = fmaf(-lr, vc, x[c]);
          } else {
            x[c] = fmaf(-lr, gc * inv_b, x[c]);
          }
        }
        if (s == my_k && tid == kThreads - 1) {     // a lane of the last wavefront: idle when d is small
          float sq = 0.0f;
          for (int j = 0; j < batch; ++j) sq = fmaf(res[j], res[j], sq);
          losses[i] = 0.5f * sq * inv_b;
        }
      }
    }
  }
  __syncthreads();
  for (int c = tid; c < d; c += kThreads) {
    x_glob[c] = x[c];
    if (v_glob != nullptr) v_glob[c] = vel[c];
  }
  for (int j = tid; j < batch; j += kThreads)
    idx[(size_t)i * batch + j] = sample_row(seed, (uint32_t)i, t0 + (uint64_t)my_k, (uint32_t)j, log2n);
}

// Sums over the wavefront of R values per lane, each returned in every lane.  The values share the exchange steps: after
// the first one or two, lane l holds a partial sum of value l % R, and one register goes through the others.
template <int CTRL> __device__ __forceinline__ float lane_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int R> __device__ __forceinline__ void wave_sums(float (&v)[R], int lane) {
  static_assert(R == 1 || R == 2 || R == 4, "values that share the exchange");
  constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kRor4 = 0x124, kRor8 = 0x128;   // quad_perm [1,0,3,2], [2,3,0,1]; row_ror
  const bool b0 = (lane & 1) != 0, b1 = (lane & 2) != 0;
  float t;
  if constexpr (R == 1) {
    t = v[0] + lane_move<kXor1>(v[0]);
    t += lane_move<kXor2>(t);
  } else {
    float u[R / 2];
#pragma unroll
    for (int q = 0; q < R / 2; ++q) {
      const float own = b0 ? v[2 * q + 1] : v[2 * q], other = b0 ? v[2 * q] : v[2 * q + 1];
      u[q] = own + lane_move<kXor1>(other);
    }
    if constexpr (R == 2) {
      t = u[0] + lane_move<kXor2>(u[0]);
    } else {
      const float own = b1 ? u[1] : u[0], other = b1 ? u[0] : u[1];
      t = own + lane_move<kXor2>(other);
    }
  }
  t += lane_move<kRor4>(t);
  t += lane_move<kRor8>(t);
  typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
  u32x2_t h = __builtin_amdgcn_permlane16_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  t = __uint_as_float(h.x) + __uint_as_float(h.y);
  h = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  t = __uint_as_float(h.x) + __uint_as_float(h.y);
  if constexpr (R == 1) {
    v[0] = t;
  } else if constexpr (R == 2) {
    v[0] = lane_move<0xA0>(t);                      // quad_perm [0,0,2,2]
    v[1] = lane_move<0xF5>(t);                      // quad_perm [1,1,3,3]
  } else {
    v[0] = lane_move<0x00>(t);
    v[1] = lane_move<0x55>(t);
    v[2] = lane_move<0xAA>(t);
    v[3] = lane_move<0xFF>(t);
  }
}

// Iterations requested ahead by each of W wavefronts with `floats` floats per lane in each: what 128 KB of LDS hold, at
// most 63 requests in flight across a wait, and eight (sixteen are no faster).  Many workers: what 32 KB hold, and one at least.
constexpr int resident_depth(int floats, int W, bool v4, bool many) {
  int depth = (many ? 128 : 512) / W / floats;
  if (depth < 1) depth = 1;
  const int in_flight = 1 + 63 / (v4 ? floats / 4 : floats);
  if (depth > in_flight) depth = in_flight;
  return depth > 8 ? 8 : depth;
}

// Variant for d <= 512 and minibatches of at most 64 rows whose arithmetic stays in registers.  A wavefront owns R
// rows of the minibatch: lane l holds columns l, l + 64, ... of them and of x, so the row products, the residuals and
// the rows' share of the gradient never leave its registers.  Only the W shares of the gradient meet in LDS:
// with four wavefronts every one of them adds the shares and updates a copy of x of its own (one workgroup barrier per
// iteration), with eight each column is added by one thread (two).  The index stream being stateless, the rows
// of iteration s + D are requested D iterations early, straight into LDS; the places are the wavefront's own, so that
// it waits for nothing but its own requests.  A lane draws the R rows of one of 64 iterations at a time (they are
// words of one or two Philox calls) and fetches their targets with them.
// What bounds it: the chain of one iteration (requests, products, wavefront sums, LDS exchange: 880 cycles with d = 64 and 16
// rows), and with the largest minibatches what a compute unit takes in (64 rows of 512: 128 KB in 2.1 us).  Per
// iteration, against the kernels below: 4 x (16 x 64) 0.48 and about 0.95 us, 8 x (64 x 100) 0.85 and 3.9 us, 8 x (33 x
// 300) 2.2 and 21 us, 64 x (64 x 512) 2.9 and 74 us (the last two took the plain kernel).
//
// `interval` > 0: the launch goes on over restarts.  After every iteration whose number is a multiple of the interval
// (but the last of the call) each worker publishes its point and takes the average of all N of them, in the order of
// the restart kernels.  A published float travels with the restart's number in one 8-byte store, so that a
// reader polls the data itself and no separate arrival flag is waited for; two sets of slots alternate: a worker
// can only publish restart e + 2 after everybody has read restart e.  The wait is bounded; on giving up, the abort
// flag ends every workgroup without writing.  A restart takes 1.4 us with 4 workers of 64 floats and 2 us with 64, against
// 17 us for ending a launch, the averaging launch and the start of the next.
template <int CPL, int R, int W, bool V4, bool MANY>
__global__ __launch_bounds__(64 * W) void lsq_resident_kernel(LsqArgs p) {
  static_assert(R == 1 || R == 2 || R == 4 || R == 8, "rows of a wavefront are words of one or two Philox calls");
  constexpr int DC = 64 * CPL;                      // columns held
  static_assert(!V4 || R * CPL >= 4, "a request of 16 bytes per lane is 256 floats");
  constexpr int REQ = V4 ? R * CPL / 4 : R * CPL;   // requests per wavefront and iteration
  constexpr int D = resident_depth(R * CPL, W, V4, MANY);
  static_assert((D - 1) * REQ <= 63, "requests that a wait can leave in flight");
  constexpr bool kOwnSum = W > 4;                   // a column is added by one thread
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];   // [W][D][R][DC] requested rows
  __shared__ float part[kOwnSum ? 1 : 2][W][DC];
  __shared__ float xs[kOwnSum ? DC : 1];
  __shared__ float quarter[4][MANY ? 1 : DC];       // sums of a restart
  __shared__ float resl[W * R];
  __shared__ int bad;

  const int i = blockIdx.x;
  const int my_k = p.worker_steps != nullptr ? min(p.worker_steps[i], p.k) : p.k;
  if (my_k <= 0) return;
  const bool restarts = !MANY && p.interval > 0;
  uint32_t tag = 0;
  if (restarts) {
    if (__hip_atomic_load(p.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
    tag = p.sync[0];                                // restarts published before this launch
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = p.d;
  const float* feat_i = p.features + (size_t)i * p.rows * d;
  const float* targ_i = p.targets + (size_t)i * p.rows;
  const float inv_b = 1.0f / (float)p.batch;
  const int n_rows = min(max(p.batch - wave * R, 0), R);      // rows of this wavefront
  if (tid == 0) bad = 0;

  const float* x_start = p.src + (size_t)i * p.src_stride;
  const bool mom = p.velocity != nullptr;
  float* v_glob = mom ? p.velocity + (size_t)i * p.m_pad : nullptr;
  float x[CPL], vel[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const int col = lane + 64 * c;
    x[c] = col < d ? x_start[col] : 0.0f;
    vel[c] = !kOwnSum && mom && col < d ? v_glob[col] : 0.0f;
  }
  // with one thread per column: its own copy of that column
  float x_own = 0.0f, v_own = 0.0f;
  if (kOwnSum && tid < d) {             // 64 W >= d
    x_own = x_start[tid];
    if (mom) v_own = v_glob[tid];
  }

  // addresses of the rows of iterations 64 chunk + lane (counted from 0 in this call), and their targets
  uint32_t row_lo[R], row_hi[R];
  float y_i[R], y_c[R];                             // of the chunk being requested, and of the one being computed
  auto draw = [&](int chunk) {
    int row[R];
    const uint64_t t = p.t0 + 1 + (uint64_t)chunk * 64 + lane;
    const uint32_t j0 = (uint32_t)(wave * R);
    uint32_t w[4];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r % 4 == 0)
        philox4x32_10((j0 + r) >> 2, (uint32_t)t, (uint32_t)(t >> 32), (uint32_t)i, (uint32_t)p.seed,
                      (uint32_t)(p.seed >> 32), w);
      // j0 is a multiple of R: the words start at the first one unless R < 4
      const uint32_t lo = R >= 4 ? w[r % 4] : R == 2 ? w[r] : (j0 & 1) ? w[1] : w[0];
      const uint32_t hi = R >= 4 ? w[r % 4] : R == 2 ? w[2 + r] : (j0 & 1) ? w[3] : w[2];
      const uint32_t word = (j0 & 2) != 0 ? hi : lo;
      row[r] = p.log2n == 0 ? 0 : (int)(word >> (32 - p.log2n));
    }
    // places past the minibatch repeat its first row (their residuals are set to zero)
    if (n_rows < R) {
      const int row0 = sample_row(p.seed, (uint32_t)i, t, 0, p.log2n);
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r >= n_rows) row[r] = row0;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      y_i[r] = targ_i[row[r]];
      const uint64_t at = (uint64_t)(uintptr_t)(feat_i + (size_t)(uint32_t)row[r] * d);
      row_lo[r] = (uint32_t)at;
      row_hi[r] = (uint32_t)(at >> 32);
    }
  };
  // columns past d repeat the last ones and meet zeros of x, which stay zero
  constexpr int RPR = V4 && CPL < 4 ? 4 / CPL : 1;  // rows of a request
  constexpr int CPR = V4 ? (CPL < 4 ? 1 : CPL / 4) : CPL;            // requests of a row
  uint32_t col_off[CPR];
#pragma unroll
  for (int c = 0; c < CPR; ++c)
    col_off[c] = V4 ? 4u * (uint32_t)min(4 * (RPR > 1 ? lane % (64 / RPR) : lane) + 256 * c, d - 4)
                    : 4u * (uint32_t)min(lane + 64 * c, d - 1);
  float lr[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) lr[c] = lane + 64 * c < d ? p.lr : 0.0f;
  const float lr_own = tid < d ? p.lr : 0.0f;
  const float* ring = reinterpret_cast<const float*>(lds_raw) + (size_t)wave * D * R * DC;
  const uint32_t ring0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds_raw +
                         (uint32_t)(wave * D * R * DC * 4);
  // requests the rows of iteration e of this call into its place; past the last iteration: rows that are not used
  auto request = [&](int e, int place) __attribute__((always_inline)) {
    const int from = e & 63;                        // the lane that drew this iteration
    const uint32_t to = ring0 + (uint32_t)(place * R * DC) * 4u;
    if constexpr (RPR > 1) {
#pragma unroll
      for (int r = 0; r < R; r += RPR) {
        uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)row_lo[r], from);
        uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)row_hi[r], from);
#pragma unroll
        for (int q = 1; q < RPR; ++q) {
          const uint32_t lo_q = (uint32_t)__builtin_amdgcn_readlane((int)row_lo[r + q], from);
          const uint32_t hi_q = (uint32_t)__builtin_amdgcn_readlane((int)row_hi[r + q], from);
          lo = lane >= q * (64 / RPR) ? lo_q : lo;
          hi = lane >= q * (64 / RPR) ? hi_q : hi;
        }
        load_x4_to_lds((((uint64_t)hi << 32) | lo) + col_off[0], to + (uint32_t)(r * DC) * 4u);
      }
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint64_t base = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)row_lo[r], from) |
                              ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)row_hi[r], from) << 32);
#pragma unroll
        for (int c = 0; c < CPR; ++c) {
          if constexpr (V4) load_to_lds(reinterpret_cast<const void*>(base), col_off[c], to + (uint32_t)(r * DC + 256 * c) * 4u);
          else load_dword_to_lds(reinterpret_cast<const void*>(base), col_off[c], to + (uint32_t)(r * DC + 64 * c) * 4u);
        }
      }
    }
  };
  float a[R][CPL];                                  // rows of the iteration being computed
  auto take = [&](int place) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int c = 0; c < CPL; ++c) a[r][c] = ring[(place * R + r) * DC + 64 * c + lane];
  };

  // the targets are waited for here: a wait left to their use would sit in every iteration, behind its requests
  auto take_targets = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      y_c[r] = y_i[r];
      asm volatile("" : "+v"(y_c[r]));
    }
  };
  draw(0);
  take_targets();
#pragma unroll
  for (int u = 0; u < D; ++u) request(u, u);
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"((D - 1) * REQ) : "memory");
  // a wavefront past the minibatch that requests nothing more: no later wait would be for these
  if (MANY && n_rows == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  take(0);
  __syncthreads();

  int to_restart = 0;                               // iterations left in this epoch
  if (restarts) to_restart = p.interval - (int)(p.t0 % (uint64_t)p.interval);

  auto restart = [&]() -> bool {
    ++tag;
    unsigned long long* slots = p.exchange + (size_t)(tag & 1) * p.n_workers * d;
    if (kOwnSum) {
      if (tid < d)
        __hip_atomic_store(slots + (size_t)i * d + tid, ((unsigned long long)tag << 32) | __float_as_uint(x_own),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (wave == 0) {
#pragma unroll
      for (int c = 0; c < CPL; ++c)
        if (lane + 64 * c < d)
          __hip_atomic_store(slots + (size_t)i * d + lane + 64 * c,
                             ((unsigned long long)tag << 32) | __float_as_uint(x[c]), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    }
    const int n = p.n_workers, n_q = n >= 8 ? 4 : 1, n_per = (n + n_q - 1) / n_q;   // as the restart kernels add
    unsigned polls = 0;
    for (int e = tid; e < n_q * d; e += 64 * W) {
      const int q = e / d, c = e - q * d;
      const int lo = min(n, q * n_per), hi = min(n, lo + n_per);
      const unsigned long long* from = slots + c;
      float acc = 0.0f;
      for (int i0 = lo; i0 < hi; i0 += 16) {
        unsigned long long v[16];
        for (;;) {
          bool all = true;
#pragma unroll
          for (int u = 0; u < 16; ++u)
            v[u] = __hip_atomic_load(from + (size_t)min(i0 + u, hi - 1) * d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
          for (int u = 0; u < 16; ++u) all = all && (uint32_t)(v[u] >> 32) == tag;
          if (all) break;
          if (++polls > p.spin_limit ||
              ((polls & 15) == 0 &&
               __hip_atomic_load(p.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
            __hip_atomic_store(p.abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bad = 1;
            break;
          }
        }
#pragma unroll
        for (int u = 0; u < 16; ++u)
          if (i0 + u < hi) acc += __uint_as_float((uint32_t)v[u]);
      }
      quarter[q][c] = acc;
    }
    __syncthreads();
    if (bad != 0) return false;
    auto mean_of = [&](int c) {
      float total = quarter[0][c];
      if (n_q == 4) total = ((total + quarter[1][c]) + quarter[2][c]) + quarter[3][c];
      return total / (float)n;
    };
#pragma unroll
    for (int c = 0; c < CPL; ++c)
      if (lane + 64 * c < d) x[c] = mean_of(lane + 64 * c);
    if (kOwnSum && tid < d) x_own = mean_of(tid);
    return true;                                    // an iteration's barrier comes before the next write of `quarter`
  };

  int place = 0;                                    // of iteration s
  for (int s = 0; s < my_k; ++s) {
    if (((s + D) & 63) == 0) draw((s + D) >> 6);
    if ((s & 63) == 0 && s > 0) take_targets();
    // This iteration's rows are in registers.  With many workers a wavefront past the minibatch keeps the rows of the first D
    // iterations, which meet residuals of zero.  With one workgroup per compute unit the branch costs more than the requests: 38 x
    // (58 x 205) 3.57 and 3.74 us per iteration, 7 x (16 x 19) 0.73 and 0.76 (but 3 x (19 x 360) 1.98 and 1.77).
    if (!MANY || n_rows > 0) request(s + D, place);
    place = place + 1 == D ? 0 : place + 1;
    float res[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float dot = 0.0f;
#pragma unroll
      for (int c = 0; c < CPL; ++c) dot = fmaf(a[r][c], x[c], dot);
      res[r] = dot;
    }
#pragma unroll
    for (int q = 0; q < R; q += 4) {
      float(&four)[R < 4 ? R : 4] = *reinterpret_cast<float(*)[R < 4 ? R : 4]>(&res[q]);
      wave_sums(four, lane);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      res[r] -= __int_as_float(__builtin_amdgcn_readlane(__float_as_int(y_c[r]), s & 63));
      if (r >= n_rows) res[r] = 0.0f;               // the same in all lanes
    }
    float g[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) g[c] = 0.0f;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int c = 0; c < CPL; ++c) g[c] = fmaf(a[r][c], res[r], g[c]);
    float(*pt)[DC] = part[kOwnSum ? 0 : s & 1];
#pragma unroll
    for (int c = 0; c < CPL; ++c) pt[wave][lane + 64 * c] = g[c];
    if (s == my_k - 1 && lane == 0) {
#pragma unroll
      for (int r = 0; r < R; ++r) resl[wave * R + r] = res[r];
    }
    // the rows of the next iteration, requested before the D - 1 that may still be under way
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((D - 1) * REQ) : "memory");
    take(place);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if constexpr (kOwnSum) {
      if (tid < DC) {
        float gc = pt[0][tid];
#pragma unroll
        for (int w = 1; w < W; ++w) gc += pt[w][tid];
        if (mom) { v_own = fmaf(p.mu, v_own, gc * inv_b); x_own = fmaf(-lr_own, v_own, x_own); }
        else x_own = fmaf(-lr_own, gc * inv_b, x_own);
        xs[tid] = x_own;
      }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
      for (int c = 0; c < CPL; ++c) x[c] = xs[lane + 64 * c];
    } else {
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        float gc = pt[0][lane + 64 * c];
#pragma unroll
        for (int w = 1; w < W; ++w) gc += pt[w][lane + 64 * c];
        if (mom) { vel[c] = fmaf(p.mu, vel[c], gc * inv_b); x[c] = fmaf(-lr[c], vel[c], x[c]); }
        else x[c] = fmaf(-lr[c], gc * inv_b, x[c]);
      }
    }
    if (restarts && --to_restart == 0) {
      to_restart = p.interval;
      if (s + 1 < my_k && !restart()) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no request into LDS outlives the workgroup

  __syncthreads();
  float* x_glob = p.params + (size_t)i * p.m_pad;
  if constexpr (kOwnSum) {
    if (tid < d) {
      x_glob[tid] = x_own;
      if (mom) v_glob[tid] = v_own;
    }
  } else if (wave == 0) {
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      const int col = lane + 64 * c;
      if (col < d) {
        x_glob[col] = x[c];
        if (mom) v_glob[col] = vel[c];
      }
    }
  }
  if (tid < p.batch)
    p.idx[(size_t)i * p.batch + tid] =
        sample_row(p.seed, (uint32_t)i, p.t0 + (uint64_t)my_k, (uint32_t)tid, p.log2n);
  if (tid == 0) {
    float sq = 0.0f;
    for (int j = 0; j < p.batch; ++j) sq = fmaf(resl[j], resl[j], sq);
    p.losses[i] = 0.5f * sq * inv_b;
    if (restarts && i == 0) p.sync[0] = tag;        // everybody has read it: all took part in the last restart
  }
}

constexpr int kResidentDim = 512, kResidentBatch = 64;
// From more workers than compute units on, several workgroups have to share one, and each hides the others' latency: rings of a
// quarter, no restart sums.  Per iteration with a launch after every eighth, rings of 128 KB and of 32 KB: 512 x (64 x 64) 4.4 and
// 3.1 us, 1024 x (1 x 512) 7.0 and 4.3, 4000 x (32 x 128) 27.7 and 15.8 (staged kernel 5.5, 4.4 and 19.9).
constexpr int kManyWorkers = 256;
static bool lsq_resident(int d, int batch) { return d <= kResidentDim && batch <= kResidentBatch; }

template <int CPL, int R, int W, bool V4, bool MANY> static hipError_t launch_resident_v(const LsqArgs& p, hipStream_t s) {
  constexpr size_t kRing = (size_t)W * resident_depth(R * CPL, W, V4, MANY) * R * CPL * 256;
  auto kernel = lsq_resident_kernel<CPL, R, W, V4, MANY>;
  static std::atomic<bool> configured{false};
  if (!configured.load(std::memory_order_acquire)) {      // rows and shares can exceed the 64 KB default
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRing);
    if (e != hipSuccess) return e;
    configured.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(kernel, dim3(p.n_workers), dim3(64 * W), kRing, s, p);
  return hipGetLastError();
}
template <int CPL, int R, int W> static hipError_t launch_resident(const LsqArgs& p, hipStream_t s) {
  const bool many = p.n_workers > kManyWorkers;
  if constexpr (R * CPL >= 4) {
    if ((p.d & 3) == 0)                                                      // 16-byte aligned rows
      return many ? launch_resident_v<CPL, R, W, true, true>(p, s) : launch_resident_v<CPL, R, W, true, false>(p, s);
  }
  return many ? launch_resident_v<CPL, R, W, false, true>(p, s) : launch_resident_v<CPL, R, W, false, false>(p, s);
}
template <int CPL> static hipError_t launch_resident_rows(const LsqArgs& p, hipStream_t s) {
  if (p.batch <= 4) return launch_resident<CPL, 1, 4>(p, s);
  if (p.batch <= 8) return launch_resident<CPL, 2, 4>(p, s);
  if (p.batch <= 16) return launch_resident<CPL, 4, 4>(p, s);
  if (p.batch <= 32) return launch_resident<CPL, 4, 8>(p, s);
  return launch_resident<CPL, 8, 8>(p, s);
}

// Whether one launch may go on over restarts: every workgroup reads every worker's point (N d 8 bytes), and all
// of them have to be resident together.
bool lsq_restarts_in_launch(int n_workers, int d, int batch) {
  return lsq_resident(d, batch) && n_workers <= kLsqMaxTeam && (long)n_workers * d <= kLsqMaxExchange;
}
size_t lsq_exchange_bytes(int n_workers, int d) { return 2 * sizeof(unsigned long long) * (size_t)n_workers * d; }

hipError_t launch_lsq_steps(LsqArgs p, hipStream_t s) {
  if (p.k <= 0) return hipSuccess;
  p.log2n = ilog2_rows(p.rows);
  const int d = p.d, batch = p.batch;
  if (lsq_resident(d, batch)) {
    if (d <= 64) return launch_resident_rows<1>(p, s);
    if (d <= 128) return launch_resident_rows<2>(p, s);
    if (d <= 256) return launch_resident_rows<4>(p, s);
    return launch_resident_rows<8>(p, s);
  }
  if (p.interval > 0) return hipErrorInvalidValue;
  const long floats = (long)batch * d;
  if ((d & 3) == 0 && floats <= kMaxStagedFloats && batch <= kMaxStagedBatch) {
    const int pfv = (int)((floats / 4 + kThreads - 1) / kThreads);
#define STAGED(PFV, D)                                                                                  \
  do {                                                                                                  \
    const size_t lds_b = (2 * (size_t)floats + 2 * (size_t)d + 3 * (size_t)batch + 3 * (size_t)D * batch) * \
                         sizeof(float);                                                                 \
    if (lds_b > 48 * 1024) {                                                                            \
      const hipError_t ea = hipFuncSetAttribute(                                                        \
          reinterpret_cast<const void*>(lsq_steps_staged_kernel<PFV, D>),                               \
          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_b);                                      \
      if (ea != hipSuccess) return ea;                                                                  \
    }                                                                                                   \
    hipLaunchKernelGGL((lsq_steps_staged_kernel<PFV, D>), dim3(p.n_workers), dim3(kThreads), lds_b, s, p); \
    return hipGetLastError();                                                                           \
  } while (0)
    if (pfv <= 1) STAGED(1, 8);
    if (pfv <= 2) STAGED(2, 4);
    if (pfv <= 4) STAGED(4, 2);
    STAGED(8, 1);
#undef STAGED
  }
  // at most (2 * 8192 + 2 * 4096) floats = 96 KiB: inside the 160 KiB of a compute unit, but
  // above the default limit of a launch
  const size_t lds_bytes = (2 * (size_t)d + 2 * (size_t)batch) * sizeof(float);
  if (lds_bytes > 48 * 1024) {
    const hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(lsq_steps_kernel),
                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (ea != hipSuccess) return ea;
  }
  hipLaunchKernelGGL(lsq_steps_kernel, dim3(p.n_workers), dim3(kThreads), lds_bytes, s, p);
  return hipGetLastError();
}

}  // namespace prsgd
