// Minibatch draw zeta_i^t and the loss head of the MLP.
//
// Section 1 of the paper only requires unbiased stochastic gradients that are independent
// across workers and iterations.  Here worker i draws B rows of its own shard uniformly with
// replacement; slot j of iteration t is a pure function of (seed, i, t, j) through
// Philox4x32-10, so the stream needs no state and can be replayed from any t.
#include <cstring>
#include <type_traits>

#include "prsgd_internal.h"

namespace prsgd {

static int ilog2(long n) {
  int l = 0;
  while ((1L << l) < n) ++l;
  return l;
}

// One workgroup per (slot j, worker i): draw the row, copy it into the batch buffer.  Bound by the latency of the row's
// loads: all of a round (4 vectors or 8 single words per thread, clamped to the row so that no load is conditional) are
// issued before the first store, which the compiler cannot move them across, and the label is stored last.  Per iteration,
// against a load and a store in turn: 8 workers, 512 rows of 3072 215.9 -> 212.8 us, 16 workers, 64 rows 144.3 -> 143.8 us.
template <bool BF16>
__device__ __forceinline__ void gather_row(const GatherArgs& a, int j, int i) {
  const int32_t row = sample_row(a.seed, (uint32_t)i, a.t, (uint32_t)j, a.log2n);
  const size_t slot = (size_t)i * a.batch + j;
  const int32_t label = a.labels[(size_t)i * a.rows + row];
  const int d0 = a.d0, ld0 = a.ld0;
  const float* src = a.features + ((size_t)i * a.rows + row) * d0;
  if ((d0 & 3) == 0) {
    constexpr int U = 4;
    const int n4 = d0 / 4;
    typedef float f32x4_t __attribute__((ext_vector_type(4)));      // arrays of float4 structs end in scratch memory
    const f32x4_t* src4 = reinterpret_cast<const f32x4_t*>(src);
    for (int c0 = threadIdx.x; c0 < n4; c0 += U * kThreads) {
      f32x4_t v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const f32x4_t* at = src4 + min(c0 + u * kThreads, n4 - 1);
        v[u] = a.once ? __builtin_nontemporal_load(at) : *at;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + u * kThreads;
        if (c >= n4) break;
        if (BF16) {
          uint2 h;
          h.x = f32x2_to_bf16x2_rne(v[u].x, v[u].y);
          h.y = f32x2_to_bf16x2_rne(v[u].z, v[u].w);
          reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.xb) + slot * ld0)[c] = h;
        } else {
          reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(a.xb) + slot * ld0)[c] = v[u];
        }
      }
    }
  } else {
    constexpr int U = 8;
    for (int c0 = threadIdx.x; c0 < d0; c0 += U * kThreads) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float* at = src + min(c0 + u * kThreads, d0 - 1);
        v[u] = a.once ? __builtin_nontemporal_load(at) : *at;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) asm volatile("" : "+v"(v[u]));         // a load is not moved to its conditional store
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + u * kThreads;
        if (c >= d0) break;
        if (BF16) reinterpret_cast<uint16_t*>(a.xb)[slot * ld0 + c] = f32_to_bf16_rne(v[u]);
        else reinterpret_cast<float*>(a.xb)[slot * ld0 + c] = v[u];
      }
    }
  }
  if (threadIdx.x == 0) {
    a.idx[slot] = row;
    a.yb[slot] = label;
  }
}

// ... of the i-th of the workers that draw; nothing for an i past them.
template <bool BF16>
__device__ __forceinline__ void gather_group(const GatherArgs& a, int j, int i) {
  if (i >= a.workers) return;
  gather_row<BF16>(a, j, worker_of(a.order, i));
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void gather_kernel(GatherArgs a) {
  gather_group<BF16>(a, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kThreads) void sample_indices_kernel(int32_t* __restrict__ out,
                                                                  int n_workers, int batch, int log2n,
                                                                  uint64_t seed, uint64_t t_first,
                                                                  size_t total) {
  for (size_t k = (size_t)blockIdx.x * kThreads + threadIdx.x; k < total;
       k += (size_t)gridDim.x * kThreads) {
    const uint32_t j = (uint32_t)(k % batch);
    const uint32_t i = (uint32_t)((k / batch) % n_workers);
    const uint64_t s = k / ((size_t)batch * n_workers);
    out[k] = sample_row(seed, i, t_first + s, j, log2n);
  }
}

// Logits of classes c0, c0 + STRIDE, ... of one row: the product's output, or (split contraction) the bias plus the partial
// sums in split order.  All Q (S + 1) loads are in flight together: indices are clamped, no load is conditional.
template <int Q, int STRIDE, int S>
__device__ __forceinline__ void fetch_logits_parts(float (&z)[Q], const float* __restrict__ row, long part_stride,
                                                   const float* __restrict__ bias, int c0, int n_classes) {
  float v[Q][S], add[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int c = min(c0 + STRIDE * q, n_classes - 1);
    add[q] = bias != nullptr ? bias[c] : 0.0f;
#pragma unroll
    for (int s = 0; s < S; ++s) v[q][s] = row[(size_t)s * part_stride + c];
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    float t = add[q];
#pragma unroll
    for (int s = 0; s < S; ++s) t += v[q][s];
    z[q] = c0 + STRIDE * q < n_classes ? t : -INFINITY;
  }
}
template <int Q, int STRIDE>
__device__ __forceinline__ void fetch_logits(float (&z)[Q], const float* __restrict__ row, int n_parts, long part_stride,
                                             const float* __restrict__ bias, int c0, int n_classes) {
  if (n_parts == kMaxLogitSplits) return fetch_logits_parts<Q, STRIDE, kMaxLogitSplits>(z, row, part_stride, bias, c0, n_classes);
  if (n_parts == 2) return fetch_logits_parts<Q, STRIDE, 2>(z, row, part_stride, bias, c0, n_classes);
  fetch_logits_parts<Q, STRIDE, 1>(z, row, part_stride, bias, c0, n_classes);
}

// Bytes of arguments that the loss heads have at least (what they have in front of the gather's, and the gather's).
constexpr size_t kHeadArgBytes = 88 + sizeof(GatherArgs);
// Softmax cross-entropy head: one wavefront per minibatch row (4 rows per workgroup).  The same
// launch can carry the row gather of the next iteration in extra workgroups.
//   row_loss[b] = -log softmax(z_b)[c_b],   delta = (softmax(z) - onehot(c)) / B
template <bool BF16>
__global__ __launch_bounds__(kThreads) void softmax_xent_kernel(
    const float* __restrict__ logits, int n_parts, long part_stride, const float* __restrict__ bias,
    long bias_gs, const int32_t* __restrict__ yb, void* __restrict__ delta,
    float* __restrict__ row_loss, int batch, int n_classes, int ldc,
    const int* __restrict__ order, int head_blocks, GatherArgs next) {
  fetch_kernel_args<kHeadArgBytes>();
  int g = blockIdx.y;
  // workgroups beyond the loss head's own: the minibatch draw of the NEXT iteration, which depends
  // on nothing this iteration computes (zeta_i^t is a function of seed, i, t and the slot alone)
  if ((int)blockIdx.x >= head_blocks) {
    gather_group<BF16>(next, (int)blockIdx.x - head_blocks, g);
    return;
  }
  g = worker_of(order, g);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = blockIdx.x * (kThreads / kWave) + wave;
  if (b >= batch) return;
  const float inv_b = 1.0f / (float)batch;
  const size_t r = (size_t)g * batch + b;
  // logit of class c: the product's output, or (split contraction) the bias plus the partial
  // sums in split order
  const float* bias_g = bias != nullptr ? bias + (size_t)g * bias_gs : nullptr;
  auto logit = [&](int c) {
    float z = bias_g != nullptr ? bias_g[c] : 0.0f;
    for (int s = 0; s < n_parts; ++s) z += logits[(size_t)s * part_stride + r * ldc + c];
    return z;
  };
  const int label = yb[r];
  constexpr int ZR = 4;                              // classes per lane held in registers
  if (n_classes <= ZR * kWave) {
    float z[ZR];
    float mx = -INFINITY;
    fetch_logits<ZR, kWave>(z, logits + r * ldc, n_parts, part_stride, bias_g, lane, n_classes);
#pragma unroll
    for (int q = 0; q < ZR; ++q) mx = fmaxf(mx, z[q]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    float zl = 0.0f, se = 0.0f;                      // the label's logit lives in one lane
#pragma unroll
    for (int q = 0; q < ZR; ++q) {
      const int c = lane + kWave * q;
      if (c == label && c < n_classes) zl = z[q];
      z[q] = c < n_classes ? expf(z[q] - mx) : 0.0f;
      se += z[q];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      se += __shfl_xor(se, o);
      zl += __shfl_xor(zl, o);
    }
#pragma unroll
    for (int q = 0; q < ZR; ++q) {
      const int c = lane + kWave * q;
      if (c < ldc) {
        const float d = c < n_classes ? (z[q] / se - (c == label ? 1.0f : 0.0f)) * inv_b : 0.0f;
        if (BF16) reinterpret_cast<uint16_t*>(delta)[r * ldc + c] = f32_to_bf16_rne(d);
        else reinterpret_cast<float*>(delta)[r * ldc + c] = d;
      }
    }
    // an out-of-range label selects nothing (zl stays 0)
    if (lane == 0) row_loss[r] = (mx + logf(se)) - zl;
    return;
  }
  float mx = -INFINITY;
  for (int c = lane; c < n_classes; c += kWave) mx = fmaxf(mx, logit(c));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  float se = 0.0f;
  for (int c = lane; c < n_classes; c += kWave) se += expf(logit(c) - mx);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) se += __shfl_xor(se, o);
  for (int c = lane; c < ldc; c += kWave) {
    float d = 0.0f;
    if (c < n_classes) d = (expf(logit(c) - mx) / se - (c == label ? 1.0f : 0.0f)) * inv_b;
    if (BF16) reinterpret_cast<uint16_t*>(delta)[r * ldc + c] = f32_to_bf16_rne(d);
    else reinterpret_cast<float*>(delta)[r * ldc + c] = d;
  }
  // an out-of-range label must not index outside the row
  const float z_label = (label >= 0 && label < n_classes) ? logit(label) : 0.0f;
  if (lane == 0) row_loss[r] = (mx + logf(se)) - z_label;
}

// The same head for wide class counts (257 .. 1024): one workgroup per minibatch row, at most four
// classes per thread, so that a row's loads are spread over four wavefronts instead of queueing in
// one (1000 classes, four partial sums per logit: 20 loads per lane instead of 80).
template <bool BF16>
__global__ __launch_bounds__(kThreads) void softmax_xent_row_kernel(
    const float* __restrict__ logits, int n_parts, long part_stride, const float* __restrict__ bias,
    long bias_gs, const int32_t* __restrict__ yb, void* __restrict__ delta,
    float* __restrict__ row_loss, int batch, int n_classes, int ldc,
    const int* __restrict__ order, int head_blocks, GatherArgs next) {
  fetch_kernel_args<kHeadArgBytes>();
  int g = blockIdx.y;
  if ((int)blockIdx.x >= head_blocks) {                 // the minibatch draw of the next iteration
    gather_group<BF16>(next, (int)blockIdx.x - head_blocks, g);
    return;
  }
  g = worker_of(order, g);
  __shared__ float red[3][kThreads / kWave];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const size_t r = (size_t)g * batch + blockIdx.x;
  const float inv_b = 1.0f / (float)batch;
  const float* bias_g = bias != nullptr ? bias + (size_t)g * bias_gs : nullptr;
  const int label = yb[r];
  constexpr int ZT = 4;                                 // classes per thread
  float z[ZT];
  float mx = -INFINITY;
  fetch_logits<ZT, kThreads>(z, logits + r * ldc, n_parts, part_stride, bias_g, tid, n_classes);
#pragma unroll
  for (int q = 0; q < ZT; ++q) mx = fmaxf(mx, z[q]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  if (lane == 0) red[0][wave] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
  float se = 0.0f, zl = 0.0f;                           // the label's logit lives in one thread
#pragma unroll
  for (int q = 0; q < ZT; ++q) {
    const int c = tid + kThreads * q;
    if (c == label && c < n_classes) zl = z[q];
    z[q] = c < n_classes ? expf(z[q] - mx) : 0.0f;
    se += z[q];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    se += __shfl_xor(se, o);
    zl += __shfl_xor(zl, o);
  }
  if (lane == 0) { red[1][wave] = se; red[2][wave] = zl; }
  __syncthreads();
  se = ((red[1][0] + red[1][1]) + red[1][2]) + red[1][3];     // fixed order
  zl = ((red[2][0] + red[2][1]) + red[2][2]) + red[2][3];
#pragma unroll
  for (int q = 0; q < ZT; ++q) {
    const int c = tid + kThreads * q;
    if (c < ldc) {
      const float d = c < n_classes ? (z[q] / se - (c == label ? 1.0f : 0.0f)) * inv_b : 0.0f;
      if (BF16) reinterpret_cast<uint16_t*>(delta)[r * ldc + c] = f32_to_bf16_rne(d);
      else reinterpret_cast<float*>(delta)[r * ldc + c] = d;
    }
  }
  if (tid == 0) row_loss[r] = (mx + logf(se)) - zl;     // an out-of-range label selects nothing
}

// Head of at most 64 classes: the logits product is taken here as well,
//   z_b = H_{L-1}[b, :] W_L + b_L        (bf16 operands: bf16(W_L)),
// 16 minibatch rows per workgroup on the matrix cores, the contraction dealt to the four wavefronts in pieces; the four
// partial blocks are added in order.  Then 16 lanes per row, CT classes each (classes past the last are zero columns).
//   bf16: v_mfma_f32_16x16x32; a wavefront takes its H fragments straight from memory and turns its rows of W_L through LDS
//         of its own
//   fp32: v_mfma_f32_16x16x4; contraction element 4 q4 + q of every 16 in step q, so that an H fragment is one 16-byte load
// It saves the launch of a small product: an iteration of 784-300-100-10 in fp32 (8 workers, 50 rows) 49.6 -> 44.5 us, of
// 1000-500-300-37 in bf16 (6 workers, 100 rows) 50.5 -> 46.3 us; with up to 16 classes in bf16 it replaces a wavefront per row with
// multiply-adds, which was bound by its instructions (16 workers of 3072-1024-1024-10, 64 rows: 147.5 -> 144.2 us).
constexpr int kHeadRows = 16;
constexpr int kHeadClasses = 64;

template <int CTRL> __device__ __forceinline__ float row_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float head_row_max(float v) {                 // over 16 lanes
  v = fmaxf(v, row_move<0xB1>(v));
  v = fmaxf(v, row_move<0x4E>(v));
  v = fmaxf(v, row_move<0x141>(v));
  return fmaxf(v, row_move<0x140>(v));
}
__device__ __forceinline__ float head_row_sum(float v) {
  v += row_move<0xB1>(v);
  v += row_move<0x4E>(v);
  v += row_move<0x141>(v);
  return v + row_move<0x140>(v);
}

// With DX the workgroup also takes its rows' delta one layer down, D_{L-1} = (D_L W_L^T) phi'(H_{L-1}): it has D_L, and reads
// W_L a second time (softmax_narrow_delta_pays bounds that).  Transposed, 16 units by 16 rows, so that a lane holds four consecutive
// units of a row; the operand of W_L comes straight from memory, four tiles of it per wavefront in flight.  One launch fewer: 16
// iterations of eight workers of 784-300-100-10 in fp32 605 -> 565 us, of six of 1000-500-300-37 in bf16 633 -> 598 us.
template <bool BF16, int CT, bool DX>
__global__ __launch_bounds__(kThreads) void softmax_xent_narrow_kernel(
    const void* __restrict__ h_any, long h_gs, int ldh, int k_dim, const void* __restrict__ w_any,
    long w_gs, const float* __restrict__ bias, long bias_gs, const int32_t* __restrict__ yb,
    void* __restrict__ delta, float* __restrict__ row_loss, int batch, int n_classes, int ldc,
    const int* __restrict__ order, int head_blocks, GatherArgs next, HeadDelta below) {
  fetch_kernel_args<kHeadArgBytes + 16 + sizeof(HeadDelta)>();
  int g = blockIdx.y;
  if ((int)blockIdx.x >= head_blocks) {                 // the minibatch draw of the next iteration
    gather_group<BF16>(next, (int)blockIdx.x - head_blocks, g);
    return;
  }
  g = worker_of(order, g);
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
  constexpr int NW = kThreads / kWave;
  __shared__ float part[NW][kHeadRows][16 * CT + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n16 = lane & 15, q4 = lane >> 4;
  const int b0 = (int)blockIdx.x * kHeadRows;
  const size_t h_row = (size_t)g * h_gs + (size_t)min(b0 + n16, batch - 1) * ldh;        // rows past the end: not stored
  // what the softmax part needs from memory is requested before the product: 1000-500-300-37 in bf16 46.1 -> 45.7 us per iteration
  const int row = tid >> 4, l16 = tid & 15, b = b0 + row;
  const int label = yb[(size_t)g * batch + min(b, batch - 1)];
  float bias_c[CT];
  f32x4_t acc[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    bias_c[ct] = bias[(size_t)g * bias_gs + min(16 * ct + l16, n_classes - 1)];
    acc[ct] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
  }
  if constexpr (BF16) {
    typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4_t;
    typedef __attribute__((address_space(3))) bf16x4_t* lds_bf16x4_ptr;
    constexpr int kPiece = 256 / CT;                    // contraction elements of a wavefront and step
    constexpr int CPR = 2 * CT, RPL = kWave / CPR;      // 16-byte chunks of a row, rows of a load
    __shared__ __attribute__((aligned(16))) uint16_t w_lds[NW][kPiece][16 * CT];
    const uint16_t* h_r = reinterpret_cast<const uint16_t*>(h_any) + h_row;
    const uint16_t* w_g = reinterpret_cast<const uint16_t*>(w_any) + (size_t)g * w_gs;   // [k_dim][ldc]
    const u32x4_t zero = {0u, 0u, 0u, 0u};
    const int wr = lane / CPR, wc = 8 * (lane % CPR);
    for (int k0 = wave * kPiece; k0 < k_dim; k0 += NW * kPiece) {
      u32x4_t a[kPiece / 32], w[kPiece / RPL];
#pragma unroll
      for (int u = 0; u < kPiece / 32; ++u) {           // columns [k_dim, ldh) of H are zero
        const int k = k0 + 32 * u + 8 * q4;
        a[u] = k < k_dim ? *reinterpret_cast<const u32x4_t*>(h_r + k) : zero;
      }
#pragma unroll
      for (int u = 0; u < kPiece / RPL; ++u) {
        const int k = k0 + RPL * u + wr;
        w[u] = k < k_dim && wc < ldc ? *reinterpret_cast<const u32x4_t*>(w_g + (size_t)k * ldc + wc) : zero;
      }
#pragma unroll
      for (int u = 0; u < kPiece / RPL; ++u) *reinterpret_cast<u32x4_t*>(&w_lds[wave][RPL * u + wr][wc]) = w[u];
      __builtin_amdgcn_wave_barrier();                  // the piece is this wavefront's own
#pragma unroll
      for (int u = 0; u < kPiece / 32; ++u)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          // lane (class n16, q4) takes W[32 u + 8 q4 .. + 7][n16]: two transposed reads of four rows (see frag_trans)
          const uint16_t* p = &w_lds[wave][32 * u + 8 * q4 + (n16 >> 2)][16 * ct + 4 * (n16 & 3)];
          const bf16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p));
          const bf16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p + 4 * 16 * CT));
          const bf16x8_t wf = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a[u]), wf, acc[ct], 0, 0, 0);
        }
      __builtin_amdgcn_wave_barrier();
    }
  } else {
    const float* h_r = reinterpret_cast<const float*>(h_any) + h_row;
    const float* w_g = reinterpret_cast<const float*>(w_any) + (size_t)g * w_gs;
    constexpr int U = CT == 1 ? 4 : 2;                  // 16-deep pieces in flight
    for (int k0 = wave * 16 * U; k0 < k_dim; k0 += NW * 16 * U) {
      f32x4_t a[U];
      float w[U][4][CT];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = k0 + 16 * u + 4 * q4;
        a[u] = k < k_dim ? *reinterpret_cast<const f32x4_t*>(h_r + k) : (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
            w[u][q][ct] = k + q < k_dim && 16 * ct + n16 < ldc ? w_g[(size_t)(k + q) * ldc + 16 * ct + n16] : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
            acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][q], w[u][q][ct], acc[ct], 0, 0, 0);
    }
  }
  // element v of lane (n16, q4) is row 4 q4 + v, class n16 of the tile
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int v = 0; v < 4; ++v) part[wave][4 * q4 + v][16 * ct + n16] = acc[ct][v];
  constexpr int KC = BF16 && CT == 1 ? 32 : 16 * CT;    // classes as the contraction of D_{L-1}: past the last ones zeros
  using DE = std::conditional_t<BF16, uint16_t, float>;
  constexpr int DS = KC + 16 / (int)sizeof(DE);         // row stride of D_L in LDS
  __shared__ __attribute__((aligned(16))) DE d_lds[DX ? kHeadRows * DS : 1];
  if (DX)
    for (int e = tid; e < kHeadRows * DS; e += kThreads) d_lds[e] = 0;
  __syncthreads();
  if (!DX && b >= batch) return;                        // whole groups of 16 lanes
  if (b < batch) {
    const size_t r = (size_t)g * batch + b;
    float z[CT], mx = -INFINITY;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int c = 16 * ct + l16;
      z[ct] = -INFINITY;
      if (c < n_classes)
        z[ct] = (((part[0][row][c] + part[1][row][c]) + part[2][row][c]) + part[3][row][c]) + bias_c[ct];
      mx = fmaxf(mx, z[ct]);
    }
    mx = head_row_max(mx);
    float e[CT], se = 0.0f, zl = 0.0f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int c = 16 * ct + l16;
      if (c == label && c < n_classes) zl = z[ct];        // an out-of-range label selects nothing
      e[ct] = c < n_classes ? expf(z[ct] - mx) : 0.0f;
      se += e[ct];
    }
    se = head_row_sum(se);
    zl = head_row_sum(zl);
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int c = 16 * ct + l16;
      if (c < ldc) {
        const float d = c < n_classes ? (e[ct] / se - (c == label ? 1.0f : 0.0f)) * (1.0f / (float)batch) : 0.0f;
        if (BF16) reinterpret_cast<uint16_t*>(delta)[r * ldc + c] = f32_to_bf16_rne(d);
        else reinterpret_cast<float*>(delta)[r * ldc + c] = d;
        if constexpr (DX) {
          if constexpr (BF16) d_lds[row * DS + c] = f32_to_bf16_rne(d);
          else d_lds[row * DS + c] = d;
        }
      }
    }
    if (l16 == 0) row_loss[r] = (mx + logf(se)) - zl;
  }
  if constexpr (DX) {
    __syncthreads();
    const bool row_ok = b0 + n16 < batch;
    constexpr int U = 4;                                // tiles in flight
    const int tiles = (below.ld + 15) / 16;
    DE* out = reinterpret_cast<DE*>(below.out) + (size_t)g * below.gs + (size_t)min(b0 + n16, batch - 1) * below.ld;
    const DE* h_r = reinterpret_cast<const DE*>(h_any) + h_row;
    const DE* w_g = reinterpret_cast<const DE*>(w_any) + (size_t)g * w_gs;
    typedef std::conditional_t<BF16, uint2, f32x4_t> H4;   // four units of H_{L-1}
    constexpr int NF = BF16 ? KC / 32 : CT;             // 16-byte pieces of a lane along the classes
    u32x4_t df[NF];
#pragma unroll
    for (int s = 0; s < NF; ++s)
      df[s] = *reinterpret_cast<const u32x4_t*>(&d_lds[n16 * DS + (BF16 ? 32 * s + 8 * q4 : 16 * s + 4 * q4)]);
    for (int t0 = wave; t0 < tiles; t0 += NW * U) {
      u32x4_t w[U][NF];
      H4 hv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j0 = 16 * min(t0 + NW * u, tiles - 1);
#pragma unroll
        for (int s = 0; s < NF; ++s) {
          const int c = BF16 ? 32 * s + 8 * q4 : 16 * s + 4 * q4;
          w[u][s] = c < ldc ? *reinterpret_cast<const u32x4_t*>(w_g + (size_t)min(j0 + n16, k_dim - 1) * ldc + c)
                            : (u32x4_t){0u, 0u, 0u, 0u};      // and not some other class: zero times infinity is a NaN
        }
        hv[u] = *reinterpret_cast<const H4*>(h_r + min(j0 + 4 * q4, ldh - 4));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = 16 * (t0 + NW * u) + 4 * q4;
        f32x4_t z = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < NF; ++s) {                  // both are zero past the last class
          if constexpr (BF16) {
            z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[u][s]),
                                                        __builtin_bit_cast(bf16x8_t, df[s]), z, 0, 0, 0);
          } else {
            const f32x4_t wf = __builtin_bit_cast(f32x4_t, w[u][s]), dv = __builtin_bit_cast(f32x4_t, df[s]);
#pragma unroll
            for (int q = 0; q < 4; ++q) z = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[q], dv[q], z, 0, 0, 0);
          }
        }
        float hf[4];
        if constexpr (BF16) {
          hf[0] = bf16_to_f32((uint16_t)hv[u].x); hf[1] = bf16_to_f32((uint16_t)(hv[u].x >> 16));
          hf[2] = bf16_to_f32((uint16_t)hv[u].y); hf[3] = bf16_to_f32((uint16_t)(hv[u].y >> 16));
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) hf[e] = hv[u][e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float slope = below.act == PRSGD_TANH ? 1.0f - hf[e] * hf[e] : hf[e] > 0.0f ? 1.0f : 0.0f;
          z[e] = j + e < k_dim ? z[e] * slope : 0.0f;
        }
        if (row_ok && j < below.ld) {
          if constexpr (BF16) {
            uint2 v;
            v.x = f32x2_to_bf16x2_rne(z[0], z[1]);
            v.y = f32x2_to_bf16x2_rne(z[2], z[3]);
            *reinterpret_cast<uint2*>(out + j) = v;
          } else {
            *reinterpret_cast<f32x4_t*>(out + j) = z;
          }
        }
      }
    }
  }
}

// Minibatch loss of each worker: mean of its row losses, rows summed in slot order.
__global__ void loss_mean_kernel(const float* __restrict__ row_loss, float* __restrict__ losses,
                                 int n_workers, int batch) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n_workers) return;
  float s = 0.0f;
  for (int b = 0; b < batch; ++b) s += row_loss[(size_t)g * batch + b];
  losses[g] = s / (float)batch;
}

hipError_t launch_gather(const GatherArgs& a, bool bf16, hipStream_t s) {
  dim3 grid(a.batch, a.workers);
  if (bf16) hipLaunchKernelGGL(gather_kernel<true>, grid, dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL(gather_kernel<false>, grid, dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

GatherArgs gather_args(const float* features, const int32_t* labels, void* xb, int32_t* yb, int32_t* idx,
                       int batch, int d0, int ld0, long rows, uint64_t seed, int64_t t, const int* order, int workers) {
  GatherArgs a;
  a.features = features; a.labels = labels; a.xb = xb; a.yb = yb; a.idx = idx;
  a.batch = batch; a.d0 = d0; a.ld0 = ld0; a.rows = rows; a.log2n = ilog2(rows);
  a.seed = seed; a.t = (uint64_t)t;
  a.order = order; a.workers = workers;
  a.once = 0;
  return a;
}

hipError_t launch_sample_indices(uint64_t seed, int n_workers, int batch, long rows, int64_t t_first,
                                 int n_steps, int32_t* out, hipStream_t s) {
  const size_t total = (size_t)n_steps * n_workers * batch;
  if (total == 0) return hipSuccess;
  size_t blocks = (total + kThreads - 1) / kThreads;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(sample_indices_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, s, out,
                     n_workers, batch, ilog2(rows), seed, (uint64_t)t_first, total);
  return hipGetLastError();
}

hipError_t launch_softmax_xent(const float* logits, int n_parts, long part_stride, const float* bias,
                               long bias_gs, const int32_t* yb, void* delta, float* row_loss,
                               int n_workers, int batch, int n_classes, int ldc, bool bf16,
                               const int* order, const GatherArgs* next, hipStream_t s) {
  if (n_parts != 1 && n_parts != 2 && n_parts != kMaxLogitSplits) return hipErrorInvalidValue;
  GatherArgs ga;
  memset(&ga, 0, sizeof(ga));
  if (next != nullptr) ga = *next;
  if (n_classes > 256 && n_classes <= 4 * kThreads && ldc <= 4 * kThreads) {   // one workgroup per row
    dim3 grid(batch + (next != nullptr ? next->batch : 0), n_workers);
    if (bf16)
      hipLaunchKernelGGL(softmax_xent_row_kernel<true>, grid, dim3(kThreads), 0, s, logits, n_parts, part_stride,
                         bias, bias_gs, yb, delta, row_loss, batch, n_classes, ldc, order, batch, ga);
    else
      hipLaunchKernelGGL(softmax_xent_row_kernel<false>, grid, dim3(kThreads), 0, s, logits, n_parts, part_stride,
                         bias, bias_gs, yb, delta, row_loss, batch, n_classes, ldc, order, batch, ga);
    return hipGetLastError();
  }
  const int head_blocks = (batch + kThreads / kWave - 1) / (kThreads / kWave);
  dim3 grid(head_blocks + (next != nullptr ? next->batch : 0), n_workers);
  if (bf16)
    hipLaunchKernelGGL(softmax_xent_kernel<true>, grid, dim3(kThreads), 0, s, logits, n_parts, part_stride,
                       bias, bias_gs, yb, delta, row_loss, batch, n_classes, ldc, order,
                       head_blocks, ga);
  else
    hipLaunchKernelGGL(softmax_xent_kernel<false>, grid, dim3(kThreads), 0, s, logits, n_parts, part_stride,
                       bias, bias_gs, yb, delta, row_loss, batch, n_classes, ldc, order,
                       head_blocks, ga);
  return hipGetLastError();
}

// A workgroup multiplies its 16 rows with all of W_L, in class tiles of 16 or 64: up to kHeadBytes of it in whole tiles the launch
// saved is worth more (bf16 with at most 16 classes, whose product has a split contraction to pay for as well: always).  By
// W_L's own bytes, 1024 x 17 in fp32 would be taken too and loses: 4 workers of 128-64-1024-17, 256 rows, 55.2 us per iteration
// with the product apart and 58.9 here, 16 workers, 64 rows, 51.8 and 55.6.
constexpr long kHeadBytes = 128 << 10;
bool softmax_narrow_applies(int n_classes, int ldc, int k_dim, bool bf16) {
  if (n_classes < 1 || n_classes > kHeadClasses || ldc > kHeadClasses || (ldc & 7) != 0) return false;
  return (bf16 && n_classes <= 16) || (long)k_dim * (ldc <= 16 ? 16 : 64) * (bf16 ? 2 : 4) <= kHeadBytes;
}

// A product of its own spreads D_{L-1} over the chip; in the head every workgroup of 16 rows walks all units, 256 at a time, and so
// the launch saved (1.3 to 2 us) is used up by their number, and sooner where more workgroups read W_L.  Per iteration, product apart
// and delta in the head; workgroups of the head in brackets.
//   bf16, 256-d-10: [32] 256 units 17.6 and 16.0 us, 512 18.0 and 17.5, 768 21.3 and 20.9; [128] 256 29.3 and 27.6, 448 31.0 and 30.0,
//   768 34.4 and 34.8; [256] 448 27.6 and 27.7, 768 32.5 and 33.8.  1024 units: [32] 21.9 and 22.3, [256] 37.3 and 41.1; 4096: [32] 31.7
//   and 45.2, [256] 97.4 and 116.6
//   bf16, 256-d-37: [32] 448 20.0 and 19.3, 576 20.8 and 21.1; [256] 256 25.8 and 25.1, 448 30.7 and 31.2, 700 36.4 and 37.4
//   bf16, 256-d-64: [32] 440 22.0 and 21.1, 512 21.8 and 22.1; [256] 280 28.6 and 28.4, 440 31.2 and 32.4; [512] 192 36.0 and 36.7
//   fp32, 128-64-d-10: [64] 640 37.5 and 37.0, 896 42.1 and 42.9; [128] 448 38.4 and 36.9, 640 46.0 and 46.8; [256] 448 48.5 and 47.5,
//   512 51.4 and 51.9; 2048 units: [64] 65.9 and 75.5
//   fp32, 128-64-256-37: [64] 33.2 and 31.6, [256] 45.8 and 45.8; 320 units [128] 39.9 and 42.2; 128-64-256-64: [64] 33.2 and 32.9, [256] 46.4
//   and 49.1; 128-64-64-64: [96] 32.6 and 33.6
bool softmax_narrow_delta_pays(int ldc, int k_dim, int head_blocks, bool bf16) {
  const bool few = head_blocks < 128, narrow = ldc <= 16;     // workgroups on less than half of the compute units
  const long w = (long)k_dim * ldc;
  if (bf16) return few ? k_dim <= (narrow ? 768 : 512) && w <= 28 << 10
                       : k_dim <= 448 && w <= 18 << 10 && (ldc < 64 || head_blocks <= 256);
  if (narrow) return k_dim <= (few ? 640 : 448);
  return k_dim <= 256 && (head_blocks <= 64 || (ldc < 64 && w <= 10 << 10));
}
int softmax_narrow_blocks(int n_workers, int batch) { return n_workers * ((batch + kHeadRows - 1) / kHeadRows); }

hipError_t launch_softmax_xent_narrow(const void* h, long h_gs, int ldh, int k_dim, const void* w,
                                      long w_gs, const float* bias, long bias_gs, const int32_t* yb,
                                      void* delta, float* row_loss, int n_workers, int batch, int n_classes,
                                      int ldc, bool bf16, const int* order, const GatherArgs* next,
                                      const HeadDelta* below, hipStream_t s) {
  if (!softmax_narrow_applies(n_classes, ldc, k_dim, bf16) || (ldh % 8) != 0) return hipErrorInvalidValue;
  HeadDelta hd;
  memset(&hd, 0, sizeof(hd));
  if (below != nullptr) hd = *below;
  const bool dx = below != nullptr;
  const int head_blocks = (batch + kHeadRows - 1) / kHeadRows;
  GatherArgs ga;
  memset(&ga, 0, sizeof(ga));
  if (next != nullptr) ga = *next;
  dim3 grid(head_blocks + (next != nullptr ? next->batch : 0), n_workers);
  auto of = [&](auto plain, auto delta) { return dx ? delta : plain; };
  auto kernel = bf16 ? (ldc <= 16 ? of(softmax_xent_narrow_kernel<true, 1, false>, softmax_xent_narrow_kernel<true, 1, true>)
                                  : of(softmax_xent_narrow_kernel<true, 4, false>, softmax_xent_narrow_kernel<true, 4, true>))
                     : (ldc <= 16 ? of(softmax_xent_narrow_kernel<false, 1, false>, softmax_xent_narrow_kernel<false, 1, true>)
                                  : of(softmax_xent_narrow_kernel<false, 4, false>, softmax_xent_narrow_kernel<false, 4, true>));
  hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s, h, h_gs, ldh, k_dim, w, w_gs, bias,
                     bias_gs, yb, delta, row_loss, batch, n_classes, ldc, order, head_blocks, ga, hd);
  return hipGetLastError();
}

hipError_t launch_loss_mean(const float* row_loss, float* losses, int n_workers, int batch,
                            hipStream_t s) {
  hipLaunchKernelGGL(loss_mean_kernel, dim3((n_workers + 63) / 64), dim3(64), 0, s, row_loss, losses,
                     n_workers, batch);
  return hipGetLastError();
}

}  // namespace prsgd
