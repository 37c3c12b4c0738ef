// Backward step of the FIRST layer fused with the forward product of the NEXT iteration.
//
// Layer 1 has no delta to pass down, and it is the last kernel of an iteration's backward pass; the
// first kernel of the next iteration's forward pass reads exactly the weights it has just written,
//   H_1^{t+1} = phi(X^{t+1} bf16(W_1^{t}) + b_1^{t}),
// and the minibatch X^{t+1} is already there (zeta_i^{t+1} is drawn during iteration t; it depends
// on nothing iteration t computes).  So the pass over the fp32 master that applies eq. (3),
//   dW_1 = X^{t T} D_1,  db_1 = colsum(D_1),  W_1 <- W_1 - gamma dW_1,  b_1 <- b_1 - gamma db_1,
// also feeds the updated tile, rounded to bf16 in registers (the shadow's value), to the matrix cores
// for the next forward product: W_1 crosses HBM once per iteration instead of twice (the stand-alone
// forward launch and its read of the bf16 shadow are gone).
//
// For the contraction of X^{t+1} W_1 over the rows k of W_1 to stay inside one workgroup, the walk is
// transposed against the other layers' kernel: a workgroup owns a band of NB columns n of W_1 of one
// replica and walks down all rows in tiles of 64.  The B x NB accumulators of the next pre-activation
// and the matrix fragments of D_1[:, n-band] stay in registers; X^t[:, k-tile] and X^{t+1}[:, k-tile] (both
// L2-resident) are requested straight into LDS.  A wavefront owns a 32 x 32 block of every weight tile:
// it multiplies the block's gradient, turns it through a piece of LDS of its own into the row-major
// layout of the 16-byte weight loads, updates, stores, and leaves the new block as bf16 for the next
// product.  Tile i's gradient and tile i - 1's share of the next pre-activation are independent, so
// they run in the same phase, and a tile costs ONE workgroup barrier.  Requests go out at the start
// of a phase, X one tile and W_1 two tiles ahead: the memory pipe returns in order, so that the wait
// for an X tile also covers the weights requested before it, which have had two phases by then.
// What bounds it: the weight stream (8 B per element), and per compute unit the X tiles beside it --
// 128 columns per workgroup of eight wavefronts where that still gives every compute unit one (B = 128:
// 96 instead of 128 KB pass through the unit per 32 KB of weights), 64 columns and four otherwise.
// Measured against five barriers per tile and X tiles through registers: 8 x (4096 x 4096), 128 rows 242 ->
// 208 us (5.2 TB/s of weight bytes); 16 x (3072 x 1024), 64 rows 85 -> 76 us (5.3 TB/s).
//
// Every output block accumulates over k in the order of the stand-alone forward product.  Layers of whole tiles (bwd_first_fwd_shape)
// sum the bias as the other layers' whole-tile kernel does, so H_1^{t+1} and the parameters have the bits the two separate launches
// give.  From 512 rows of W_1 on any minibatch and any rows are taken too, with columns that the layout pads to whole tiles; apart, such
// layers run in kernels that sum the bias in another order, and the two forms agree up to its rounding (asserted: 1e-3 of the points after
// seven steps).  5 workers of 4005-2688-100, 64 rows, 177 -> 104 us per iteration, 12 of 3001-1472-333-20 208 -> 146; with momentum
// 282 -> 179 and 316 -> 257.
#include <atomic>
#include <type_traits>

#include "prsgd_internal.h"

namespace prsgd {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

namespace {

constexpr int BT = 64;              // weight rows per step
constexpr int ST = 36;              // LDS row stride of a wavefront's 32 x 32 transposition piece (floats)

__device__ __forceinline__ f32x16_t mfma_bf16(bf16x8_t a, bf16x8_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float act_from_z(float z, int act) {
  return act == PRSGD_TANH ? tanhf(z) : fmaxf(z, 0.0f);
}

// LDS of a workgroup: two X^t tiles, three X^{t+1} tiles, two new weight tiles, the wavefronts'
// transposition pieces, partial column sums and the new bias.  The D_1 band passes through the X^{t+1}
// tiles before the walk.
constexpr size_t first_lds_bytes(int mb, int nb) {
  const size_t x_tile = 32 * (size_t)mb * 128, waves = (size_t)nb / 16;
  return 5 * x_tile + 2 * (size_t)BT * nb * 2 + waves * 32 * ST * 4 + 5 * (size_t)nb * 4;
}

// MB: 32-row tiles of the minibatch (B = 32 MB).  NB: band width, 64 or 128.  NT: non-temporal weight
// traffic.  MOM: momentum form of the local update, v <- mu v + G, x <- x - gamma v, with the velocity
// tile streamed beside the weights.  The bf16 shadow of W_1 is left as it is: only the stand-alone forward
// product reads it, and the caller refreshes it when the chain of activations from here breaks.
// RAG: any number of rows of W_1 (p.Nn: its columns with the padding, whole bands) and of the minibatch.  Weights are read and written
// with range-checked accesses, so that a row past the last one reads as zeros and is written nowhere, and every phase issues as
// many accesses as the waits count.
template <int MB, int NB, bool NT, bool MOM, bool RAG>
__global__ __launch_bounds__(4 * NB, MOM ? 1 : 2) void bwd_first_fwd_kernel(BwdArgs p) {
  fetch_kernel_args<sizeof(BwdArgs)>();
  constexpr int BR = 32 * MB;
  constexpr int NW = NB / 16, NTHR = 64 * NW;         // wavefronts: 2 (rows) x NB / 32 (columns)
  constexpr int NBLK = MB * (NB / 32);                // next-activation blocks (32 x 32)
  constexpr int NZ = (NBLK + NW - 1) / NW;            // ... per wavefront
  constexpr int XT = BR * 128;                        // bytes of an X tile [BR][64]
  constexpr int WT = BT * NB * 2;                     // bytes of a new weight tile [BT][NB]
  constexpr int REQ = (XT / 1024 + NW - 1) / NW;      // requests per wavefront and X tile

  const int bands = p.Nn / NB;
  int g, band;
  if ((p.n_groups & 7) == 0) {                        // all bands of a replica on one XCD
    const int slot = blockIdx.x >> 3;
    g = (blockIdx.x & 7) + 8 * (slot / bands);
    band = slot % bands;
  } else {
    g = blockIdx.x / bands;
    band = blockIdx.x % bands;
  }
  g = worker_of(p.order, g);
  const int n0 = band * NB;

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  unsigned char* const Hk = smem;                                        // [2][BR][64]  X^t tiles
  unsigned char* const Xk = Hk + 2 * XT;                                 // [3][BR][64]  X^{t+1} tiles
  unsigned char* const Wl = Xk + 3 * XT;                                 // [2][BT][NB]  new W tiles, bf16
  float* const Tl = reinterpret_cast<float*>(Wl + 2 * WT);               // [NW][32][ST]
  float* const Bs = Tl + NW * 32 * ST;                                   // [4][NB] partial column sums
  float* const Bn = Bs + 4 * NB;                                         // [NB]    new bias of the band
  uint16_t* const Dn = reinterpret_cast<uint16_t*>(Xk);                  // [BR][NB] D_1 band, before the walk
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr32 = lane & 31, kb = lane >> 5;
  const int wk = wave & 1, wn = wave >> 1;            // this wavefront's block of the weight tile

  const uint16_t* h_g = p.h + (size_t)g * p.h_gs;               // X^t      [B][ldh]
  const uint16_t* x_g = p.x_next + (size_t)g * p.x_gs;          // X^{t+1}  [B][ldx]
  const uint16_t* d_g = p.d + (size_t)g * p.d_gs;               // D_1      [B][ldd]
  const bool nt_read = NT && p.src_gs != 0;           // a shared source is re-read by every replica

  // the wavefront's block of a weight tile, row-major: vector q at row 8 q + lane / 8, column 4 (lane % 8)
  const int trow = lane >> 3, tcol = 4 * (lane & 7);
  const size_t w_first = (size_t)p.w_off + (size_t)(wk * 32 + trow) * p.ldw + n0 + wn * 32 + tcol;
  float* const w_g = p.params + (size_t)g * p.p_gs + w_first;
  const float* const wsrc_g = p.src + (size_t)g * p.src_gs + w_first;
  float* const v_g = MOM ? p.vel + (size_t)g * p.p_gs + w_first : nullptr;
  const size_t row8 = (size_t)8 * p.ldw;
  constexpr int kStream = NT ? 2 : 0;                 // buffer access cache policy: the nt bit
  const uint32_t lane_first = 4u * ((uint32_t)(wk * 32 + trow) * (uint32_t)p.ldw + (uint32_t)(n0 + wn * 32 + tcol));
  auto rsrc = [&](const float* base, size_t first) __attribute__((always_inline)) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base + first), 0, (int)((uint32_t)p.K * (uint32_t)p.ldw * 4u), 0x00020000);
  };
  auto at = [&](int it, int q) __attribute__((always_inline)) {
    return (int)(lane_first + 4u * (uint32_t)(it * BT + 8 * q) * (uint32_t)p.ldw);
  };
  const __amdgpu_buffer_rsrc_t w_src = rsrc(p.src, (size_t)g * p.src_gs + p.w_off);
  const __amdgpu_buffer_rsrc_t w_dst = rsrc(p.params, (size_t)g * p.p_gs + p.w_off);
  const __amdgpu_buffer_rsrc_t v_all = rsrc(MOM ? p.vel : p.params, (size_t)g * p.p_gs + p.w_off);
  auto fetch = [&](f32x4_t (&reg)[4], const float* base, const __amdgpu_buffer_rsrc_t& all, int it, bool stream) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if constexpr (RAG) {
        reg[q] = __builtin_bit_cast(f32x4_t, stream ? __builtin_amdgcn_raw_buffer_load_b128(all, at(it, q), 0, 2)
                                                    : __builtin_amdgcn_raw_buffer_load_b128(all, at(it, q), 0, 0));
        continue;
      }
      const f32x4_t* src = reinterpret_cast<const f32x4_t*>(base + (size_t)it * BT * p.ldw + q * row8);
      reg[q] = stream ? __builtin_nontemporal_load(src) : *src;
    }
  };

  // requests of an X tile: this lane's chunk of piece q * NW + wave (8 rows of 128 bytes)
  uint32_t h_off[REQ], x_off[REQ];
  auto offsets = [&](uint32_t (&h_o)[REQ], uint32_t (&x_o)[REQ], int cols) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < REQ; ++q) {
      const int r = (q * NW + wave) * 8 + (lane >> 3), pos = lane & 7;
      const int row = RAG ? min(r, p.B - 1) : r < BR ? r : BR - 1;
      int hc = ((((pos >> 2) ^ lds_seg_xor<128>(r)) << 2) | (pos & 3)) * 8, xc = lds_chunk(r, pos) * 8;
      if (RAG) { hc = min(hc, (cols - 1) & ~7); xc = min(xc, (cols - 1) & ~7); }
      h_o[q] = (uint32_t)(((size_t)row * p.ldh + hc) * 2);
      x_o[q] = (uint32_t)(((size_t)row * p.ldx + xc) * 2);
    }
  };
  offsets(h_off, x_off, BT);
  const int n_t = RAG ? (p.K + BT - 1) / BT : p.K / BT;          // steps of the walk down the rows (at least 4)
  const int tail = RAG ? p.K - (n_t - 1) * BT : BT;              // rows of the last one
  auto request_x = [&](int it, int hbuf, int xbuf) __attribute__((always_inline)) {
    if (RAG && it == n_t - 1 && tail < BT) offsets(h_off, x_off, tail);        // copies of the last columns past them
#pragma unroll
    for (int q = 0; q < REQ; ++q) {
      if ((q * NW + wave) * 1024 < XT) {                                 // uniform over the wavefront
        load_to_lds(h_g + it * BT, h_off[q], lds0 + hbuf * XT + (q * NW + wave) * 1024);
        load_to_lds(x_g + it * BT, x_off[q], lds0 + (2 + xbuf) * XT + (q * NW + wave) * 1024);
      }
    }
  };

  f32x4_t wr[3][4];
  f32x4_t vr[MOM ? 3 : 1][4];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    fetch(wr[j], wsrc_g, w_src, j, nt_read);
    if (MOM) fetch(vr[j], v_g, v_all, j, NT);
  }

  // the D_1 band: through LDS for the column sums and into fragments
  for (int e = tid; e < BR * (NB / 8); e += NTHR) {
    const int b = e / (NB / 8), c = e % (NB / 8);
    *reinterpret_cast<u32x4_t*>(reinterpret_cast<unsigned char*>(Dn) + b * (NB * 2) +
                                ((((c >> 2) ^ lds_seg_xor<NB * 2>(b)) << 6) | ((c & 3) << 4))) =
        RAG && b >= p.B ? (u32x4_t){0u, 0u, 0u, 0u} : *reinterpret_cast<const u32x4_t*>(d_g + (size_t)b * p.ldd + n0 + 8 * c);
  }
  __syncthreads();
  bf16x8_t df[BR / 16];
#pragma unroll
  for (int kk = 0; kk < BR / 16; ++kk)
    df[kk] = lds_frag_trans<NB * 2>(reinterpret_cast<const unsigned char*>(Dn), wn, kk, lane);
  // b_1 <- b_1 - gamma db_1: four quarter sums over the minibatch rows, added in order
  {
    const int n = tid % NB, quarter = tid / NB;                          // NTHR = 4 NB
    float cs = 0.0f;
#pragma unroll 8
    for (int b = quarter * (BR / 4); b < (quarter + 1) * (BR / 4); ++b)
      cs += bf16_to_f32(Dn[b * NB + (((n >> 5) ^ lds_seg_xor<NB * 2>(b)) << 5) + (n & 31)]);
    Bs[quarter * NB + n] = cs;
  }
  __syncthreads();                                    // the band's place is free for the X tiles
  request_x(0, 0, 0);
  if (tid < NB) {
    float cs = ((Bs[tid] + Bs[NB + tid]) + Bs[2 * NB + tid]) + Bs[3 * NB + tid];
    const size_t bo = p.b_off + (size_t)n0 + tid;
    if (MOM) {
      float* vb = p.vel + (size_t)g * p.p_gs + bo;
      cs = fmaf(p.mu, *vb, cs);
      *vb = cs;
    }
    const float b_new = fmaf(-p.lr, cs, p.src[(size_t)g * p.src_gs + bo]);
    p.params[(size_t)g * p.p_gs + bo] = b_new;
    Bn[tid] = b_new;
  }

  f32x16_t acc_z[NZ];
#pragma unroll
  for (int t = 0; t < NZ; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc_z[t][v] = 0.0f;
  float* const T = Tl + wave * 32 * ST;

  // next pre-activation [b][n] += X^{t+1}[:, k-tile] bf16(W_new tile): contraction over the tile's rows
  // (past `rows` of them zeros; the new weights of such rows are zeros as well)
  auto next_product = [&](int wbuf, int xbuf, int rows) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NZ; ++t) {
      const int blk = wave + NW * t;
      if (NBLK % NW == 0 || blk < NBLK) {
        const int mb = blk / (NB / 32), nblk = blk % (NB / 32);
#pragma unroll
        for (int kk = 0; kk < BT / 16; ++kk) {
          bf16x8_t xf = lds_frag_contig(Xk + xbuf * XT, mb, kk, lane);
          if (RAG && rows < BT) {
            u32x4_t u = __builtin_bit_cast(u32x4_t, xf);
            const int c = 16 * kk + 8 * kb;
#pragma unroll
            for (int e = 0; e < 4; ++e)
              u[e] &= (c + 2 * e < rows ? 0xFFFFu : 0u) | (c + 2 * e + 1 < rows ? 0xFFFF0000u : 0u);
            xf = __builtin_bit_cast(bf16x8_t, u);
          }
          acc_z[t] = mfma_bf16(xf, lds_frag_trans<NB * 2>(Wl + wbuf * WT, nblk, kk, lane), acc_z[t]);
        }
      }
    }
  };

  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  int hbuf = 0, xbuf = 0;                             // buffers of tile it (its new weights: Wl[hbuf])
  // Phase of tile it (weights in register set SLOT).  FIRST: no previous tile.  The requests past the
  // last tile repeat it and are not used.
  auto phase = [&](int it, auto slot_tag, auto first_tag) __attribute__((always_inline)) {
    constexpr int SLOT = decltype(slot_tag)::value, AHEAD = (SLOT + 2) % 3;
    constexpr bool FIRST = decltype(first_tag)::value;
    const int xprev = xbuf == 0 ? 2 : xbuf - 1, xnext = xbuf == 2 ? 0 : xbuf + 1;
    request_x(min(it + 1, n_t - 1), hbuf ^ 1, xnext);
    const int ahead = min(it + 2, n_t - 1);
    fetch(wr[AHEAD], wsrc_g, w_src, ahead, nt_read);
    if (MOM) fetch(vr[AHEAD], v_g, v_all, ahead, NT);
    // gradient block: contraction over the minibatch
    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll
    for (int kk = 0; kk < BR / 16; ++kk) acc = mfma_bf16(lds_frag_trans<128>(Hk + hbuf * XT, wk, kk, lane), df[kk], acc);
    if (!FIRST) next_product(hbuf ^ 1, xprev, BT);
    // accumulator element v of lane (lr32, kb) is C[8 (v/4) + 4 kb + v%4][lr32]
#pragma unroll
    for (int v = 0; v < 16; ++v) T[(8 * (v / 4) + 4 * kb + (v % 4)) * ST + lr32] = acc[v];
    __builtin_amdgcn_wave_barrier();                  // the piece is this wavefront's own
    f32x4_t grad[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) grad[q] = *reinterpret_cast<const f32x4_t*>(T + (8 * q + trow) * ST + tcol);
    // eq. (3) on the block, in the layout of the weight loads; the new block also goes to LDS as bf16
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4_t gr = grad[q];
      const size_t off = (size_t)it * BT * p.ldw + q * row8;
      if (MOM) {
        gr.x = fmaf(p.mu, vr[SLOT][q].x, gr.x);
        gr.y = fmaf(p.mu, vr[SLOT][q].y, gr.y);
        gr.z = fmaf(p.mu, vr[SLOT][q].z, gr.z);
        gr.w = fmaf(p.mu, vr[SLOT][q].w, gr.w);
        if (RAG) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, gr), v_all, at(it, q), 0, kStream);
        else if (NT) __builtin_nontemporal_store(gr, reinterpret_cast<f32x4_t*>(v_g + off));
        else *reinterpret_cast<f32x4_t*>(v_g + off) = gr;
      }
      f32x4_t w = wr[SLOT][q];
      w.x = fmaf(-p.lr, gr.x, w.x);
      w.y = fmaf(-p.lr, gr.y, w.y);
      w.z = fmaf(-p.lr, gr.z, w.z);
      w.w = fmaf(-p.lr, gr.w, w.w);
      u32x2_t hv2 = {f32x2_to_bf16x2_rne(w.x, w.y),
                     f32x2_to_bf16x2_rne(w.z, w.w)};
      if (RAG) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, w), w_dst, at(it, q), 0, kStream);
        if (it * BT + wk * 32 + 8 * q + trow >= p.K) hv2 = (u32x2_t){0u, 0u};
      } else if (NT) {
        __builtin_nontemporal_store(w, reinterpret_cast<f32x4_t*>(w_g + off));
      } else {
        *reinterpret_cast<f32x4_t*>(w_g + off) = w;
      }
      const int k = wk * 32 + 8 * q + trow;
      *reinterpret_cast<u32x2_t*>(Wl + hbuf * WT + k * (NB * 2) + ((wn ^ lds_seg_xor<NB * 2>(k)) << 6) + 2 * tcol) = hv2;
    }
    // The next X tile has landed (younger than its requests: this phase's weight loads and stores), the
    // new weights are in LDS, and nobody reads this phase's tiles any more.
    constexpr int YOUNGER = MOM ? 16 : 8;
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(YOUNGER) : "memory");
    hbuf ^= 1;
    xbuf = xnext;
  };

  const std::integral_constant<int, 0> set0{};
  const std::integral_constant<int, 1> set1{};
  const std::integral_constant<int, 2> set2{};
  phase(0, set0, std::true_type{});
  for (int it = 1;;) {
    phase(it, set1, std::false_type{});
    if (++it == n_t) break;
    phase(it, set2, std::false_type{});
    if (++it == n_t) break;
    phase(it, set0, std::false_type{});
    if (++it == n_t) break;
  }
  next_product(hbuf ^ 1, xbuf == 0 ? 2 : xbuf - 1, tail);        // the last tile's share
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // no request into LDS outlives the workgroup

  // ---- H_1^{t+1} = phi(Z + b_1) for this band ------------------------------------------------------
  uint16_t* hn_g = p.h_next + (size_t)g * p.hn_gs;
#pragma unroll
  for (int t = 0; t < NZ; ++t) {
    const int blk = wave + NW * t;
    if (NBLK % NW == 0 || blk < NBLK) {
      const int mb = blk / (NB / 32), nblk = blk % (NB / 32);
      const int n = nblk * 32 + lr32;
      const float bn = Bn[n];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int b = mb * 32 + 8 * (v / 4) + 4 * kb + (v % 4);
        if (!RAG || b < p.B) hn_g[(size_t)b * p.ldhn + n0 + n] = f32_to_bf16_rne(act_from_z(acc_z[t][v] + bn, p.act));
      }
    }
  }
}

template <int MB, int NB, bool NT, bool MOM, bool RAG>
hipError_t launch_first_one(const BwdArgs& p, hipStream_t s) {
  constexpr size_t kLds = first_lds_bytes(MB, NB);
  static_assert(kLds <= 160 * 1024, "LDS of a compute unit");
  auto kernel = bwd_first_fwd_kernel<MB, NB, NT, MOM, RAG>;
  static std::atomic<bool> configured{false};
  if (!configured.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
    if (e != hipSuccess) return e;
    configured.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL(kernel, dim3((unsigned)(p.Nn / NB * p.n_groups)), dim3(4 * NB), kLds, s, p);
  return hipGetLastError();
}

template <int MB, int NB, bool NT, bool RAG>
hipError_t launch_first_nt(const BwdArgs& p, hipStream_t s) {
  if constexpr (NB == 64) {
    if (p.vel != nullptr) return launch_first_one<MB, NB, NT, true, RAG>(p, s);
  }
  return launch_first_one<MB, NB, NT, false, RAG>(p, s);
}

// 128-column bands where they still give every compute unit a workgroup; not with momentum, whose second
// stream of tiles does not fit the registers of eight wavefronts.
template <int MB, bool RAG> hipError_t launch_first_mb(const BwdArgs& p, hipStream_t s) {
  const bool wide = p.vel == nullptr && (p.Nn % 128) == 0 && (long)(p.Nn / 128) * p.n_groups >= 256;
  if (wide) return p.streaming ? launch_first_nt<MB, 128, true, RAG>(p, s) : launch_first_nt<MB, 128, false, RAG>(p, s);
  return p.streaming ? launch_first_nt<MB, 64, true, RAG>(p, s) : launch_first_nt<MB, 64, false, RAG>(p, s);
}
template <bool RAG> hipError_t launch_first_rag(const BwdArgs& p, hipStream_t s) {
  if (p.B <= 32) return launch_first_mb<1, RAG>(p, s);
  if (p.B <= 64) return launch_first_mb<2, RAG>(p, s);
  return launch_first_mb<4, RAG>(p, s);
}

}  // namespace

// Layer shapes made of whole tiles, whose two forms have the same bits.  An odd number of column tiles is nothing that the other layers'
// whole-tile kernel takes: such a layer counts as ragged, unless it is so short that it is fused in any case.
static bool bwd_first_fwd_shape(int batch, int d_in, int d_out) {
  return (batch == 32 || batch == 64 || batch == 128) && d_in >= 4 * BT && (d_in % (2 * BT)) == 0 &&
         d_out >= BT && (d_out % BT) == 0 && (d_in <= 8 * BT || (d_out / BT) % 2 == 0);
}

// A band walks its d_0 / 64 row tiles one after the other, at 0.8 us each behind the two launches that it replaces (0.4 us more than
// their own share of a tile with up to 64 minibatch rows, 0.9 with 128), while those spread the layer over the chip; their backward
// pass walks d_1 / 64 column tiles at 0.75 us.  So a tall layer is taken apart until its bands are so many that its bytes count.
// Per iteration, fused less apart, bands in brackets: 64 rows, 2560 x 256 [8] +13 us, [64] +8.6; 4096 x 1024 [32] +19.1, [64] +4.6, [80]
// -2.8, [128] -19.2; 2048 x 1024 [16] +3.2, [80] -3.1; 1536 x 1024 [16] -2.0; 768 x 2048 [32] -16; 512 x 256 [4] -1.4.  128 rows:
// 2560 x 1024 [16] +21, [96] +7.9, [128] -1.6; 1280 x 1024 [16] +4.1, [128] -1.9.  (4 workers of 2560-256-40, 64 rows: 41.8 and 27.7 us.)
// With momentum 4096 x 2048 [64] 32 rows -26, 64 rows -5; 128 rows, 2048 x 1024 [64] +12.8, [80] -0.2, [96] -3.6.  Up to eight row tiles
// there is next to nothing in it.
// Ragged layers apart are products that spread over the chip however few the bands (kernels_bwd.hip).  32 rows: 2001 x 1100 [54] +7.3, [90]
// -3.5, 700 x 1300 [105] +0.2, [168] -5.6; 64 rows: 2001 x 1100 [90] +0.9, [144] -9.3,
// 3001 x 1472 [115] -9.0, 1000 x 555 [108] +4.2; 128 rows: 2001 x 1100 [144] +1.6, [216] -23.2, 4005 x 2688 [126] +15.9, [210] -84 (208
// apart).  With momentum 32 rows: 2001 x 1100 [90] -1.0, [144] -10.8, 4005 x 600 [120] -1.3; 64 rows: 3001 x 1472 [115] -1.5, 4005 x 2688
// [126] +2.3, 2001 x 1100 [144] -13.9; 128 rows: 4005 x 600 [120] +40, 4005 x 2688 [126] +18.6, 2001 x 1100 [144] -11.2.
static bool bwd_first_fwd_pays(const BwdArgs& p, bool ragged) {
  const int rows = (p.K + BT - 1) / BT, cols = p.Nn / BT;
  const long bands = (long)cols * p.n_groups;
  if (ragged && p.vel == nullptr) return bands >= (p.B <= 32 ? 96 : p.B <= 64 ? 112 : 152);
  if (ragged) return bands >= (p.B <= 32 ? 100 : p.B <= 64 ? 132 : 144);
  if (rows <= 8) return true;
  if (bands >= (p.vel != nullptr ? (p.B <= 64 ? 64 : 96) : p.B <= 64 ? 80 : 128)) return true;
  return p.B <= 64 ? 5 * rows <= 8 * cols + 20 : 20 * rows <= 17 * cols + 60;
}

// The layer as the kernel walks it: over its padded columns where those are whole tiles (zeros, whose gradient is zero).
static BwdArgs bwd_first_padded(const BwdArgs& p) {
  BwdArgs q = p;
  if ((p.Nn % BT) != 0 && (p.ldw % BT) == 0 && p.ldw - p.Nn < BT) q.Nn = p.ldw;
  return q;
}
static bool bwd_first_ragged_shape(const BwdArgs& p) {
  return p.B >= 1 && p.B <= 128 && p.K >= 512 && p.Nn >= BT && (p.Nn % BT) == 0 && p.ldd >= p.Nn && p.ldhn >= p.Nn &&
         (size_t)(p.K + BT) * p.ldw * 4 < ((size_t)1 << 32);
}

bool bwd_first_fwd_same_bits(const BwdArgs& p) { return bwd_first_fwd_shape(p.B, p.K, p.Nn) && bwd_first_fwd_pays(p, false); }

// Whole tiles or such columns, and the buffers of the next iteration given.
bool bwd_first_fwd_applies(const BwdArgs& p_in) {
  const BwdArgs p = bwd_first_padded(p_in);
  const bool whole = bwd_first_fwd_shape(p_in.B, p_in.K, p_in.Nn);
  if ((!whole && !bwd_first_ragged_shape(p)) || !bwd_first_fwd_pays(p, !whole)) return false;
  if (p.dx != nullptr) return false;
  if (p.x_next == nullptr || p.h_next == nullptr) return false;
  return (p.ldw % 4) == 0 && (p.ldh % 8) == 0 && (p.ldx % 8) == 0 && (p.ldd % 8) == 0 && (p.w_off % 4) == 0;
}

hipError_t launch_bwd_first_fwd(const BwdArgs& p, hipStream_t s) {
  if (!bwd_first_fwd_applies(p) || p.n_groups <= 0) return hipErrorInvalidValue;
  const BwdArgs q = bwd_first_padded(p);
  return bwd_first_fwd_shape(q.B, q.K, q.Nn) ? launch_first_rag<false>(q, s) : launch_first_rag<true>(q, s);
}

}  // namespace prsgd
