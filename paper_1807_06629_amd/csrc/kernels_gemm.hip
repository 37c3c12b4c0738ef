// Grouped (replica-batched) matrix products of the per-worker MLP gradient
//   G_i^t = grad F_i(x_i^{t-1}; zeta_i^t)            (Algorithm 1, gradient observation)
// on the CDNA4 matrix cores.  One group = one worker's replica: no weights are shared between
// groups, and every group multiplies a skinny B-row activation block with its own weights.
//
//   forward   H_l    = phi(H_{l-1} W_l + b_l)              M = B,       N = d_l,     Kc = d_{l-1}
//   backward  D_{l-1} = (D_l W_l^T) * phi'(H_{l-1})        M = B,       N = d_{l-1}, Kc = d_l
//   weights   dW_l   = H_{l-1}^T D_l ; db_l = colsum(D_l)  M = d_{l-1}, N = d_l,     Kc = B
//             fused with the local update  W_l <- W_l - gamma dW_l      (Algorithm 1, eq. 3)
// With I = 1 all workers share the node average: the same products then run with one weight stream
// (group stride 0) and the weight-gradient product contracts over the stacked minibatches of all
// workers, M = d_{l-1}, N = d_l, Kc = N B, updating the average in place.
//
// Operand tiles go from memory to LDS without passing through registers: every wavefront requests
// 1024-byte pieces (64 lanes x 16 bytes) that land at consecutive LDS addresses, S tiles deep, and
// the wait for a tile leaves the requests of the following tiles in flight.  A piece cannot be padded
// on its way, so bank conflicts are avoided by permuting WHICH 16 bytes a lane requests (below).  A
// tile is 128 bytes deep along the contraction (64 bf16 or 32 fp32 elements); an operand whose
// contraction index is the strided one is transposed while its MFMA fragments are read out of LDS.
// (Tiles, fragments, placement and epilogue: gemm_tile.h.  kernels_gemm_rows.hip has the workgroups with requesting wavefronts.)
// The wavefronts of a workgroup are a WM x WN grid over the output tile times WK shares of the
// contraction: larger blocks per wavefront read fewer LDS bytes per matrix instruction (the bound of
// the large bf16 products), and a small output tile still occupies several matrix cores (the bound of
// the small fp32 products, whose instructions are 8 times as slow).  The shares are added in order
// when the output tile leaves through LDS.
#include <string.h>

#include "gemm_tile.h"

namespace prsgd {

// One output tile of product p: workgroup `block` of the product's.  MOM: momentum form of the update, v <- mu v + G, W <- W - gamma v.
template <typename T, int BM, int BN, int WM, int WN, int WK, int S, int AKIND, int BKIND, bool MOM>
__device__ __forceinline__ void gemm_tile(const GemmArgs& p, int block) {
  using E = typename T::elem;
  constexpr int NWAVE = WM * WN * WK, NTHR = 64 * NWAVE;
  using IOA = TileIO<T, BM, AKIND, NWAVE>;
  using IOB = TileIO<T, BN, BKIND, NWAVE>;
  constexpr int BK = IOA::BK;
  constexpr int TM = BM / (32 * WM), TN = BN / (32 * WN);
  constexpr int PER = IOA::NPT + IOB::NPT;
  static_assert(TM >= 1 && TN >= 1, "tile too small for the wavefront grid");
  static_assert(kSlices % WK == 0, "the slices of a tile must split evenly over the shares");
  static_assert(S >= 2 && S <= 4 && PER * (S - 1) <= 63, "wait_tiles");

  fetch_args(p);
  const TileAt at = tile_at<BM, BN>(p, block);
  const int g = at.g, m0 = at.m0, n0 = at.n0, ks = at.split, n_splits = at.n_splits;

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  constexpr int STAGE = (BM + BN) * kTileBytes;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave / (WM * WN), wm = (wave / WN) % WM, wn = wave % WN;
  const int lr32 = lane & 31, kb = lane >> 5;

  int Kc, k_lo;
  contraction_range<BK>(p, at, &k_lo, &Kc);
  const E* a_src = reinterpret_cast<const E*>(p.a) + (size_t)g * p.a_gs +
                   (AKIND == OP_CONTIG ? (size_t)m0 * p.lda + k_lo : (size_t)k_lo * p.lda + m0);
  const E* b_src = reinterpret_cast<const E*>(p.b) + (size_t)g * p.b_gs +
                   (BKIND == OP_CONTIG ? (size_t)n0 * p.ldb + k_lo : (size_t)k_lo * p.ldb + n0);
  const size_t a_step = AKIND == OP_CONTIG ? (size_t)BK : (size_t)BK * p.lda;
  const size_t b_step = BKIND == OP_CONTIG ? (size_t)BK : (size_t)BK * p.ldb;
  const size_t pg = (size_t)g * p.p_gs;
  constexpr bool kIsDw = (AKIND == OP_TRANS && BKIND == OP_TRANS);   // weight-gradient product
  const bool fused = kIsDw && (p.epi == EPI_DW_FUSED);

  const int n_k = (Kc + BK - 1) / BK;
  const int k_tail = Kc - (n_k - 1) * BK;                  // elements of the last tile
  uint32_t a_off[IOA::NPT], b_off[IOB::NPT];
  IOA::template offsets<false>(a_off, p.lda, p.M - m0, BK, wave, lane);
  IOB::template offsets<false>(b_off, p.ldb, p.N - n0, BK, wave, lane);
  auto request = [&](int j, int stage) __attribute__((always_inline)) {
    const uint32_t lds_a = lds0 + (uint32_t)stage * STAGE, lds_b = lds_a + BM * kTileBytes;
    if (j == n_k - 1 && k_tail < BK) {                     // nothing past the operands is touched
      uint32_t a_o[IOA::NPT], b_o[IOB::NPT];
      IOA::template offsets<true>(a_o, p.lda, p.M - m0, k_tail, wave, lane);
      IOB::template offsets<true>(b_o, p.ldb, p.N - n0, k_tail, wave, lane);
      IOA::request(a_src + (size_t)j * a_step, a_o, lds_a, wave);
      IOB::request(b_src + (size_t)j * b_step, b_o, lds_b, wave, !kIsDw && p.b_once);
    } else {
      IOA::request(a_src + (size_t)j * a_step, a_off, lds_a, wave);
      IOB::request(b_src + (size_t)j * b_step, b_off, lds_b, wave, !kIsDw && p.b_once);
    }
  };

  // Weight-update epilogue: the output tile leaves through LDS in row-major order, one 16-byte
  // vector per lane (EV vectors per thread).  The old weights are requested in that layout before
  // the products.
  constexpr int SC = BN + 4;                               // LDS row stride of the output tile (floats)
  constexpr int VPR_C = BN / 4, ROWS_PER_PASS = NTHR / VPR_C, EV = kIsDw ? BM / ROWS_PER_PASS : 1;
  static_assert(!kIsDw || (NTHR % VPR_C == 0 && BM % ROWS_PER_PASS == 0), "output tile must split evenly");
  const int e_row = tid / VPR_C, e_col = 4 * (tid % VPR_C);
  f32x4_t w_old[EV], v_old[MOM ? EV : 1];
  if constexpr (kIsDw) if (fused) {
    const float* wtile = p.src + (size_t)g * p.src_gs + p.w_off + (size_t)m0 * p.ldw + n0;
    const bool nt_read = p.streaming && (p.src_gs != 0 || p.p_gs == 0);          // a source that several groups share is read again
#pragma unroll
    for (int q = 0; q < EV; ++q) {
      const int r = q * ROWS_PER_PASS + e_row;
      const bool ok = m0 + r < p.M && n0 + e_col < p.N;
      const f32x4_t* wp = reinterpret_cast<const f32x4_t*>(
          wtile + (ok ? __umul24((uint32_t)r, (uint32_t)p.ldw) + (uint32_t)e_col : 0u));
      w_old[q] = nt_read ? __builtin_nontemporal_load(wp) : *wp;
      if constexpr (MOM) {
        const f32x4_t* vp = reinterpret_cast<const f32x4_t*>(p.vel + pg + p.w_off + (size_t)m0 * p.ldw + n0 +
                                                             (ok ? __umul24((uint32_t)r, (uint32_t)p.ldw) + (uint32_t)e_col : 0u));
        v_old[q] = p.streaming ? __builtin_nontemporal_load(vp) : *vp;
      }
    }
  }

  // ... and the old bias, by the workgroups of the first row band (one column per thread)
  static_assert(!kIsDw || BN <= NTHR, "one bias column per thread");
  const bool bias_thread = kIsDw && m0 == 0 && tid < BN && n0 + tid < p.N;
  const float b_old = fused && bias_thread ? p.src[(size_t)g * p.src_gs + p.b_off + n0 + tid] : 0.0f;
  const float vb_old = MOM && bias_thread ? p.vel[pg + p.b_off + n0 + tid] : 0.0f;

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

  // db_l = colsum(D_l): the workgroups of the first row band feed the delta fragments they hold
  // anyway through one more matrix instruction against an all-ones operand
  const bool bias_wave = kIsDw && m0 == 0 && wm == 0;
  f32x16_t accb[kIsDw ? TN : 1];
#pragma unroll
  for (int j = 0; j < (kIsDw ? TN : 1); ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) accb[j][v] = 0.0f;

  // Software pipeline over S LDS stages and two fragment sets.  A wavefront reads the fragments of
  // the next slice while the matrix instructions of the current one run; before it reads the first
  // slice of the next tile it waits for its own requests of that tile and meets the others: then the
  // tile has landed for all, and nobody reads the current tile any more (the fragments have arrived,
  // lgkmcnt(0)), so that its stage takes tile it + S.  The matrix instructions of the last slice
  // are issued after that meeting and run over the latency of the new fragments.
  constexpr int KW = kSlices / WK;                         // slices of this wavefront's share of a tile
  Frag<T> af[2][TM], bf[2][TN];
  auto load = [&](int stage, int u, int set) __attribute__((always_inline)) {
    const unsigned char* a_t = smem + stage * STAGE;
    const unsigned char* b_t = a_t + BM * kTileBytes;
    const int kk = wk * KW + u;
#pragma unroll
    for (int i = 0; i < TM; ++i) af[set][i] = load_frag<T, BM, AKIND, NWAVE>(a_t, wm * TM + i, kk, lane);
#pragma unroll
    for (int j = 0; j < TN; ++j) bf[set][j] = load_frag<T, BN, BKIND, NWAVE>(b_t, wn * TN + j, kk, lane);
    __builtin_amdgcn_sched_barrier(0);                     // ahead of the matrix instructions below
  };
  auto multiply = [&](int u, int set, bool ragged) __attribute__((always_inline)) {
    if (ragged) {
      const int kk = wk * KW + u;
      if (kk * (BK / kSlices) >= k_tail) return;           // nothing but zeros
#pragma unroll
      for (int i = 0; i < TM; ++i) mask_frag(af[set][i], kk, lane, k_tail);
#pragma unroll
      for (int j = 0; j < TN; ++j) mask_frag(bf[set][j], kk, lane, k_tail);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = mma(af[set][i], bf[set][j], acc[i][j]);
    if constexpr (kIsDw) {
      if (bias_wave) {
        Frag<T> ones;
        set_ones(ones);
#pragma unroll
        for (int j = 0; j < TN; ++j) accb[j] = mma(ones, bf[set][j], accb[j]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  int it = 0, stage = 0;                                   // tile being multiplied, and its stage
  // Tile `it`, whose first slice is in fragment set FIRST; ends with the first slice of tile it + 1
  // in the set after its own last one (past the last tile: stale LDS contents, never multiplied).
  auto tile_step = [&](auto first_tag) __attribute__((always_inline)) {
    constexpr int FIRST = decltype(first_tag)::value;
    const bool ragged = it == n_k - 1 && k_tail < BK;
#pragma unroll
    for (int u = 0; u + 1 < KW; ++u) {
      load(stage, u + 1, (FIRST + u + 1) & 1);
      multiply(u, (FIRST + u) & 1, ragged);
    }
    const int ahead = n_k - 2 - it;                        // tiles requested after tile it + 1
    if (ahead >= S - 2) wait_tiles<PER, S - 1>(S - 2); else wait_tiles<PER, S - 1>(max(ahead, 0));
    asm volatile("s_barrier" ::: "memory");
    if (it + S < n_k) request(it + S, stage);
    stage = stage + 1 == S ? 0 : stage + 1;
    load(stage, 0, (FIRST + KW) & 1);
    multiply(KW - 1, (FIRST + KW - 1) & 1, ragged);
    ++it;
  };
#pragma unroll 1                                           // one copy of a request, and one in the loop
  for (int j = 0; j < min(S, n_k); ++j) request(j, j);
  if (n_k > 0) {
    wait_tiles<PER, S - 1>(min(S, n_k) - 1);
    asm volatile("s_barrier" ::: "memory");
    load(0, 0, 0);
    for (;;) {
      tile_step(std::integral_constant<int, 0>{});
      if (it == n_k) break;
      if constexpr ((KW & 1) != 0) {                       // the fragment sets swap roles every tile
        tile_step(std::integral_constant<int, 1>{});
        if (it == n_k) break;
      }
    }
  }
  RowsEpilogue<T, BM, BN, NTHR, BKIND == OP_CONTIG> out(m0, n0, tid);
  if constexpr (!kIsDw) out.request(p, g);
  __syncthreads();                                         // every wavefront is done with the last tile

  // ---- epilogue: accumulator element v of lane (lr32, kb) is C[8*(v/4) + 4*kb + v%4][lr32]; the
  // tile leaves through LDS (the operand stages are free now) in row-major vectors
  float* c_lds = reinterpret_cast<float*>(smem);           // [WK][BM][SC]
  float* cs_lds = c_lds + WK * BM * SC;                    // [WK][BN] column sums
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        c_lds[(wk * BM + (wm * TM + i) * 32 + 8 * (v / 4) + 4 * kb + (v % 4)) * SC + (wn * TN + j) * 32 + lr32] =
            acc[i][j][v];
  if constexpr (kIsDw) {
    if (bias_wave && kb == 0) {       // row 0 of the ones product: lane lr32 holds column lr32
#pragma unroll
      for (int j = 0; j < TN; ++j) cs_lds[wk * BN + (wn * TN + j) * 32 + lr32] = accb[j][0];
    }
  }
  __syncthreads();
  auto c_read = [&](int r, int c) __attribute__((always_inline)) {
    f32x4_t s = *reinterpret_cast<const f32x4_t*>(c_lds + r * SC + c);
#pragma unroll
    for (int w = 1; w < WK; ++w) {
      const f32x4_t o = *reinterpret_cast<const f32x4_t*>(c_lds + (w * BM + r) * SC + c);
      s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
    }
    return s;
  };

  if constexpr (kIsDw) {
    const size_t tile = pg + p.w_off + (size_t)m0 * p.ldw + n0;
    float* wtile = (fused ? p.params : p.grads) + tile;
    uint16_t* stile = p.shadow + tile;
#pragma unroll
    for (int q = 0; q < EV; ++q) {
      const int r = q * ROWS_PER_PASS + e_row;
      if (m0 + r < p.M && n0 + e_col < p.N) {
        f32x4_t gr = c_read(r, e_col);
        const uint32_t off = __umul24((uint32_t)r, (uint32_t)p.ldw) + (uint32_t)e_col;
        if (fused) {
          if constexpr (MOM) {
            gr.x = fmaf(p.mu, v_old[q].x, gr.x);
            gr.y = fmaf(p.mu, v_old[q].y, gr.y);
            gr.z = fmaf(p.mu, v_old[q].z, gr.z);
            gr.w = fmaf(p.mu, v_old[q].w, gr.w);
            f32x4_t* vp = reinterpret_cast<f32x4_t*>(p.vel + tile + off);
            if (p.streaming) __builtin_nontemporal_store(gr, vp);
            else *vp = gr;
          }
          f32x4_t w = w_old[q];
          w.x = fmaf(-p.lr, gr.x, w.x);
          w.y = fmaf(-p.lr, gr.y, w.y);
          w.z = fmaf(-p.lr, gr.z, w.z);
          w.w = fmaf(-p.lr, gr.w, w.w);
          const u32x2_t hv = {f32x2_to_bf16x2_rne(w.x, w.y),
                              f32x2_to_bf16x2_rne(w.z, w.w)};
          if (p.streaming) {
            __builtin_nontemporal_store(w, reinterpret_cast<f32x4_t*>(wtile + off));
            if (p.shadow != nullptr)
              __builtin_nontemporal_store(hv, reinterpret_cast<u32x2_t*>(stile + off));
          } else {
            *reinterpret_cast<f32x4_t*>(wtile + off) = w;
            if (p.shadow != nullptr) *reinterpret_cast<u32x2_t*>(stile + off) = hv;
          }
        } else {
          *reinterpret_cast<f32x4_t*>(wtile + off) = gr;
        }
      }
    }
    if (bias_thread) {
      float colsum = cs_lds[tid];
#pragma unroll
      for (int w = 1; w < WK; ++w) colsum += cs_lds[w * BN + tid];
      if constexpr (MOM) {
        colsum = fmaf(p.mu, vb_old, colsum);
        p.vel[pg + p.b_off + n0 + tid] = colsum;
      }
      if (fused) p.params[pg + p.b_off + n0 + tid] = fmaf(-p.lr, colsum, b_old);
      else p.grads[pg + p.b_off + n0 + tid] = colsum;
    }
  }
  if constexpr (!kIsDw) out.store(p, g, ks, c_read);
}

template <typename T, int BM, int BN, int WM, int WN, int WK, int S, int AKIND, int BKIND>
__global__ __launch_bounds__(64 * WM * WN * WK, 2) void grouped_gemm_kernel(GemmArgs p) {
  gemm_tile<T, BM, BN, WM, WN, WK, S, AKIND, BKIND, false>(p, (int)blockIdx.x);
}

// Several products in one launch: product i has the workgroups first[i] .. first[i + 1] - 1 (past the last product: none).
struct GemmSet {
  int first[kMaxGemmSet];
  GemmArgs p[kMaxGemmSet];
};
template <typename T, int BM, int BN, int WM, int WN, int WK, int S, int AKIND, int BKIND, bool MOM>
__global__ __launch_bounds__(64 * WM * WN * WK, 2) void grouped_gemm_set_kernel(GemmSet set) {
  int i = 0, first = 0;
#pragma unroll
  for (int k = 1; k < kMaxGemmSet; ++k)
    if ((int)blockIdx.x >= set.first[k]) { i = k; first = set.first[k]; }
  gemm_tile<T, BM, BN, WM, WN, WK, S, AKIND, BKIND, MOM>(set.p[i], (int)blockIdx.x - first);
}

template <typename T, int BM, int BN, int WM, int WN, int WK, int S, int AKIND, int BKIND>
static hipError_t launch_one(const GemmArgs& p, int n_groups, hipStream_t s) {
  return launch_tiles<T, BM, BN, WK, S, WM * WN * WK, grouped_gemm_kernel<T, BM, BN, WM, WN, WK, S, AKIND, BKIND>>(
      p, n_groups, s);
}
constexpr int kComputeUnits = 256;

// Batch-row products (forward, backward-data).  A launch takes the tile with which the busiest compute unit requests the fewest bytes:
// tiles per compute unit, rounded up, times rows + columns of a tile.  Not all are bound by that intake (128 x 128 tiles and small
// launches divide requests and products between wavefronts, kernels_gemm_rows.hip), but it orders the tiles well: over 600 products of
// 8 to 512 rows, 1 to 64 workers and 64 to 4096 columns and contraction elements the rule's tile is within 3 % of the best one on 88 %,
// within 10 % on 94 %.  The worst have contractions of one or two tiles behind the epilogue of 128 x 128 (31 x (128 x 128) x 2088 15.4 us, in
// 128 x 64 10.4).  Launched by itself in 32 x 64, 64 x 64, 128 x 64 and 128 x 128 tiles, the rule's in brackets: 8 x (128 x 4096) x 4096 with shared
// weights 72.5, 53.2, 45.2, [34.4] us, backward-data 71.3, 55.1, 46.9, [34.3]; 6 x (128 x 896) x 3776 22.0, 14.8, 13.3, [11.7]; 8 x (95 x
// 3456) x 3760 74.7, 57.8, 47.4, [33.0]; 64 x (128 x 1024) x 1024 43.5, 33.3, 30.9, [30.5]; 6 x (100 x 500) x 300 [4.4], 4.9, 6.6, 7.8.
// bf16 adds the contraction in one ascending chain in every tile: the first layer's backward kernel
// computes the same product ahead and must give the same bits.
// No tile is taller than the minibatch: half of a 128-row tile of 64 rows is copies of the last row, multiplied
// and thrown away (measured on an earlier kernel, 128 x (64 x 256) x 1024: 30.6 -> 21.0 us in 64 x 64 tiles; fp32 16 x (8 x 2048) x 2048:
// 47.7 -> 32.3 us forward, 43.6 -> 26.1 us backward-data in 32- instead of 64-row tiles).
// fp32 is bound by its matrix instructions, 8 times as slow: 32 x 32 tiles whose wavefronts share the
// contraction (8 x (50 x 784) x 300: 27.5 -> 12 us), until the chip is full either way.
struct RowsTile { int bm, bn; };
static RowsTile rows_tile(const GemmArgs& p, int n_groups, bool bf16) {
  auto tiles = [&](RowsTile t) {
    return (long)((p.M + t.bm - 1) / t.bm) * ((p.N + t.bn - 1) / t.bn) * n_groups;
  };
  const int tallest = p.M <= 32 ? 32 : p.M <= 64 ? 64 : 128;
  if (!bf16) return tallest >= 64 && tiles({64, 64}) >= 2 * kComputeUnits ? RowsTile{64, 64} : RowsTile{32, 32};
  RowsTile best = {32, 64};
  auto cost = [&](RowsTile t) { return (tiles(t) + kComputeUnits - 1) / kComputeUnits * (t.bm + t.bn); };
  for (const RowsTile t : {RowsTile{64, 64}, RowsTile{128, 64}, RowsTile{128, 128}})
    if (t.bm <= tallest && cost(t) <= cost(best)) best = t;
  return best;
}

// Tiles in flight per workgroup of the plain kernel, whose wavefronts all multiply.  Three cover the latency of one workgroup; with six or
// eight (74 to 147 KB of LDS) a compute unit held one workgroup of two to eight wavefronts, and a launch of more tiles than
// compute units ran in rounds.  With eight and with three tiles: 64 x (8 x 1024) x 1024 in 32 x 64 tiles 36.1
// and 15.8 us, 128 x (8 x 64) x 1024 25.3 and 10.6 us; 64 x (64 x 1024) x 256 in 64 x 64 tiles 24.2 and 13.9 us.  Two lose where a compute
// unit has one workgroup (4 x (8 x 4096) x 1024 three 20.6, two 32.1 us), which is where the requesting kernel stands now (11.4).
constexpr int kRowStages = 3;
static_assert(kRowStages == kFedStages, "128 x 64 tiles of either kernel");

// Workgroups with requesting wavefronts (kernels_gemm_rows.hip) take the 128 x 128 tiles, and launches of fewer than two smaller tiles per
// compute unit: from then on several workgroups of the plain kernel share a unit and hide each other's requests (its 48 KB of LDS
// allow three, four tiles in flight two).  Per iteration, plain and with requesting wavefronts: 6 workers of 1000-500-300-37, 100 rows,
// 37.7 and 35.3 us; 5 of 640-1024-448-960-29, 18 rows, 56.8 and 51.1; 16 of 600-300-100, 40 rows, 29.0 and 27.3; 24 of 520-520-520-520-30, 64
// rows (216 tiles of 64 x 64), 89.4 and 86.6; 48 of 700-400-400-120 (336) 87.6 and 86.6; 50 of 800-500-500-500-100, 50 rows (400) 194.6 and
// 193.4; 60 of it, 30 rows (480 of 32 x 64) 213.6 and 211.4.  At 512 it is one way with weights of every worker's own or a contraction
// in ranges (the logits product of 8 of 4096-4096-4096-4096-1000, 128 rows, interval 1, 24.2 and 25.7 us, an iteration 522.1 and 524.6; 32 of
// 1000-1000-1000-50, 32 and 64 rows, 195.6 and 196.4, 206.6 and 207.1) and the other way with shared ones (64 of 1024-512-512-512-40, 64 rows,
// interval 1, 104.0 and 102.7).  64 of 1000-1000-1000-50, 32 rows (1024), 347.4 and 349.2.  128 x 64 tiles, the launch alone, forward and
// backward-data: 5 x (101 x 2688) x 4005 48.9 and 49.6 us, 5 x (101 x 2362) x 2688 26.7 and 24.4, 20.8 and 17.6; 6 x (128 x 2624) x 2880
// 26.5 and 23.6; 10 x (128 x 832) x 1472 12.2 and 10.2; 10 x (128 x 1472) x 832 10.1 and 8.4; 13 x (128 x 640) x 708 9.2 and 8.3.
constexpr long kFedTiles = 2 * kComputeUnits;
static long rows_tiles(RowsTile t, int rows, int cols, int splits, int n_groups) {
  return (long)((rows + t.bm - 1) / t.bm) * ((cols + t.bn - 1) / t.bn) * (splits > 1 ? splits : 1) * n_groups;
}
static bool rows_fed(RowsTile t, const GemmArgs& p, int n_groups) {
  if (t.bn == 128) return true;
  const long tiles = rows_tiles(t, p.M, p.N, p.k_splits, n_groups);
  return tiles < kFedTiles || (tiles == kFedTiles && p.b_gs == 0 && p.k_splits <= 1);
}

// fp32 tiles of 32 x 32: a step of the plain kernel is 256 cycles of matrix instructions and 130 in which the same wavefronts are held up
// in their requests.  Launch alone, plain and with requesting wavefronts: 8 x (50 x 300) x 784 10.1 and 8.2 us, 4 x (16 x 66) x 997 12.4 and
// 8.9, 6 x (43 x 66) x 771 10.4 and 7.5, 5 x (73 x 383) x 457 8.7 and 6.6, 3 x (10 x 75) x 320 5.4 and 5.0.  Per iteration, tiles of the first
// layer in brackets: 512-1024-512-10, 8 rows, [256] 48.2 and 42.5 us, [512] 61.7 and 57.6, [1024] 96.8 and 94.9, [4096] 407 and 408;
// 256-256-256-10, 50 rows, [512] 41.5 and 41.7, [2048] 96.2 and 98.6.
static bool f32_fed(const GemmArgs& p, int n_groups) { return rows_tiles({32, 32}, p.M, p.N, p.k_splits, n_groups) <= kFedTiles; }

template <int AKIND, int BKIND>
static hipError_t launch_rows_bf16(const GemmArgs& p, int n_groups, hipStream_t s) {
  const RowsTile t = rows_tile(p, n_groups, true);
  if (rows_fed(t, p, n_groups))
    return BKIND == OP_CONTIG ? launch_gemm_dx_fed(p, n_groups, t.bm, t.bn, s) : launch_gemm_fwd_fed(p, n_groups, t.bm, t.bn, s);
  if (t.bm == 32) return launch_one<TBF16, 32, 64, 1, 2, 1, kRowStages, AKIND, BKIND>(p, n_groups, s);
  if (t.bm == 64) return launch_one<TBF16, 64, 64, 2, 2, 1, kRowStages, AKIND, BKIND>(p, n_groups, s);
  return launch_one<TBF16, 128, 64, 4, 2, 1, kRowStages, AKIND, BKIND>(p, n_groups, s);
}
template <int AKIND, int BKIND>
static hipError_t launch_rows_f32(const GemmArgs& p, int n_groups, hipStream_t s) {
  if (rows_tile(p, n_groups, false).bm == 64)
    return launch_one<TF32, 64, 64, 2, 2, 1, 4, AKIND, BKIND>(p, n_groups, s);
  if (f32_fed(p, n_groups))
    return BKIND == OP_CONTIG ? launch_gemm_dx_fed(p, n_groups, 32, 32, s) : launch_gemm_fwd_fed(p, n_groups, 32, 32, s);
  return launch_one<TF32, 32, 32, 1, 1, 4, kRowStages, AKIND, BKIND>(p, n_groups, s);
}

void gemm_rows_shape(int rows, int cols, int n_groups, bool bf16, int* tile_rows, int* tile_cols, size_t* lds_bytes) {
  GemmArgs p;
  memset(&p, 0, sizeof(p));
  p.M = rows; p.N = cols;
  p.b_gs = 1;                                              // every worker has weights of its own
  const RowsTile t = rows_tile(p, n_groups, bf16);
  const bool fed = rows_fed(t, p, n_groups);
  *tile_rows = t.bm;
  *tile_cols = t.bn;
  *lds_bytes = !bf16 ? (t.bm == 64 ? gemm_lds_bytes<TF32, 64, 64, 1, 4>()
                        : f32_fed(p, n_groups) ? gemm_lds_bytes<TF32, 32, 32, 4, kFedSmallStages>()
                                               : gemm_lds_bytes<TF32, 32, 32, 4, kRowStages>())
               : t.bm == 32 ? (fed ? gemm_lds_bytes<TBF16, 32, 64, 1, kFedSmallStages>() : gemm_lds_bytes<TBF16, 32, 64, 1, kRowStages>())
               : t.bm == 64 ? (fed ? gemm_lds_bytes<TBF16, 64, 64, 1, kFedSmallStages>() : gemm_lds_bytes<TBF16, 64, 64, 1, kRowStages>())
               : t.bn == 64 ? gemm_lds_bytes<TBF16, 128, 64, 1, kRowStages>() : gemm_lds_bytes<TBF16, 128, 128, 1, kFedStages>();
}

// A logits product that leaves most compute units idle (few classes) cuts its contraction into
// 2 or 4 ranges of whole tiles, every range non-empty and at least two tiles long.
int gemm_logit_splits(const GemmArgs& p, int n_groups, bool bf16) {
  const int bk = kTileBytes / (bf16 ? 2 : 4);
  const int n_k = (p.Kc + bk - 1) / bk;
  const RowsTile t = rows_tile(p, n_groups, bf16);
  const long wgs = (long)((p.M + t.bm - 1) / t.bm) * ((p.N + t.bn - 1) / t.bn) * n_groups;
  for (int s = kMaxLogitSplits; s >= 2; s >>= 1) {
    const int per = (n_k + s - 1) / s;
    if (wgs * s <= 2 * kComputeUnits && per >= 2 && (long)per * (s - 1) < n_k) return s;
  }
  return 1;
}

hipError_t launch_gemm_fwd(const GemmArgs& p, int n_groups, bool bf16, hipStream_t s) {
  return bf16 ? launch_rows_bf16<OP_CONTIG, OP_TRANS>(p, n_groups, s)
              : launch_rows_f32<OP_CONTIG, OP_TRANS>(p, n_groups, s);
}
hipError_t launch_gemm_dx(const GemmArgs& p, int n_groups, bool bf16, hipStream_t s) {
  return bf16 ? launch_rows_bf16<OP_CONTIG, OP_CONTIG>(p, n_groups, s)
              : launch_rows_f32<OP_CONTIG, OP_CONTIG>(p, n_groups, s);
}
// Weight-gradient products.  128 x 128 tiles in workgroups of four wavefronts, two of them per compute
// unit, so that the weight read-modify-write of one runs beside the products of the other: 4096 x 4096
// with 1024 stacked rows 87 -> 70 us, 8 x (3072 x 1024) with 512 rows 102 -> 79 us.  Launches without two such
// tiles per compute unit: 64 x 64 tiles.  Layers that share a launch take the large tiles if one of them does: the old weights of
// one workgroup then run beside the products of others that have come out of step, where launches of two rounds move and multiply in
// turn, and small layers cost no rounds of their own.  Kernels of an iteration, launches apart and one: 8 x 4096-4096-4096-4096-1000 at
// interval 1 225 and 213 us; 8 x 3072-1024-1024-10 with 512 rows 111 and 105; 4 x 2112-2944-2880-2472-465, 128 rows, interval 1, all
// launches 228 and 192; 10 x 2116-576-576-28, 194 rows, 98 and 89.
static bool dw_large(const GemmArgs& p, int n_groups, bool bf16) {
  return bf16 && (long)((p.M + 127) / 128) * ((p.N + 127) / 128) * n_groups >= 2 * kComputeUnits;
}
// Launches without two such tiles per compute unit are bound by latency, not by what they move
// (7 us for a single 64 x 64 tile: launch, first operand and weight loads, write-back), so the layers'
// products, which depend on nothing of each other, share one launch (fp32 784-300-100-10, eight workers:
// 11.8 + 6.9 + 7.1 us in three launches, 12.7 us in one).
template <typename T, int BM, int BN, int WM, int S, bool MOM = false> static hipError_t launch_dw_set(const GemmArgs* ps, int n, int n_groups, hipStream_t s) {
  constexpr size_t kLds = gemm_lds_bytes<T, BM, BN, 1, S>();
  auto kernel = grouped_gemm_set_kernel<T, BM, BN, WM, 2, 1, S, OP_TRANS, OP_TRANS, MOM>;
  static std::atomic<bool> configured{false};
  if (!configured.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
    if (e != hipSuccess) return e;
    configured.store(true, std::memory_order_release);
  }
  GemmSet set;
  memset(&set, 0, sizeof(set));
  int used = 0, total = 0;
  for (int i = 0; i < n; ++i) {
    if (ps[i].M <= 0 || ps[i].N <= 0 || n_groups <= 0) continue;
    if (ps[i].k_splits > 1) return hipErrorInvalidValue;
    set.first[used] = total;
    set.p[used] = ps[i];
    total += place_tiles(&set.p[used], BM, BN, n_groups);
    ++used;
  }
  if (used == 0) return hipSuccess;
  for (int i = used; i < kMaxGemmSet; ++i) set.first[i] = total;
  hipLaunchKernelGGL(kernel, dim3((unsigned)total), dim3(128 * WM), kLds, s, set);
  return hipGetLastError();
}
// With momentum, bf16 layers of up to 128 rows: large tiles in eight wavefronts, since old weights and velocities of four do not fit
// their registers.
static hipError_t launch_dw_momentum(const GemmArgs* ps, int n, int n_groups, bool bf16, hipStream_t s) {
  if (!bf16) return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i)
    if (ps[i].epi != EPI_DW_FUSED || ps[i].vel == nullptr || ps[i].Kc > 128) return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i)
    if (dw_large(ps[i], n_groups, bf16)) return launch_dw_set<TBF16, 128, 128, 4, 2, true>(ps, n, n_groups, s);
  return launch_dw_set<TBF16, 64, 64, 2, 2, true>(ps, n, n_groups, s);
}
hipError_t launch_gemm_dw(const GemmArgs* ps, int n, int n_groups, bool bf16, hipStream_t s) {
  if (n < 0 || n > kMaxGemmSet) return hipErrorInvalidValue;
  if (n > 0 && ps[0].vel != nullptr) return launch_dw_momentum(ps, n, n_groups, bf16, s);
  if (n == 1 && dw_large(ps[0], n_groups, bf16))
    return launch_one<TBF16, 128, 128, 2, 2, 1, 2, OP_TRANS, OP_TRANS>(ps[0], n_groups, s);
  // contractions of one or two tiles: two stages, and the more workgroups on a compute unit
  int depth = 0;
  for (int i = 0; i < n; ++i) depth = depth > ps[i].Kc ? depth : ps[i].Kc;
  const bool shallow = depth <= 2 * kTileBytes / (bf16 ? 2 : 4);
  // one product: a kernel that has its arguments at fixed places is 0.5 us faster (7.0 and 7.5 us for 165 x 10, 32 rows)
  if (n == 1) {
    if (bf16)
      return shallow ? launch_one<TBF16, 64, 64, 2, 2, 1, 2, OP_TRANS, OP_TRANS>(ps[0], n_groups, s)
                     : launch_one<TBF16, 64, 64, 2, 2, 1, 4, OP_TRANS, OP_TRANS>(ps[0], n_groups, s);
    return shallow ? launch_one<TF32, 64, 64, 2, 2, 1, 2, OP_TRANS, OP_TRANS>(ps[0], n_groups, s)
                   : launch_one<TF32, 64, 64, 2, 2, 1, 4, OP_TRANS, OP_TRANS>(ps[0], n_groups, s);
  }
  for (int i = 0; i < n; ++i)
    if (dw_large(ps[i], n_groups, bf16)) return launch_dw_set<TBF16, 128, 128, 2, 2>(ps, n, n_groups, s);
  if (bf16) return shallow ? launch_dw_set<TBF16, 64, 64, 2, 2>(ps, n, n_groups, s) : launch_dw_set<TBF16, 64, 64, 2, 4>(ps, n, n_groups, s);
  return shallow ? launch_dw_set<TF32, 64, 64, 2, 2>(ps, n, n_groups, s) : launch_dw_set<TF32, 64, 64, 2, 4>(ps, n, n_groups, s);
}

}  // namespace prsgd
