// Batch-row products (forward, backward-data) whose workgroups divide the work by kind of instruction: those in 128 x 128 tiles, and
// launches of few smaller ones (kernels_gemm.hip says which).
#include "gemm_tile.h"

namespace prsgd {

// The same tile of a batch-row product in a workgroup whose wavefronts share the work by kind: four multiply, CM x CN over the
// output tile, four request.  A wavefront that requests is held up until its requests are taken (65 cycles each per SIMD, 32 of them for
// a 128 x 128 tile), and then its matrix instructions wait with it; a SIMD has one wavefront of each kind.  The multiplying
// wavefronts hold the fragments of a whole tile and read the next tile's behind the matrix instructions, so that they meet the
// others once per tile, and with 64 x 64 outputs each they read 64 KB of LDS per 128 x 128 tile where eight of 64 x 32 read 96.
// Same order of the contraction, same bits as gemm_tile.  Workers x (rows x contraction) x columns, against eight wavefronts that do
// both: 8 x (128 x 4096) x 4096 with shared weights 46 -> 36 us forward, 44 -> 35 us backward-data, launched by itself; in an iteration
// at interval 1, with the weights in HBM and clocks at the power limit, 50 -> 46 and 40 -> 33 us.
// fp32, whose tiles are 32 x 32: the multiplying wavefronts share the contraction (WK), and the shares are added in order.
template <typename T, int BM, int BN, int CM, int CN, int WK, int S, int AKIND, int BKIND>
__device__ __forceinline__ void gemm_rows_fed(const GemmArgs& p, int block) {
  using E = typename T::elem;
  constexpr int NREQ = 4, NMUL = CM * CN * WK, NTHR = 64 * (NREQ + NMUL);          // requesting, multiplying wavefronts; threads
  constexpr int KW = kSlices / WK;                         // slices of a multiplying wavefront
  using IOA = TileIO<T, BM, AKIND, NREQ>;
  using IOB = TileIO<T, BN, BKIND, NREQ>;
  constexpr int BK = IOA::BK, PER = IOA::NPT + IOB::NPT;
  constexpr int TM = BM / (32 * CM), TN = BN / (32 * CN);
  static_assert(NMUL <= 4 && kSlices % WK == 0, "at most a multiplying and a requesting wavefront per SIMD");
  static_assert(TM >= 1 && TN >= 1, "tile too small for the wavefront grid");
  static_assert(S >= 2 && S <= 4 && PER * (S - 1) <= 63, "wait_tiles");

  fetch_args(p);
  const TileAt at = tile_at<BM, BN>(p, block);
  const int g = at.g, m0 = at.m0, n0 = at.n0;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  constexpr int STAGE = (BM + BN) * kTileBytes;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool multiplies = wave < NMUL;
  const int wk = wave / (CM * CN), wm = (wave / CN) % CM, wn = wave % CN;
  int Kc, k_lo;
  contraction_range<BK>(p, at, &k_lo, &Kc);
  const int n_k = (Kc + BK - 1) / BK;
  const int k_tail = Kc - (n_k - 1) * BK;                  // elements of the last tile

  // The workgroup meets n_k times.  At meeting t tile t has landed, and every fragment of tile t - 1 has been read, so that
  // its stage takes tile t - 1 + S.
  f32x16_t acc[TM][TN];
  if (!multiplies) {
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const int w = wave - NMUL;
    const E* a_src = reinterpret_cast<const E*>(p.a) + (size_t)g * p.a_gs +
                     (AKIND == OP_CONTIG ? (size_t)m0 * p.lda + k_lo : (size_t)k_lo * p.lda + m0);
    const E* b_src = reinterpret_cast<const E*>(p.b) + (size_t)g * p.b_gs +
                     (BKIND == OP_CONTIG ? (size_t)n0 * p.ldb + k_lo : (size_t)k_lo * p.ldb + n0);
    const size_t a_step = AKIND == OP_CONTIG ? (size_t)BK : (size_t)BK * p.lda;
    const size_t b_step = BKIND == OP_CONTIG ? (size_t)BK : (size_t)BK * p.ldb;
    uint32_t a_off[IOA::NPT], b_off[IOB::NPT];
    IOA::template offsets<false>(a_off, p.lda, p.M - m0, BK, w, lane);
    IOB::template offsets<false>(b_off, p.ldb, p.N - n0, BK, w, lane);
    auto request = [&](int j, int stage) __attribute__((always_inline)) {
      const uint32_t lds_a = lds0 + (uint32_t)stage * STAGE, lds_b = lds_a + BM * kTileBytes;
      if (j == n_k - 1 && k_tail < BK) {                   // nothing past the operands is touched
        IOA::template offsets<true>(a_off, p.lda, p.M - m0, k_tail, w, lane);
        IOB::template offsets<true>(b_off, p.ldb, p.N - n0, k_tail, w, lane);
      }
      IOA::request(a_src + (size_t)j * a_step, a_off, lds_a, w);
      IOB::request(b_src + (size_t)j * b_step, b_off, lds_b, w, p.b_once != 0);
    };
#pragma unroll 1                                           // one copy of a request, and one in the loop
    for (int j = 0; j < min(S, n_k); ++j) request(j, j);
    int stage = S - 1;                                     // of tile t - 1
    for (int t = 0; t < n_k; ++t) {
      const int ahead = min(n_k - 1 - t, t == 0 ? S - 1 : S - 2);      // tiles requested after tile t
      if (ahead == S - 2) wait_tiles<PER, S - 1>(S - 2); else wait_tiles<PER, S - 1>(ahead);
      asm volatile("s_barrier" ::: "memory");
      if (t > 0 && t - 1 + S < n_k) request(t - 1 + S, stage);
      stage = stage + 1 == S ? 0 : stage + 1;
    }
  } else {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    Frag<T> af[2][KW][TM], bf[2][KW][TN];
    auto load = [&](int stage, int u, int set) __attribute__((always_inline)) {
      const unsigned char* a_t = smem + stage * STAGE;
#pragma unroll
      for (int i = 0; i < TM; ++i) af[set][u][i] = load_frag<T, BM, AKIND, NREQ>(a_t, wm * TM + i, wk * KW + u, lane);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        bf[set][u][j] = load_frag<T, BN, BKIND, NREQ>(a_t + BM * kTileBytes, wn * TN + j, wk * KW + u, lane);
    };
    int stage = 0;
    // multiplies the tile in set SET; not the last one: reads the next tile into the other set
    auto step = [&](auto set_tag, auto last_tag) __attribute__((always_inline)) {
      constexpr int SET = decltype(set_tag)::value;
      constexpr bool LAST = decltype(last_tag)::value;
      if constexpr (!LAST) {
        stage = stage + 1 == S ? 0 : stage + 1;
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      }
#pragma unroll
      for (int u = 0; u < KW; ++u) {
        if constexpr (!LAST) load(stage, u, SET ^ 1);
        if (LAST && (wk * KW + u) * (BK / kSlices) >= k_tail) continue;          // nothing but zeros
        if (LAST && k_tail < BK) {
#pragma unroll
          for (int i = 0; i < TM; ++i) mask_frag(af[SET][u][i], wk * KW + u, lane, k_tail);
#pragma unroll
          for (int j = 0; j < TN; ++j) mask_frag(bf[SET][u][j], wk * KW + u, lane, k_tail);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = mma(af[SET][u][i], bf[SET][u][j], acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    using Set0 = std::integral_constant<int, 0>;
    using Set1 = std::integral_constant<int, 1>;
    if (n_k > 0) {
      asm volatile("s_barrier" ::: "memory");
#pragma unroll
      for (int u = 0; u < KW; ++u) load(0, u, 0);
      int t = 0;
      for (; t + 2 < n_k; t += 2) {                        // one way out: the accumulators stay where they are
        step(Set0{}, std::false_type{});
        step(Set1{}, std::false_type{});
      }
      if (t + 2 == n_k) {
        step(Set0{}, std::false_type{});
        step(Set1{}, std::true_type{});
      } else {
        step(Set0{}, std::true_type{});
      }
    }
  }
  RowsEpilogue<T, BM, BN, NTHR, BKIND == OP_CONTIG> out(m0, n0, tid);
  out.request(p, g);
  __syncthreads();                                         // every wavefront is done with the last tile
  constexpr int SC = BN + 4;
  float* c_lds = reinterpret_cast<float*>(smem);           // [WK][BM][SC]
  if (multiplies) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          c_lds[(wk * BM + (wm * TM + i) * 32 + 8 * (v / 4) + 4 * (lane >> 5) + (v % 4)) * SC + (wn * TN + j) * 32 + (lane & 31)] =
              acc[i][j][v];
  }
  __syncthreads();
  out.store(p, g, at.split, [&](int r, int c) __attribute__((always_inline)) {
    f32x4_t s = *reinterpret_cast<const f32x4_t*>(c_lds + r * SC + c);
#pragma unroll
    for (int w = 1; w < WK; ++w) {
      const f32x4_t o = *reinterpret_cast<const f32x4_t*>(c_lds + (w * BM + r) * SC + c);
      s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
    }
    return s;
  });
}

template <typename T, int BM, int BN, int CM, int CN, int WK, int S, int AKIND, int BKIND>
__global__ __launch_bounds__(64 * (4 + CM * CN * WK), 2) void grouped_rows_kernel(GemmArgs p) {
  gemm_rows_fed<T, BM, BN, CM, CN, WK, S, AKIND, BKIND>(p, (int)blockIdx.x);
}
template <typename T, int BM, int BN, int CM, int CN, int WK, int S, int AKIND, int BKIND>
static hipError_t launch_fed_tiles(const GemmArgs& p, int n_groups, hipStream_t s) {
  return launch_tiles<T, BM, BN, WK, S, 4 + CM * CN * WK, grouped_rows_kernel<T, BM, BN, CM, CN, WK, S, AKIND, BKIND>>(p, n_groups, s);
}

template <int AKIND, int BKIND> static hipError_t launch_fed(const GemmArgs& p, int n_groups, int bm, int bn, hipStream_t s) {
  constexpr int S = kFedStages, T = kFedSmallStages;
  if (bn == 32) return launch_fed_tiles<TF32, 32, 32, 1, 1, 4, T, AKIND, BKIND>(p, n_groups, s);
  if (bm == 32) return launch_fed_tiles<TBF16, 32, 64, 1, 2, 1, T, AKIND, BKIND>(p, n_groups, s);
  if (bm == 64) return launch_fed_tiles<TBF16, 64, 64, 2, 2, 1, T, AKIND, BKIND>(p, n_groups, s);
  if (bn == 64) return launch_fed_tiles<TBF16, 128, 64, 2, 2, 1, S, AKIND, BKIND>(p, n_groups, s);
  return launch_fed_tiles<TBF16, 128, 128, 2, 2, 1, S, AKIND, BKIND>(p, n_groups, s);
}
hipError_t launch_gemm_fwd_fed(const GemmArgs& p, int n_groups, int bm, int bn, hipStream_t s) {
  return launch_fed<OP_CONTIG, OP_TRANS>(p, n_groups, bm, bn, s);
}
hipError_t launch_gemm_dx_fed(const GemmArgs& p, int n_groups, int bm, int bn, hipStream_t s) {
  return launch_fed<OP_CONTIG, OP_CONTIG>(p, n_groups, bm, bn, s);
}

}  // namespace prsgd
