// What the grouped products share: operand tiles requested into LDS, MFMA fragments, the workgroup's place, and the
// epilogue of the batch-row products (gfx950 only).
#pragma once

#include <atomic>
#include <type_traits>

#include "prsgd_internal.h"

namespace prsgd {

enum { OP_CONTIG = 0, OP_TRANS = 1 };

struct TF32 {
  using elem = float;
  static constexpr bool kBf16 = false;
};
struct TBF16 {
  using elem = uint16_t;
  static constexpr bool kBf16 = true;
};
constexpr int kTileBytes = 128;        // depth of a tile along the contraction
constexpr int kSlices = 4;             // 32-byte slices of it, one fragment step each

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float act_fwd(float z, int act) {
  return act == PRSGD_TANH ? tanhf(z) : fmaxf(z, 0.0f);
}
__device__ __forceinline__ float act_bwd_from_h(float h, int act) {
  return act == PRSGD_TANH ? (1.0f - h * h) : (h > 0.0f ? 1.0f : 0.0f);
}

// One operand tile of ROWS output rows (or columns) in LDS, and the requests that fill it.
//   OP_CONTIG: element (r, c) at src[r * ld + c]; LDS [ROWS][128 bytes], chunks at lds_chunk
//   OP_TRANS : element (r, c) at src[c * ld + r]; LDS [depth][ROWS], bf16 segments at lds_seg_xor
// Rows past the operand are requested as copies of the last one (their results are not stored).
template <typename T, int ROWS, int KIND, int NWAVE> struct TileIO {
  using E = typename T::elem;
  static constexpr int ES = (int)sizeof(E), BK = kTileBytes / ES, V = 16 / ES;
  static constexpr int BYTES = ROWS * kTileBytes;
  static constexpr int NPT = BYTES / 1024 / NWAVE;         // requests per wavefront and tile
  static_assert(BYTES % (1024 * NWAVE) == 0, "a tile must split evenly over the wavefronts");
  static constexpr int ROW_BYTES = KIND == OP_CONTIG ? kTileBytes : ROWS * ES;
  static constexpr int CH = ROW_BYTES / 16;                // 16-byte chunks of an LDS row

  // permutation of the 64-byte segments of contraction row c (OP_TRANS)
  __device__ static __forceinline__ int seg_xor(int c) { return T::kBf16 ? lds_seg_xor<ROW_BYTES>(c) : 0; }
  // offsets (bytes from the tile's base address, 32 bits: a tile is at most 128 rows of 2^20 elements) of this lane's requests.
  // n_rows: rows of the operand from the tile's first; n_c (RAGGED): contraction elements from the tile's first, clamped like
  // the rows
  template <bool RAGGED>
  __device__ static __forceinline__ void offsets(uint32_t (&off)[NPT], int ld, int n_rows, int n_c, int wave,
                                                 int lane) {
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      const uint32_t chunk = (uint32_t)(q * NWAVE + wave) * 64 + (uint32_t)lane;       // position in the LDS tile
      const int lr = (int)(chunk / CH), pos = (int)(chunk % CH);
      if (KIND == OP_CONTIG) {
        const int row = min(lr, n_rows - 1);
        int c = lds_chunk(lr, pos) * V;
        if (RAGGED) c = min(c, (n_c - 1) & ~(V - 1));
        off[q] = (__umul24((uint32_t)row, (uint32_t)ld) + (uint32_t)c) * ES;
      } else {
        const int c = RAGGED ? min(lr, n_c - 1) : lr;
        const int row = min(((((pos >> 2) ^ seg_xor(lr)) << 2) | (pos & 3)) * V, (n_rows - 1) & ~(V - 1));
        off[q] = (__umul24((uint32_t)c, (uint32_t)ld) + (uint32_t)row) * ES;
      }
    }
  }
  __device__ static __forceinline__ void request(const E* tile_base, const uint32_t (&off)[NPT], uint32_t lds_tile,
                                                 int wave, bool once = false) {
    if (once) {
#pragma unroll
      for (int q = 0; q < NPT; ++q)
        load_to_lds<true>(tile_base, off[q], lds_tile + (uint32_t)(q * NWAVE + wave) * 1024u);
    } else {
#pragma unroll
      for (int q = 0; q < NPT; ++q)
        load_to_lds(tile_base, off[q], lds_tile + (uint32_t)(q * NWAVE + wave) * 1024u);
    }
  }
};

// MFMA operand fragments of a 32-row block for the kk-th 32-byte slice.  Lane (r = lane % 32,
// kb = lane / 32) holds contraction elements of row r; A and B fragments use the same assignment,
// which is all the instruction needs for the product to be the plain sum over c.
//   bf16: the eight elements 16 kk + 8 kb + 0..7 of one v_mfma_f32_32x32x16
//   fp32: the four elements   8 kk + 4 kb + 0..3 of four v_mfma_f32_32x32x2
template <typename T> struct Frag;
template <> struct Frag<TBF16> { bf16x8_t v; };
template <> struct Frag<TF32> { f32x4_t v; };

template <typename T, int ROWS, int KIND, int NWAVE>
__device__ __forceinline__ Frag<T> load_frag(const unsigned char* tile, int block, int kk, int lane) {
  using IO = TileIO<T, ROWS, KIND, NWAVE>;
  Frag<T> f;
  const int r = lane & 31, kb = lane >> 5;
  if constexpr (KIND == OP_CONTIG && T::kBf16) {
    f.v = lds_frag_contig(tile, block, kk, lane);
  } else if constexpr (KIND == OP_CONTIG) {
    f.v = *reinterpret_cast<const f32x4_t*>(tile + (block * 32 + r) * kTileBytes + (lds_chunk(r, 2 * kk + kb) << 4));
  } else if constexpr (T::kBf16) {
    f.v = lds_frag_trans<IO::ROW_BYTES>(tile, block, kk, lane);
  } else {
    const unsigned char* p = tile + (8 * kk + 4 * kb) * IO::ROW_BYTES + (block * 32 + r) * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) f.v[e] = *reinterpret_cast<const float*>(p + e * IO::ROW_BYTES);
  }
  return f;
}

__device__ __forceinline__ f32x16_t mma(const Frag<TBF16>& a, const Frag<TBF16>& b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, b.v, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16_t mma(const Frag<TF32>& a, const Frag<TF32>& b, f32x16_t c) {
#pragma unroll
  for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[e], b.v[e], c, 0, 0, 0);
  return c;
}
// Fragment of all ones: as A operand every row of the 32 x 32 result holds the column sums of B.
__device__ __forceinline__ void set_ones(Frag<TBF16>& f) {
  const u16x8_t u = {0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80};
  f.v = __builtin_bit_cast(bf16x8_t, u);
}
__device__ __forceinline__ void set_ones(Frag<TF32>& f) { f.v = (f32x4_t){1.0f, 1.0f, 1.0f, 1.0f}; }

// Zeroes the contraction elements at and past n_c (the last tile of a ragged contraction; what was
// requested there is some other element of the operand).
__device__ __forceinline__ void mask_frag(Frag<TBF16>& f, int kk, int lane, int n_c) {
  u32x4_t u = __builtin_bit_cast(u32x4_t, f.v);
  const int c = 16 * kk + 8 * (lane >> 5);
#pragma unroll
  for (int e = 0; e < 4; ++e)
    u[e] &= (c + 2 * e < n_c ? 0xFFFFu : 0u) | (c + 2 * e + 1 < n_c ? 0xFFFF0000u : 0u);
  f.v = __builtin_bit_cast(bf16x8_t, u);
}
__device__ __forceinline__ void mask_frag(Frag<TF32>& f, int kk, int lane, int n_c) {
  const int c = 8 * kk + 4 * (lane >> 5);
#pragma unroll
  for (int e = 0; e < 4; ++e) f.v[e] = c + e < n_c ? f.v[e] : 0.0f;
}

// Waits until all but the newest `ahead` tiles (PER requests each, `ahead` at most MOST) have landed.
template <int PER, int MOST> __device__ __forceinline__ void wait_tiles(int ahead) {
#define PRSGD_WAIT(n) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"((n) * PER > 63 ? 63 : (n) * PER) : "memory")
  if (MOST >= 3 && ahead >= 3) PRSGD_WAIT(3);
  else if (MOST >= 2 && ahead >= 2) PRSGD_WAIT(2);
  else if (MOST >= 1 && ahead >= 1) PRSGD_WAIT(1);
  else PRSGD_WAIT(0);
#undef PRSGD_WAIT
}

template <typename T, int BM, int BN, int WK, int S> constexpr size_t gemm_lds_bytes() {
  const size_t stages = (size_t)S * (BM + BN) * kTileBytes;
  const size_t out = sizeof(float) * ((size_t)WK * BM * (BN + 4) + (size_t)WK * BN);
  return stages > out ? stages : out;
}

// Workgroup -> (group, tile).  The hardware deals consecutive workgroups round-robin to the 8
// XCDs; each XCD gets a contiguous range of the tiles, so that a group's activations and weight
// panel stay in that XCD's L2.  The order is by group; with one weight stream for all groups
// (b_gs == 0) by column tile first, and with a single group in 8-high strips of tiles.
// What the divisions need is worked out on the host (place_tiles): eight of them by values that the compiler does not know
// were half of the 430 to 570 instructions, at 5 cycles each and more, in front of a workgroup's first request (16 iterations of
// 784-300-100-10 in fp32, eight workers, 691 -> 655 us; of 1000-500-300-37, six workers, 702 -> 665 us).
// n / d = (mulhi(mul, n) + n) >> shift for n < 2^31 (Granlund and Montgomery, "Division by invariant integers using
// multiplication", 1994)
constexpr TileDivisor tile_divisor(uint32_t d) {
  uint32_t shift = 0;
  while ((1ull << shift) < d) ++shift;
  return TileDivisor{(uint32_t)((((1ull << shift) - d) << 32) / d + 1), shift, d};
}
constexpr bool divides(uint32_t d) {                       // at both ends of the first and the last quotients
  const TileDivisor v = tile_divisor(d);
  for (uint32_t i = 0; i < 16; ++i) {
    const uint32_t q = i < 8 ? i : 0x7FFFFFFFu / d - (i - 8), lo = q * d, hi = 0x7FFFFFFFu - lo < d ? 0x7FFFFFFFu : lo + d - 1;
    if ((i >= 8 && 0x7FFFFFFFu / d < 16) || lo > 0x7FFFFFFFu) continue;
    for (const uint32_t n : {lo, hi})
      if ((uint32_t)((((uint64_t)v.mul * n) >> 32) + n) >> v.shift != n / d) return false;
  }
  return true;
}
constexpr bool divides_up_to(uint32_t d) { return d == 0 || (divides(d) && divides_up_to(d - 1)); }
static_assert(divides_up_to(400) && divides(641) && divides(4096) && divides(65537) && divides(1000003), "tile_divisor");
__device__ __forceinline__ int quotient(const TileDivisor& v, int n) {
  return (int)((__umulhi(v.mul, (uint32_t)n) + (uint32_t)n) >> v.shift);
}
// Fills in the placement of p's tiles of bm x bn; returns the workgroups of the product.
inline int place_tiles(GemmArgs* p, int bm, int bn, int n_groups) {
  const int tiles_m = (p->M + bm - 1) / bm, tiles_n = (p->N + bn - 1) / bn;
  const int n_splits = p->k_splits > 1 ? p->k_splits : 1;  // 1, 2 or 4
  const int total = tiles_m * tiles_n * n_splits * n_groups;
  TilePlace& t = p->place;
  t.xcd_tiles = total >> 3;
  t.xcd_extra = total & 7;
  t.split_shift = n_splits == 4 ? 2 : n_splits == 2 ? 1 : 0;
  t.order = n_groups == 1 ? 2 : p->b_gs == 0 ? 1 : 0;
  t.first = tile_divisor(t.order == 2 ? 8 * tiles_n : t.order == 1 ? tiles_m : tiles_m * tiles_n);
  t.second = tile_divisor(t.order == 2 ? 8 : t.order == 1 ? n_groups : tiles_n);
  t.whole_strips = tiles_m >> 3;
  t.last_strip = tile_divisor((tiles_m & 7) != 0 ? tiles_m & 7 : 1);
  return total;
}
// Asks for every line of a product's arguments at once, and for what the first request of an operand tile needs, and waits for them.
// Left alone, each is asked for where it is first used, in four to six waits behind each other, and the lines are in no cache
// when a launch begins: 16 iterations of 784-300-100-10 in fp32, eight workers, 655 -> 631 us, of 1000-500-300-37, six
// workers, 665 -> 636 us.
__device__ __forceinline__ void fetch_args(const GemmArgs& p) {
  static_assert(sizeof(GemmArgs) <= 5 * 64, "a word of every 64 bytes");
  const int* w = reinterpret_cast<const int*>(&p);
  asm volatile("" :: "s"(w[0]), "s"(w[16]), "s"(w[32]), "s"(w[48]), "s"(w[sizeof(GemmArgs) / 4 - 1]),
               "s"(p.a), "s"(p.a_gs), "s"(p.lda), "s"(p.b), "s"(p.b_gs), "s"(p.ldb), "s"(p.M), "s"(p.N), "s"(p.Kc),
               "s"(p.place.first.mul), "s"(p.place.second.mul), "s"(p.place.order), "s"(p.order));
}
struct TileAt { int g, m0, n0, split, n_splits; };         // worker; split: contraction range of n_splits
template <int BM, int BN> __device__ __forceinline__ TileAt tile_at(const GemmArgs& p, int block) {
  const TilePlace& t = p.place;
  TileAt r;
  const int xcd = block & 7;
  int idx = xcd * t.xcd_tiles + min(xcd, t.xcd_extra) + (block >> 3);
  r.n_splits = 1 << t.split_shift;
  r.split = idx & (r.n_splits - 1);
  idx >>= t.split_shift;
  const int q = quotient(t.first, idx), in = idx - q * (int)t.first.d;
  int tm, tn;
  if (t.order == 2) {                                      // strip q, `high` tiles high
    TileDivisor high = t.second;
    if (q == t.whole_strips) high = t.last_strip;
    tn = quotient(high, in);
    tm = 8 * q + in - tn * (int)high.d;
    r.g = 0;
  } else {
    const int of = t.order == 1 ? q : in, u = quotient(t.second, of), v = of - u * (int)t.second.d;
    tm = t.order == 1 ? in : u;
    tn = t.order == 1 ? u : v;
    r.g = t.order == 1 ? v : q;
  }
  r.g = worker_of(p.order, r.g);
  r.m0 = tm * BM;
  r.n0 = tn * BN;
  return r;
}
// Its contraction range [k_lo, k_lo + Kc): whole tiles per split.
template <int BK> __device__ __forceinline__ void contraction_range(const GemmArgs& p, const TileAt& t, int* k_lo, int* Kc) {
  *Kc = p.Kc;
  *k_lo = 0;
  if (t.n_splits > 1) {
    const int per = (((p.Kc + BK - 1) / BK + t.n_splits - 1) >> p.place.split_shift) * BK;
    *k_lo = t.split * per;
    *Kc = max(0, min(p.Kc - *k_lo, per));
    if (*Kc == 0) *k_lo = 0;
  }
}

// Epilogue of a batch-row product (DX: backward-data, otherwise forward): 16 bytes of output per thread, the same columns in
// every pass over the rows.  Bias and phi' operand are requested before the output tile is
// collected in LDS, so that a workgroup ends on one memory latency instead of one per pass (16 iterations of six workers of
// 1000-500-300-37 728 -> 716 us; of eight of 4096-4096-4096-4096-1000 at interval 1 8766 -> 8681 us).
// The instruction cache is shared by the launches of an iteration, and what a launch runs has to be fetched again when they exceed
// it (0.6 to 1 us per launch): a kernel holds one of the two epilogues, and tanh, 8 of which are 3 KB, once and not per pass.
// In fp32 16 bytes are four columns, so that all threads of a 32 x 32 tile have some: with eight, half of them were idle beside
// tanh (16 iterations of eight workers of 784-300-100-10 631 -> 605 us).
template <typename T, int BM, int BN, int NTHR, bool DX> struct RowsEpilogue {
  using E = typename T::elem;
  static constexpr int C = T::kBf16 ? 8 : 4;               // columns per thread
  static constexpr int VPR = BN / C, ROWS = NTHR / VPR, NV = (BM + ROWS - 1) / ROWS;
  using Aux = std::conditional_t<T::kBf16, u16x8_t, f32x4_t>;
  static constexpr int NH = DX ? NV : 1;
  int r0, c, m0, n;                                        // first row and column in the tile; tile's first row; column
  f32x4_t b[C / 4];                                        // bias
  Aux h[NH];                                               // phi' operand

  __device__ __forceinline__ RowsEpilogue(int m0_, int n0, int tid)
      : r0(tid / VPR), c(C * (tid % VPR)), m0(m0_), n(n0 + C * (tid % VPR)) {}
  __device__ __forceinline__ void request(const GemmArgs& p, int g) {
    const int nc = min(n, (p.out_cols - 1) & ~(C - 1));       // copies past the operands, never stored
    if constexpr (DX) {
      const E* aux = reinterpret_cast<const E*>(p.aux) + (size_t)g * p.aux_gs + (size_t)m0 * p.ldaux;
#pragma unroll
      for (int q = 0; q < NV; ++q)
        h[q] = *reinterpret_cast<const Aux*>(aux + (__umul24((uint32_t)min(q * ROWS + r0, p.M - 1 - m0), (uint32_t)p.ldaux) +
                                                    (uint32_t)nc));
    } else if (biased(p)) {
      const float* bias = p.src + (size_t)g * p.src_gs + p.b_off + nc;
#pragma unroll
      for (int e = 0; e < C / 4; ++e) b[e] = *reinterpret_cast<const f32x4_t*>(bias + 4 * e);
    }
  }
  // partial sums of a split contraction carry no bias: the loss head adds it once
  __device__ static __forceinline__ bool biased(const GemmArgs& p) { return p.k_splits <= 1; }
  // c_read(r, c): four floats of the output tile.  Padding columns [N, out_cols) are written as zeros.
  template <typename F> __device__ __forceinline__ void store(const GemmArgs& p, int g, int split, F&& c_read) const {
    if constexpr (DX) {
      if (p.act == PRSGD_TANH) passes(p, g, split, c_read, [&](float (&z)[C], int q) __attribute__((always_inline)) { times_slope(z, q, PRSGD_TANH); });
      else passes(p, g, split, c_read, [&](float (&z)[C], int q) __attribute__((always_inline)) { times_slope(z, q, PRSGD_RELU); });
    } else if (p.epi == EPI_FWD_HIDDEN && p.act == PRSGD_TANH) {
#pragma unroll 1
      for (int q = 0; q < NV; ++q)
        pass(p, g, split, q, c_read, [&](float (&z)[C], int) __attribute__((always_inline)) {
#pragma unroll
          for (int e = 0; e < C; ++e) z[e] = tanhf(z[e]);
        });
    } else {
      passes(p, g, split, c_read, [&](float (&z)[C], int) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < C; ++e) z[e] = p.epi == EPI_FWD_HIDDEN ? act_fwd(z[e], PRSGD_RELU) : z[e];
      });
    }
  }

 private:
  __device__ __forceinline__ void times_slope(float (&z)[C], int q, int act) const {
#pragma unroll
    for (int e = 0; e < C; ++e) {
      if constexpr (T::kBf16) z[e] *= act_bwd_from_h(bf16_to_f32(h[q][e]), act);
      else z[e] *= act_bwd_from_h(h[q][e], act);
    }
  }
  template <typename F, typename A>
  __device__ __forceinline__ void passes(const GemmArgs& p, int g, int split, F&& c_read, A&& apply) const {
#pragma unroll
    for (int q = 0; q < NV; ++q) pass(p, g, split, q, c_read, apply);
  }
  template <typename F, typename A>
  __device__ __forceinline__ void pass(const GemmArgs& p, int g, int split, int q, F&& c_read, A&& apply) const {
    const int r = q * ROWS + r0, m = m0 + r;
    if (r >= BM || m >= p.M || n >= p.out_cols) return;
    float z[C];
#pragma unroll
    for (int e = 0; e < C; e += 4) {
      const f32x4_t v = c_read(r, c + e);
#pragma unroll
      for (int x = 0; x < 4; ++x) z[e + x] = v[x];
    }
    if (!DX && biased(p)) {
#pragma unroll
      for (int e = 0; e < C; ++e) z[e] += b[e / 4][e % 4];
    }
    apply(z, q);
#pragma unroll
    for (int e = 0; e < C; ++e) z[e] = n + e < p.N ? z[e] : 0.0f;
    const size_t base = (size_t)g * p.out_gs + (size_t)m0 * p.ldo;
    const uint32_t o = __umul24((uint32_t)r, (uint32_t)p.ldo) + (uint32_t)n;
    if (T::kBf16 && (DX || p.epi != EPI_FWD_LOGITS)) {
      Aux v;
#pragma unroll
      for (int e = 0; e < C; ++e) v[e] = f32_to_bf16_rne(z[e]);
      *reinterpret_cast<Aux*>(reinterpret_cast<uint16_t*>(p.out) + base + o) = v;
    } else {
      float* op = reinterpret_cast<float*>(p.out) + base + (!DX && p.epi == EPI_FWD_LOGITS ? (size_t)split * p.split_stride : 0) + o;
#pragma unroll
      for (int e = 0; e < C; e += 4) *reinterpret_cast<f32x4_t*>(op + e) = (f32x4_t){z[e], z[e + 1], z[e + 2], z[e + 3]};
    }
  }
};

// Products whose workgroups have requesting wavefronts (kernels_gemm_rows.hip), and their tiles in flight: 128-row tiles, the smaller ones.
// Four of these cover the latency of a workgroup that has its compute unit to itself (per iteration, 5 workers of
// 640-1024-448-960-29, 18 rows: three 53.8 us, four 51.1, five or six 51.0; 6 of 1000-500-300-37, 100 rows: 36.2, 35.3, 35.6).
constexpr int kFedStages = 3, kFedSmallStages = 4;
hipError_t launch_gemm_fwd_fed(const GemmArgs& p, int n_groups, int bm, int bn, hipStream_t s);
hipError_t launch_gemm_dx_fed(const GemmArgs& p, int n_groups, int bm, int bn, hipStream_t s);

// Launches KERNEL (WAVES wavefronts per workgroup) with one workgroup per tile of BM x BN.
template <typename T, int BM, int BN, int WK, int S, int WAVES, void (*KERNEL)(GemmArgs)>
static hipError_t launch_tiles(GemmArgs p, int n_groups, hipStream_t s) {
  if (p.M <= 0 || p.N <= 0 || n_groups <= 0) return hipSuccess;
  constexpr size_t kLds = gemm_lds_bytes<T, BM, BN, WK, S>();
  static_assert(kLds <= 160 * 1024, "LDS of a compute unit");
  // the tiles can exceed the 64 KB default; setting the limit twice is harmless
  static std::atomic<bool> configured{false};
  if (!configured.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
    if (e != hipSuccess) return e;
    configured.store(true, std::memory_order_release);
  }
  if (p.k_splits > 1 && p.epi != EPI_FWD_LOGITS) return hipErrorInvalidValue;
  // Weights of a worker's own that one row of tiles covers are read once and not kept: read into the last-level cache, they made it write
  // back what the backward kernels had left there.  8 x 4096-4096-4096-4096-1000, 128 rows: forward launches of the second and third layer 91
  // and 68 us, 58 and 57 so.  Most of that goes to the launches that still read through the cache, which now find the lines to be written
  // back: backward kernels of the layers behind the first 200 -> 208 us on average, the logits product (two rows of tiles) 28 -> 35, the loss
  // head with its draw 9 -> 12; 16 iterations 16043 -> 15850 us.  16 x 3072-1024-1024-10, 64 rows, second
  // layer 15.2 -> 11.3.  Weights that several rows of tiles or all workers read again stay: 8 x (512 x 3072) x 1024 31 us, 38 non-temporal.
  p.b_once = p.streaming && p.b_gs != 0 && p.M <= BM ? 1 : 0;
  const int tiles = place_tiles(&p, BM, BN, n_groups);
  hipLaunchKernelGGL(KERNEL, dim3((unsigned)tiles), dim3(64 * WAVES), kLds, s, p);
  return hipGetLastError();
}

}  // namespace prsgd
