// Internal declarations shared by the HIP translation units of libprsgd (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "prsgd.h"

namespace prsgd {

constexpr int kThreads = 256;        // 4 wavefronts of 64 lanes per workgroup
constexpr int kWave = 64;
constexpr int kMaxBatch = 4096;
constexpr int kMaxLsqDim = 8192;

// Device layout of one replica x_i (floats).  An MLP replica is
//   [W_1][b_1][W_2][b_2]...   W_l stored row-major as [d_{l-1}][ld_l], ld_l = d_l rounded up
// to a multiple of 8 so that every row starts 32-byte aligned; each segment starts on a
// 64-float boundary.  All padding holds zeros and stays zero under update and average.
struct Layout {
  int  n_layers;                     // L (0 for least squares)
  int  d[PRSGD_MAX_DIMS];            // logical widths d_0..d_L
  int  ld[PRSGD_MAX_DIMS];           // padded widths
  long w_off[PRSGD_MAX_DIMS];        // offset of W_l, index l-1
  long b_off[PRSGD_MAX_DIMS];        // offset of b_l, index l-1
  long m;                            // logical parameter count
  long m_pad;                        // replica stride in floats
};

enum GemmEpilogue {
  EPI_FWD_HIDDEN = 0,   // out = T(phi(acc + bias))
  EPI_FWD_LOGITS = 1,   // out = float(acc + bias)
  EPI_DX = 2,           // out = T(acc * phi'(aux))
  EPI_DW_FUSED = 3,     // W <- W - lr * acc (and bf16 shadow), b likewise from column sums
  EPI_DW_GRAD = 4,      // G_W = acc, G_b = column sums
};

// Where the tiles of a product stand among its workgroups (gemm_tile.h); filled in by the launcher.
struct TileDivisor { uint32_t mul, shift, d; };
struct TilePlace {
  int xcd_tiles, xcd_extra;           // tiles of every XCD, XCDs with one more
  int split_shift, order;             // contraction ranges (their logarithm); 0 by group, 1 by column tile, 2 in strips
  TileDivisor first, second, last_strip;
  int whole_strips;
};

// One grouped matrix product: for every group (replica) g
//   C_g[m][n] = sum_c A_g(m, c) * B_g(n, c),   m < M, n < N, c < Kc
// followed by an epilogue.  Operand element (r, c) sits at base + g*gs + r*ld + c when the
// operand is contraction-contiguous, or at base + g*gs + c*ld + r when it is transposed.
struct GemmArgs {
  const void* a; long a_gs; int lda;
  const void* b; long b_gs; int ldb;
  int M, N, Kc;
  TilePlace place;
  int epi;
  int streaming;                      // weights far exceed the caches: non-temporal accesses
  int b_once;                         // ... and every element of B is read by one workgroup only (filled in by the launcher)
  int act;                            // PRSGD_TANH | PRSGD_RELU
  float lr;
  float* vel; float mu;               // update with momentum: velocities, replica stride m_pad (nullptr: without)
  // parameters / gradients (fp32, replica stride m_pad), bf16 shadow of the parameters
  float* params; float* grads; uint16_t* shadow; long p_gs;
  // where the old parameters (forward: the bias; update: weights and bias) are read from: the
  // replicas, or (right after a restart whose broadcast was skipped) the shared node average with
  // stride 0
  const float* src; long src_gs;
  long w_off, b_off; int ldw;
  // activation-like output (element type T, or float for logits) and auxiliary input
  void* out; long out_gs; int ldo; int out_cols;
  const void* aux; long aux_gs; int ldaux;
  const int* order;                   // Algorithm 3: group g is worker order[g] (nullptr: worker g)
  // logits product of a narrow last layer: the contraction is cut into k_splits ranges, split s
  // writes its partial sums (no bias) at out + s * split_stride; the loss head adds them up
  int k_splits; long split_stride;
};
// contraction splits the forward launcher wants for the logits product described by p
int gemm_logit_splits(const GemmArgs& p, int n_groups, bool bf16);
constexpr int kMaxLogitSplits = 4;

enum KernelKind {
  KK_GATHER = 0, KK_FWD, KK_LOSS, KK_DX, KK_DW, KK_UPDATE, KK_AVERAGE, KK_MEAN, KK_BROADCAST,
  KK_LSQ, KK_FUSED2, KK_BWD, KK_RESTART_MEAN, KK_STEP_MEAN, KK_BWD_FIRST, KK_REFRESH, KK_COUNT
};

// Fused backward step of one layer with bf16 operands (kernels_bwd.hip): weight gradient, local
// update of W_l and b_l, and the delta of the layer below, in one pass over W_l.
struct BwdArgs {
  const uint16_t* h; long h_gs; int ldh;        // H_{l-1} [N][B][ldh]
  const uint16_t* d; long d_gs; int ldd;        // D_l     [N][B][ldd]
  float* params; uint16_t* shadow; long p_gs;   // fp32 master and bf16 shadow, replica stride
  const float* src; long src_gs;                // where the old parameters are read from: the
                                                // replicas (src_gs = p_gs) or the shared node
                                                // average right after a restart (src_gs = 0)
  long w_off, b_off; int ldw;
  uint16_t* dx; long dx_gs; int lddx;           // D_{l-1} [N][B][lddx]; nullptr for the first layer
  int B, K, Nn;                                 // minibatch rows, d_{l-1}, d_l
  int n_groups, act, streaming;
  float lr;
  float* vel; float mu;                         // momentum buffers [N][p_gs] (nullptr = plain SGD)
  const int* order;                             // Algorithm 3: group g is worker order[g] (nullptr: worker g)
  // first layer only (kernels_bwd_first.hip): minibatch of the next iteration [N][B][ldx] and
  // where its first hidden activation goes [N][B][ldhn]
  const uint16_t* x_next; long x_gs; int ldx;
  uint16_t* h_next; long hn_gs; int ldhn;
};
bool bwd_fused_supported(int batch);
// The kernel's walk over the columns leaves most of the chip idle: the layer's products apart are faster
// if, over the layers this holds for, their number and the widest of them say so.
bool bwd_products_apart(const BwdArgs& p);
bool bwd_apart_pays(int n_layers, int widest, int batch);
hipError_t launch_bwd_fused(const BwdArgs& p, hipStream_t s);
// Layer 1: backward step fused with the next iteration's forward product of that layer.
bool bwd_first_fwd_same_bits(const BwdArgs& p);     // layers that it takes with the bits of the walk over the weights
bool bwd_first_fwd_applies(const BwdArgs& p);
hipError_t launch_bwd_first_fwd(const BwdArgs& p, hipStream_t s);

// Epoch kernel for fp32 MLPs with one hidden layer (kernels_fused2.hip).
struct Fused2Plan {
  int KBI, NT, MT;     // template shape: W_1 row blocks per wavefront, hidden tiles, batch tiles
  int P;               // workgroups per worker
  int d2p, KB;         // padded class count, 16-column blocks of the gathered batch
  int momentum;        // 1: the variant that carries velocities
  int shares;          // places for partial pre-activations in LDS
  bool pinned_fits;    // all teams resident with each on one XCD
};
struct Fused2Args {
  const float* features; const int32_t* labels;
  float* params; long m_pad; long w1_off, b1_off, w2_off, b2_off; int ld1, ld2;
  const float* src; long src_stride;   // starting point of every worker: its replica, or the shared
                                       // node average (stride 0) right after a restart
  int n_workers, P, shares, pinned, d0, d1, d2, batch; long rows; int log2n;
  int act; float lr; uint64_t seed; uint64_t t0; int k;
  const int* worker_steps;       // Algorithm 3 step counts (nullptr: every worker takes k steps)
  int interval;                  // > 0: restarts inside the launch
  float* exchange;               // [N][P] slices on their way, then [P] averages (fused2_exchange_floats)
  unsigned long long* part;      // [N][P][B d2] partial logits with the number of their iteration, in two hops with [N][B d2]
                                 // sums behind them; two such sets, or one where scratch is short and two hops allow it
  bool spare_part; unsigned part_odd;   // ... and the slots from a set to that of odd iterations, 0 for a single one
  int share, hop_groups;         // two hops: floats that a member sums, lanes for each (these three set by launch_fused2)
  unsigned int* sync;            // [N][32]: iterations exchanged so far (word 1); [32]: abort flag, restarts so far;
                                 // with restarts inside the launch also [2][8] copies of a flag byte per workgroup
  unsigned int spin_limit;       // polls before a member gives up
  float* row_loss; int32_t* idx;
  float* vel; float mu;          // momentum buffers [N][m_pad] (nullptr = plain SGD)
};
constexpr unsigned int kFused2SpinLimit = 1u << 22;   // default bound of the team barrier's wait
size_t fused2_lds_bytes(const Fused2Plan& pl);
constexpr int kFused2MaxMembers = 1024;      // workgroups of 512 threads that 256 compute units hold
// bytes between the copies of the flags: a line each, on different memory channels
__host__ __device__ constexpr int fused2_flag_stride(int members) { return (members + 255) / 256 * 256 + 256; }
size_t fused2_part_slots(int n_workers, int d1, int d2, int batch, bool spare);
size_t fused2_exchange_floats(int n_workers, int d0, int d1, int d2);
bool fused2_shape(int n_workers, int d0, int d1, int d2, int batch, bool momentum);
bool fused2_plan(int n_workers, int d0, int d1, int d2, int batch, bool momentum, Fused2Plan* pl);
hipError_t launch_fused2(const Fused2Plan& pl, Fused2Args args, bool pinned, hipStream_t s);
// Workgroups that n_workers teams put on the fullest of the eight XCDs: pinned, a team stays on XCD i mod 8; spread, the
// workgroups are dealt to the XCDs in turn.
constexpr long xcd_workgroups(long n_workers, long team, bool pinned) {
  return pinned ? (n_workers + 7) / 8 * team : (n_workers * team + 7) / 8;
}
const char* kernel_kind_name(int kind);

// ---- launchers (each returns the hipError_t of the launch) --------------------------------
hipError_t launch_gemm_fwd(const GemmArgs& p, int n_groups, bool bf16, hipStream_t s);
hipError_t launch_gemm_dx(const GemmArgs& p, int n_groups, bool bf16, hipStream_t s);
// Tile and LDS bytes per workgroup of the batch-row product [rows] x [cols] of n_groups workers.
void gemm_rows_shape(int rows, int cols, int n_groups, bool bf16, int* tile_rows, int* tile_cols, size_t* lds_bytes);
// Weight-gradient products of up to kMaxGemmSet layers in one launch.
constexpr int kMaxGemmSet = 4;
hipError_t launch_gemm_dw(const GemmArgs* ps, int n, int n_groups, bool bf16, hipStream_t s);

// Minibatch draw of iteration t: rows of the workers' shards copied into the batch buffer.
struct GatherArgs {
  const float* features; const int32_t* labels;
  void* xb; int32_t* yb; int32_t* idx;        // batch rows [N][B][ld0], labels and row indices [N][B]
  int batch, d0, ld0; long rows; int log2n;
  uint64_t seed, t;
  const int* order; int workers;              // Algorithm 3: the workers order[0 .. workers) draw (nullptr: 0 .. workers)
  int once;                                   // the shards exceed the caches: their rows are read non-temporally
};
GatherArgs gather_args(const float* features, const int32_t* labels, void* xb, int32_t* yb, int32_t* idx,
                       int batch, int d0, int ld0, long rows, uint64_t seed, int64_t t, const int* order, int workers);
hipError_t launch_gather(const GatherArgs& a, bool bf16, hipStream_t s);
hipError_t launch_sample_indices(uint64_t seed, int n_workers, int batch, long rows, int64_t t_first,
                                 int n_steps, int32_t* out, hipStream_t s);
// Of the n_workers workers order[0 .. n_workers) (nullptr: 0 .. n_workers).  next != nullptr: the launch also gathers that
// minibatch, of as many workers at most
hipError_t launch_softmax_xent(const float* logits, int n_parts, long part_stride, const float* bias,
                               long bias_gs, const int32_t* yb, void* delta, float* row_loss,
                               int n_workers, int batch, int n_classes, int ldc, bool bf16,
                               const int* order, const GatherArgs* next, hipStream_t s);
// Narrow head (at most 64 classes): logits product, softmax and delta in one launch; below != nullptr: and the delta of the
// layer below, D_{L-1} [N][B][ld]
struct HeadDelta { void* out; long gs; int ld, act; };
bool softmax_narrow_applies(int n_classes, int ldc, int k_dim, bool bf16);
bool softmax_narrow_delta_pays(int ldc, int k_dim, int head_blocks, bool bf16);
int softmax_narrow_blocks(int n_workers, int batch);         // workgroups of a narrow head
hipError_t launch_softmax_xent_narrow(const void* h, long h_gs, int ldh, int k_dim, const void* w,
                                      long w_gs, const float* bias, long bias_gs, const int32_t* yb,
                                      void* delta, float* row_loss, int n_workers, int batch, int n_classes,
                                      int ldc, bool bf16, const int* order, const GatherArgs* next,
                                      const HeadDelta* below, hipStream_t s);
hipError_t launch_loss_mean(const float* row_loss, float* losses, int n_workers, int batch,
                            hipStream_t s);

hipError_t launch_average(float* params, uint16_t* shadow, long m_pad, int n_workers, bool streaming,
                          hipStream_t s);
hipError_t launch_mean(const float* params, float* out, uint16_t* out_shadow, long m_pad, int n_workers,
                       bool streaming, hipStream_t s);
hipError_t launch_broadcast(const float* src, float* params, uint16_t* shadow, long m_pad,
                            int n_workers, hipStream_t s);
hipError_t launch_refresh_shadow(const float* params, uint16_t* shadow, long count, hipStream_t s);
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s);
hipError_t launch_update(float* x, const float* g, uint16_t* shadow, size_t count, float lr,
                         hipStream_t s);
hipError_t launch_momentum_update(float* x, float* v, const float* g, uint16_t* shadow, size_t count,
                                  float lr, float mu, hipStream_t s);
hipError_t launch_fill_zero(float* x, size_t count, hipStream_t s);
hipError_t launch_update_workers(float* x, const float* g, uint16_t* shadow, long m_pad, const int* order,
                                 int n_workers, float lr, hipStream_t s);
hipError_t launch_store_ints(int* dst, const int* src_host, int count, int largest, hipStream_t s);

// Least squares: k local iterations of every worker (kernels_lsq.hip).
struct LsqArgs {
  const float* features; const float* targets;
  const float* src; long src_stride;     // starting points: the replicas, or the shared node average (stride 0)
  float* params; float* velocity; float mu; long m_pad;
  float* losses; int32_t* idx;
  int n_workers, d; long rows; int log2n; int batch;    // log2n is filled in by the launcher
  float lr; uint64_t seed, t0; int k;
  const int* worker_steps;               // Algorithm 3 step counts (nullptr: every worker takes k steps)
  int interval;                          // > 0: restarts inside the launch (lsq_restarts_in_launch)
  unsigned long long* exchange;          // [2][N][d] published points with the number of their restart
  unsigned int* sync;                    // restarts published so far
  unsigned int* abort_flag;
  unsigned int spin_limit;               // polls before a workgroup gives up
};
constexpr int kLsqMaxTeam = 64;          // workgroups that wait for each other: a quarter of the compute units
constexpr long kLsqMaxExchange = 32768;  // floats that everybody reads at a restart (64 workers of 512: 6 us)
bool lsq_restarts_in_launch(int n_workers, int d, int batch);
size_t lsq_exchange_bytes(int n_workers, int d);
hipError_t launch_lsq_steps(LsqArgs p, hipStream_t s);

// ---- small device helpers ------------------------------------------------------------------
// Asks for every 64-byte line of the first BYTES of a kernel's arguments at once and waits for them.  They are in no cache when a
// launch begins, and left alone each line is asked for where it is first used, one wait behind the other.
template <size_t BYTES> __device__ __forceinline__ void fetch_kernel_args() {
  constexpr int L = (int)(BYTES / 4) - 1;                  // last word
  static_assert(L / 16 < 5, "a word of every line");
  const auto* w = (const __attribute__((address_space(4))) int*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" :: "s"(w[0]), "s"(w[L < 16 ? L : 16]), "s"(w[L < 32 ? L : 32]), "s"(w[L < 48 ? L : 48]), "s"(w[L]));
}
// Worker of group g (Algorithm 3: order[g]), by a scalar load.  As a vector load it put the worker and every address behind it into vector
// registers, also where order is null: 6 workers of 3456-704-665-384-67, 128 rows, first layer 58 -> 66 us.
__device__ __forceinline__ int worker_of(const int* order, int g) {
  return order == nullptr ? g : ((const __attribute__((address_space(4))) int*)order)[g];
}
// Round to nearest even on the conversion instruction (two values per v_cvt_pk_bf16_f32; a NaN stays a
// NaN, infinities and denormals are kept).  Written out in integer operations, with the NaN case apart,
// the compiler made a divergent branch of every element: 11 instructions each, 176 of the 390 of one
// tile of the first layer's backward kernel.
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}
__device__ __forceinline__ uint32_t f32x2_to_bf16x2_rne(float lo, float hi) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  return __uint_as_float(((uint32_t)h) << 16);
}

// ---- bf16 MFMA operand fragments out of LDS ----------------------------------------------------
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

// Fragment of lane (r = lane % 32, kb = lane / 32) for the kk-th 16-deep contraction slice of a
// tile stored [row][c] (contraction index contiguous): one 16-byte read.
__device__ __forceinline__ bf16x8_t frag_contig(const uint16_t* lds, int stride, int row_block, int kk,
                                                int lane) {
  const u16x8_t u = *reinterpret_cast<const u16x8_t*>(lds + (row_block + (lane & 31)) * stride + kk * 16 +
                                                      (lane >> 5) * 8);
  return __builtin_bit_cast(bf16x8_t, u);
}
// The same fragment of a tile stored [c][row] (contraction index is the LDS row), read with the
// LDS transpose load (ds_read_b64_tr_b16): inside each group of 16 lanes, lane r supplies the
// address of a 4-element row M[r] and lane i receives M[4j + i/4][i%4], j = 0..3.  Addressing
// lane r at (c = c0 + r/4, rows 4*(r%4)..+3) therefore hands lane i the four consecutive c of
// row i: a 4(c) x 16(row) block transposed in flight.  Two such loads give the eight contraction
// elements of the fragment.
__device__ __forceinline__ bf16x8_t frag_trans(const uint16_t* lds, int stride, int row_block, int kk,
                                               int lane) {
  typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4_t;
  typedef __attribute__((address_space(3))) bf16x4_t* lds_bf16x4_ptr;
  const int g = lane >> 4, r = lane & 15;
  const int c = kk * 16 + 8 * (g >> 1) + (r >> 2);
  const int row = row_block + 16 * (g & 1) + 4 * (r & 3);
  const uint16_t* p = lds + c * stride + row;
  const bf16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p));
  const bf16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p + 4 * stride));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// ---- tiles requested straight into LDS ---------------------------------------------------------
// 64 x 16 bytes from base + per-lane offset to LDS [lds_any, lds_any + 1024), lane order.  Not visible to the
// compiler's wait counts: a kernel that uses it waits by itself, and everything the compiler waits for on its
// own is then waited for at least as long as it needs.  m0 is a reserved register, which cannot be listed as
// clobbered: nothing else in such a kernel may use it.
// NT: non-temporal, for what is read once and should leave the caches to the rest.
template <bool NT = false>
__device__ __forceinline__ void load_to_lds(const void* base_any, uint32_t lane_off, uint32_t lds_any) {
  // both are the same in every lane; said explicitly, they end up in scalar registers
  const uint64_t u = (uint64_t)(uintptr_t)base_any;
  const uint64_t base = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)u) |
                        ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32)) << 32);
  const uint32_t lds_off = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_any);
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 :: "s"(lds_off), "v"(lane_off), "s"(base) : "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_off), "v"(lane_off), "s"(base) : "memory");
}
// The same with 4 bytes per lane: any alignment of the source, 256 consecutive bytes of LDS.
__device__ __forceinline__ void load_dword_to_lds(const void* base_any, uint32_t lane_off, uint32_t lds_any) {
  const uint64_t u = (uint64_t)(uintptr_t)base_any;
  const uint64_t base = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)u) |
                        ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32)) << 32);
  const uint32_t lds_off = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_any);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
               :: "s"(lds_off), "v"(lane_off), "s"(base) : "memory");
}
// 64 x 16 bytes from an address of every lane's own.
__device__ __forceinline__ void load_x4_to_lds(uint64_t lane_addr, uint32_t lds_any) {
  const uint32_t lds_off = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_any);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :: "s"(lds_off), "v"(lane_addr) : "memory");
}
// ... and 4 bytes from an address of every lane's own.
__device__ __forceinline__ void load_lane_dword_to_lds(uint64_t lane_addr, uint32_t lds_any) {
  const uint32_t lds_off = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_any);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
               :: "s"(lds_off), "v"(lane_addr) : "memory");
}
// Workgroup barrier that leaves requests into LDS in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// A tile of 16-byte pieces cannot be padded on its way, so bank conflicts are avoided by permuting WHICH 16 bytes a lane
// requests.  [c][row], contraction index c the LDS row of ROW_BYTES: the transpose read takes 64 bytes of
// four consecutive c at a time, so the 64-byte segments of row c are exchanged (segment s at s ^ lds_seg_xor(c))
// such that the four fall on different banks.
template <int ROW_BYTES> __device__ __forceinline__ int lds_seg_xor(int c) {
  if (ROW_BYTES <= 64) return 0;
  return ROW_BYTES == 128 ? (c >> 1) & 1 : c & 3;
}
// bf16 fragment of a 32-row block out of such a tile (the lane addresses of frag_trans).
template <int ROW_BYTES>
__device__ __forceinline__ bf16x8_t lds_frag_trans(const unsigned char* tile, int block, int kk, int lane) {
  typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4_t;
  typedef __attribute__((address_space(3))) bf16x4_t* lds_bf16x4_ptr;
  const int g = lane >> 4, r = lane & 15;
  const int c = kk * 16 + 8 * (g >> 1) + (r >> 2);
  const unsigned char* p = tile + c * ROW_BYTES + ((block ^ lds_seg_xor<ROW_BYTES>(r >> 2)) << 6) + 32 * (g & 1) +
                           8 * (r & 3);
  const bf16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p));
  const bf16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p + 4 * ROW_BYTES));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
// [row][c] with 128-byte rows: the 16-byte chunk q of row r stands at lds_chunk(r, q), so that eight consecutive
// rows read one chunk each from all banks.
__device__ __forceinline__ int lds_chunk(int r, int q) { return q ^ (r & 7); }
__device__ __forceinline__ bf16x8_t lds_frag_contig(const unsigned char* tile, int block, int kk, int lane) {
  const int r = lane & 31, kb = lane >> 5;
  return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u16x8_t*>(tile + (block * 32 + r) * 128 +
                                                                       (lds_chunk(r, 2 * kk + kb) << 4)));
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two 32x32->64 multiplies
// with the key advanced by the Weyl constants between rounds.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t out[4]) {
  constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) { k0 += W0; k1 += W1; }
    const uint32_t hi0 = __umulhi(M0, c0), lo0 = M0 * c0;
    const uint32_t hi1 = __umulhi(M1, c2), lo1 = M1 * c2;
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Row drawn by worker `worker` at iteration t for minibatch slot j (top log2(n) bits).
__device__ __forceinline__ int32_t sample_row(uint64_t seed, uint32_t worker, uint64_t t, uint32_t j,
                                              int log2n) {
  uint32_t w[4];
  philox4x32_10(j >> 2, (uint32_t)t, (uint32_t)(t >> 32), worker, (uint32_t)seed,
                (uint32_t)(seed >> 32), w);
  const uint32_t sel = j & 3u;
  const uint32_t word = sel == 0 ? w[0] : sel == 1 ? w[1] : sel == 2 ? w[2] : w[3];
  return log2n == 0 ? 0 : (int32_t)(word >> (32 - log2n));
}

}  // namespace prsgd
