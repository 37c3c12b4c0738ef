// One launch = a whole epoch of local iterations (Algorithm 1, eq. 3), or a whole run with its restarts, for small
// fp32 MLPs with one hidden layer, the latency-bound regime where a chain of per-layer kernels is dominated
// by launch gaps and by re-reading weights that would fit on chip.
//
// Workers never exchange anything inside an epoch (paragraph below Algorithm 1), so the only
// coupling is inside one worker's own forward/backward pass.  Worker i is served by a TEAM of P
// workgroups; workgroup j of the team owns the W hidden units from j W on:
//   - its [d_0][W] slice of W_1 lives in REGISTERS for the whole launch, laid out so that the
//     MFMA B-operand registers of the forward product are, element for element, the accumulator
//     registers of the weight-gradient product: eq. (3) for W_1 is a register-to-register fma;
//   - its slices of b_1 and W_2 (and a private copy of b_2) live in LDS;
//   - a wavefront owns pairs of 16-row blocks of the slice, and with them the 32 columns of the minibatch in
//     LDS that the forward and the weight-gradient product of those rows read: nobody else touches
//     them, so the wavefront requests the next minibatch into their place as soon as it has multiplied them, and waits
//     for nothing but its own requests before the next forward product;
//   - one exchange per iteration: every member publishes its partial logits, each float with the iteration's number in one
//     8-byte store, and polls the others' data itself (no arrival counter, no second trip for the data),
//     summing the P partials in fixed order; everything after that (softmax, both delta blocks, dW_2, db, dW_1)
//     is local to the slice.  Two sets of slots alternate: a member can only publish iteration t + 2 after
//     everybody has read iteration t.  Where the partials are summed in two hops one set would do: nobody publishes partials of t + 1
//     before it has all sums of t, which stand for everybody's partials of t read, nor sums before all partials of t + 1.  It is
//     taken where scratch is short; two are faster (4 x (784-256-10), 32 rows, 9.8 and 10.3 us per iteration).
// The last wavefront draws the rows of the iteration after the next while the others wait for the exchange, and touches one
// word per line of the member's share of them, so that the requests of all members find them in the L2.
// Teams of different workers meet only at a restart.  Summation orders are fixed, so a run is bit-reproducible.
//
// Restarts (`interval` > 0): after every iteration whose number is a multiple of the interval, but the last of
// the call, every workgroup writes its slice into the replicas, all workgroups of the grid together take the node average (each
// a range of the parameters, in the order of the restart kernels) and load their slices of it: two grid-wide
// meetings over one flag per workgroup, each polled by one wavefront.
//
// Every wait is bounded; giving up raises the abort flag, which ends every workgroup.
//
// What bounds it: latency.  Of the 22,600 cycles of an iteration of 784-256-10 (8 workers, 32 rows) the exchange takes 5,400, the
// two large products 5,700 each (3,500 at the matrix cores' rate; two wavefronts per SIMD, 7 blocks on the busiest), the requests of
// the next minibatch 2,500, the small phases 900 to 1,400 each.  Per iteration, against an arrival counter, partials and minibatch as
// loads of their own and a launch per epoch (widths that are no multiple of 16, or of 4 for the input: against the
// chain of per-layer launches): 784-256-10 with interval 16 12.3 and 10.6 us, 64 workers of 256-128-10 with
// 8 rows, interval 8, 7.8 and 7.2 us, 4 workers of 300-100-10, 20 rows, interval 4, 26.6 and 8.9 us, 30 workers of
// 1023-255-15, 30 rows, 46.7 and 25.6 us.  A restart inside the launch takes 7 us with 0.5 MB of replicas and 14 us
// with 9 MB (the agent-scope traffic of all workgroups), 3 to 5 us less than the end of a launch, the averaging launch and a new
// start.
#include <type_traits>

#include "prsgd_internal.h"

namespace prsgd {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kTT = 512;                      // threads per team member: two wavefronts per SIMD, so
constexpr int kTW = kTT / kWave;              // that the latency-bound phases of one overlap the other's
constexpr int kPollers = kTT - kWave;         // threads that sum the partial logits: all but the drawing wavefront
// Partial logits of a team from which they are summed in two hops: 16 x 320 floats 9,200 cycles in one, 5,400 in two; with 4 x 80 one
// takes 3,000, which a second would double.
constexpr int kTwoHopFloats = 2048;
__host__ __device__ constexpr bool two_hop_exchange(int P, int floats) { return (long)P * floats >= kTwoHopFloats; }
constexpr int kAgentScope = 16;               // buffer access cache policy: the sc1 bit (agent scope)

__device__ __forceinline__ f32x4_t mfma16(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float act2_fwd(float z, int act) {
  return act == PRSGD_TANH ? tanhf(z) : fmaxf(z, 0.0f);
}
__device__ __forceinline__ float act2_bwd(float h, int act) {
  return act == PRSGD_TANH ? (1.0f - h * h) : (h > 0.0f ? 1.0f : 0.0f);
}

// Butterfly over each aligned group of 16 lanes on the data-parallel-primitive path (no LDS round
// trips): every lane of the group ends with the same max / sum.
template <int CTRL> __device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, dpp_move<0xB1>(v));      // quad_perm [1,0,3,2]
  v = fmaxf(v, dpp_move<0x4E>(v));      // quad_perm [2,3,0,1]
  v = fmaxf(v, dpp_move<0x141>(v));     // row_half_mirror
  return fmaxf(v, dpp_move<0x140>(v));  // row_mirror
}
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_move<0xB1>(v);
  v += dpp_move<0x4E>(v);
  v += dpp_move<0x141>(v);
  return v + dpp_move<0x140>(v);
}
__device__ __forceinline__ float agent_load(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_store(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool gave_up(unsigned int* abort_flag, unsigned& polls, unsigned limit) {
  if (++polls <= limit &&
      ((polls & 15) != 0 || __hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0))
    return false;
  __hip_atomic_store(abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// KBI: 16-row blocks of W_1 per wavefront (register budget); NT: 16-column tiles of the hidden
// slice; MT: 16-row tiles of the minibatch; CT: 16-column tiles of the classes.  MOM: momentum form of the local update
// (v <- mu v + G, x <- x - gamma v) with the velocity of the slice held next to the slice.
template <int KBI, int NT, int MT, int CT, bool MOM>
__global__ __launch_bounds__(kTT) void mlp2_epoch_kernel(Fused2Args p) {
  constexpr int W = NT * 16, MR = MT * 16, D2P = CT * 16;
  constexpr int XB = MR * 32;                              // floats of a pair of 16-column blocks of the minibatch
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int n16 = lane & 15, q4 = lane >> 4;

  // team mapping: consecutive workgroups go round-robin to the 8 XCDs.  Pinned: a team stays on one XCD (its
  // partial logits and the members' minibatch then stay in that XCD's L2); the grid is filled up to whole rounds.  Spread: the
  // members of a team follow each other, so that every XCD holds its share of any number of workers.  Per iteration, pinned
  // and spread: 20 x (256-128-10), 8 rows, 5.7 and 6.3 us; 2 x (784-256-10), 32 rows, 11.1 and 11.5 us.
  const int slot = p.pinned ? (int)blockIdx.x >> 3 : (int)blockIdx.x;
  const int team = slot / p.P, j = slot - team * p.P;
  const int i = p.pinned ? ((int)blockIdx.x & 7) + 8 * team : team;
  if (i >= p.n_workers) return;
  const int my_k = p.worker_steps != nullptr ? min(p.worker_steps[i], p.k) : p.k;
  if (my_k <= 0) return;                                   // uniform over the team
  const int members = p.n_workers * p.P, me = i * p.P + j;
  unsigned int* base_slot = p.sync + (size_t)i * 32 + 1;   // one 128-byte line per team
  unsigned int* abort_flag = p.sync + (size_t)p.n_workers * 32;
  unsigned int* restart_base = abort_flag + 1;
  const int flag_stride = fused2_flag_stride(members);
  unsigned char* flags = reinterpret_cast<unsigned char*>(p.sync + (size_t)(p.n_workers + 1) * 32);   // [2][8][flag_stride]
  if (__hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
  const unsigned base = *base_slot;                        // iterations exchanged before this launch
  unsigned restarts = p.interval > 0 ? *restart_base : 0;  // ... and restarts

  const int d0 = p.d0, d1 = p.d1, d2 = p.d2, B = p.batch;
  const int KB = (d0 + 15) / 16, pairs = (KB + 1) / 2;
  // row block kbi of this wavefront: blocks come in pairs, 128 bytes of a row of the minibatch
  auto block = [&](int kbi) __attribute__((always_inline)) { return 2 * (wave + kTW * (kbi >> 1)) + (kbi & 1); };
  const bool rows_x4 = (d0 & 3) == 0;                      // rows of the shard start 16-byte aligned

  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* X = lds;                                          // [pairs][MR][32]  gathered rows in pairs of column blocks
  float* red = X + (size_t)pairs * XB;                     // [shares][MR][W] partial z_1: one per wavefront, or per two
  const int shares = p.shares;
  float* h = red + shares * MR * W;                        // [MR][W]
  float* dl1 = h + MR * W;                                 // [MR][W]
  float* lg = dl1 + MR * W;                                // [MR][D2P]   delta_2
  float* w2 = lg + MR * D2P;                               // [W][D2P]
  float* b1 = w2 + W * D2P;                                // [W]
  float* b2 = b1 + W;                                      // [D2P]
  int* rows = reinterpret_cast<int*>(b2 + D2P);            // [2][MR] rows of iteration t at [t & 1]
  int* ylab = rows + 2 * MR;                               // [2][MR] their labels
  int* flag = ylab + 2 * MR;                               // [4] abort broadcast
  float* dump = reinterpret_cast<float*>(flag + 4);        // [64] what the line-touching loads bring
  float* vw2 = dump + kWave;                               // [W][D2P] velocities (MOM only)
  float* vb1 = vw2 + W * D2P;                              // [W]
  float* vb2 = vb1 + W;                                    // [D2P]
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)lds;

  const float* feat = p.features + (size_t)i * p.rows * d0;
  // Arguments that only the ends of the launch, the restarts and the drawing wavefront need: loaded where they are used, so
  // that the scalar registers are left to the iterations.
  auto cold = []() __attribute__((always_inline)) {
    auto* k = (const __attribute__((address_space(4))) Fused2Args*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(k));
    return k;
  };
  const float inv_b = 1.0f / (float)B;
  bool aborted = false;

  // Element (row, c) of W_2 (a row per hidden unit) and of delta_2 (a row per minibatch row).  Rows of 64 classes are as long as
  // the 64 banks: their 4-class chunks are exchanged by the row, so that 16 rows at one chunk (delta_1) and 4 rows at 16 classes
  // (fragments) fall on different banks.  8 x (256-128-20), 64 rows, 18.4 -> 12.1 us per iteration.
  auto cls = [](int row, int c) __attribute__((always_inline)) {
    if constexpr (CT == 1) return row * D2P + c;
    return row * D2P + (((c >> 2) ^ (((row & 3) << 2) | ((row >> 2) & 3))) << 2 | (c & 3));
  };

  // ---- minibatch ----------------------------------------------------------------------------------
  // Element (row r, column 32 i + c) stands at X[i][r][..] with the eight 4-column chunks of a row exchanged
  // by r / 2, so that the 16 rows of a forward fragment and the elements of a gradient fragment fall on
  // different banks.  Columns from d_0 on stay zero.
  auto x_chunk = [&](int r, int q) { return q ^ ((r >> 1) & 7); };
  // Requests of the rows in `rws`: where this lane's pieces of a row start (16-byte pieces; rows that are not 16-byte
  // aligned go by single words), and one pair of blocks of them.  A compute unit has about a hundred lines under way:
  // 64-byte pieces (single blocks) took twice as long.
  struct RowStarts { uint64_t at[MT * 2]; const int* rws; };
  auto row_starts = [&](const int* rws) __attribute__((always_inline)) {
    RowStarts rs;
    rs.rws = rws;
#pragma unroll
    for (int g = 0; g < MT * 2; ++g) {
      const int r = g * 8 + (lane >> 3);
      rs.at[g] = (uint64_t)(uintptr_t)(feat + (size_t)(uint32_t)rws[min(r, B - 1)] * d0 + 4 * x_chunk(r, lane & 7));
    }
    return rs;
  };
  auto request_pair = [&](const RowStarts& rs, int pi) __attribute__((always_inline)) {
    if (rows_x4 && 32 * pi + 32 <= d0) {                   // whole pairs, with copies of the last row behind it (zero deltas)
#pragma unroll
      for (int g = 0; g < MT * 2; ++g)
        load_x4_to_lds(rs.at[g] + (uint32_t)(128 * pi), lds0 + (uint32_t)(pi * XB + g * 256) * 4u);
    } else if (rows_x4) {
#pragma unroll 1
      for (int g = 0; g < MT * 2; ++g) {
        const int r = g * 8 + (lane >> 3), c = 32 * pi + 4 * x_chunk(r, lane & 7);
        if (c < d0)
          load_x4_to_lds((uint64_t)(uintptr_t)(feat + (size_t)(uint32_t)rs.rws[min(r, B - 1)] * d0 + c),
                         lds0 + (uint32_t)(pi * XB + g * 256) * 4u);
      }
    } else {
#pragma unroll 1
      for (int g = 0; g < MT * 8; ++g) {
        const int r = 2 * g + (lane >> 5), c = 32 * pi + 4 * x_chunk(r, (lane >> 2) & 7) + (lane & 3);
        if (c < d0)
          load_lane_dword_to_lds((uint64_t)(uintptr_t)(feat + (size_t)(uint32_t)rs.rws[min(r, B - 1)] * d0 + c),
                                 lds0 + (uint32_t)(pi * XB + g * 64) * 4u);
      }
    }
  };
  // one word per 128-byte line of this member's share of the rows that the lanes of this wavefront hold
  const int lines = (d0 * 4 + 127) / 128 + 1;              // a row need not start on a line
  auto touch_lines = [&](int row_of_lane) __attribute__((always_inline)) {
    for (int e0 = 0; e0 * p.P < B * lines; e0 += kWave) {
      const int e = (e0 + lane) * p.P + j;
      const int r = min(e / lines, B - 1), l = e - (e / lines) * lines;
      const int row = __shfl(row_of_lane, r);
      if (e < B * lines)
        load_lane_dword_to_lds((uint64_t)(uintptr_t)(feat + (size_t)(uint32_t)row * d0 + min(32 * l, d0 - 1)),
                               lds0 + (uint32_t)((dump - lds) * 4));
    }
  };

  // ---- the slice: W_1 in registers, W_2 / b_1 / b_2 in LDS ----------------------------------------
  float w1[KBI][NT][4];
  // Walks the slice of W_1 in register order: f(register, byte offset in a replica, exists).  The lane indices are made opaque,
  // so that no addresses or masks of the slice are kept in registers through the iterations.
  auto each_w1 = [&](auto&& f) __attribute__((always_inline)) {
    const auto* k = cold();
    int nn = n16, qq = q4;
    asm volatile("" : "+v"(nn), "+v"(qq));
    const int ld1 = k->ld1;
    const uint32_t first = 4u * (uint32_t)(k->w1_off + (long)(32 * wave + 4 * qq) * ld1 + j * W + nn);
#pragma unroll
    for (int kbi = 0; kbi < KBI; ++kbi)
      if (block(kbi) < KB) {                               // uniform
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            f(kbi, nt, q, first + 4u * (uint32_t)((32 * kTW * (kbi >> 1) + 16 * (kbi & 1) + q) * ld1 + nt * 16),
              16 * block(kbi) + 4 * qq + q < d0 && j * W + nt * 16 + nn < d1);
      }
  };
  auto at = [](auto* base, uint32_t bytes) __attribute__((always_inline)) {
    typedef std::remove_pointer_t<decltype(base)> F;
    typedef std::conditional_t<std::is_const_v<F>, const char, char> C;
    return reinterpret_cast<F*>(reinterpret_cast<C*>(base) + bytes);
  };
  auto zero_w = [&](float (&w)[KBI][NT][4]) __attribute__((always_inline)) {
#pragma unroll
    for (int kbi = 0; kbi < KBI; ++kbi)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int q = 0; q < 4; ++q) w[kbi][nt][q] = 0.0f;
  };
  // between LDS and a replica: f(LDS element of W_2 / b_1 / b_2, byte offset in a replica, exists)
  auto each_small = [&](float* lw2, float* lb1, float* lb2, auto&& f) __attribute__((always_inline)) {
    const auto* k = cold();
#pragma unroll
    for (int u = 0; u < (W * D2P + kTT - 1) / kTT; ++u) {
      const int e = tid + u * kTT, n = e / D2P, c = cls(n, e % D2P) - n * D2P;
      if ((W * D2P) % kTT == 0 || e < W * D2P)
        f(lw2[e], (uint32_t)(4 * (k->w2_off + (long)(j * W + n) * k->ld2 + c)), c < d2 && j * W + n < d1);
    }
    if (tid < W) f(lb1[tid], (uint32_t)(4 * (k->b1_off + j * W + tid)), j * W + tid < d1);
    if (tid < D2P) f(lb2[tid], (uint32_t)(4 * (k->b2_off + tid)), tid < d2);
  };
  auto draw = [&](int s, int slot_of_batch) __attribute__((always_inline)) {      // row of iteration s of this call
    const auto* k = cold();
    return sample_row(k->seed, (uint32_t)i, k->t0 + (uint64_t)s, (uint32_t)min(slot_of_batch, B - 1), k->log2n);
  };
  auto label = [&](int row) __attribute__((always_inline)) {
    const auto* k = cold();
    return k->labels[(size_t)i * k->rows + row];
  };
  // Everything that waits for memory is asked for before the first barrier, the minibatch (whose rows have to be drawn) right
  // behind it: the launch pays one latency instead of four.
  zero_w(w1);
  {
    const auto* k = cold();
    const float* src = k->src + (size_t)i * k->src_stride; // this worker's starting point
    each_w1([&](int kbi, int nt, int q, uint32_t off, bool ok) __attribute__((always_inline)) {
      if (ok) w1[kbi][nt][q] = *at(src, off);
    });
    each_small(w2, b1, b2, [&](float& l, uint32_t off, bool ok) __attribute__((always_inline)) { l = ok ? *at(src, off) : 0.0f; });
  }
  float vw1[MOM ? KBI : 1][NT][4];
  if constexpr (MOM) {
    const float* vel = cold()->vel + (size_t)i * cold()->m_pad;
    zero_w(vw1);
    each_w1([&](int kbi, int nt, int q, uint32_t off, bool ok) __attribute__((always_inline)) {
      if (ok) vw1[kbi][nt][q] = *at(vel, off);
    });
    each_small(vw2, vb1, vb2, [&](float& l, uint32_t off, bool ok) __attribute__((always_inline)) { l = ok ? *at(vel, off) : 0.0f; });
  }
  if (tid < B) rows[MR + tid] = draw(1, tid);
  for (int pi = wave; pi < pairs; pi += kTW)               // this wavefront's blocks
    for (int e = lane; e < XB / 4; e += kWave)
      reinterpret_cast<f32x4_t*>(X + (size_t)pi * XB)[e] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
  if (tid == 0) flag[0] = 0;
  lds_barrier();
  {
    const RowStarts rs = row_starts(rows + MR);
    for (int pi = wave; pi < pairs; pi += kTW) request_pair(rs, pi);
  }

  // Rows of iteration t + 1 and labels of iteration t, by the lanes of the last wavefront: the row at which a label is read is
  // drawn an iteration before the label is stored.
  const bool drawer = wave == kTW - 1;
  int lab_next = 0;
  if (drawer) {
    const int r1 = rows[MR + min(lane, B - 1)], r2 = draw(2, lane);
    if (lane < B) {
      ylab[MR + lane] = label(r1);
      rows[lane] = r2;
      lab_next = label(r2);
    }
    touch_lines(r2);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // the blocks of iteration 1 have landed
  __syncthreads();

  // ---- restart: x_i <- (1/N) sum_i x_i --------------------------------------------------------------
  // Meeting of the whole grid; false: given up.  Everything stored before it is visible to the agent-scope loads after it.
  // Nobody can be a meeting ahead of those that still look for this one's flags, so a flag is the low byte of the
  // meeting's number, and a wavefront sees 256 of them in one load.  Every XCD looks at a copy of its own.
  auto meet = [&](unsigned char* fl, unsigned number) -> bool {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid < 8)
      __hip_atomic_store(fl + tid * flag_stride + me, (unsigned char)number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (wave == 0) {
      unsigned tries = 0;
      const unsigned* words = reinterpret_cast<const unsigned*>(fl + (blockIdx.x & 7) * flag_stride);
      const unsigned want = (number & 255u) * 0x01010101u;
      for (int w0 = 0; 4 * w0 < members; w0 += kWave) {
        const int w = w0 + lane, live = min(4, members - 4 * w);           // flags of this lane's word
        const unsigned mask = live >= 4 ? ~0u : live > 0 ? (1u << (8 * live)) - 1u : 0u;
        for (;;) {
          unsigned v = want;
          if (live > 0) v = __hip_atomic_load(words + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (__all(((v ^ want) & mask) == 0)) break;
          if (gave_up(abort_flag, tries, p.spin_limit)) { flag[0] = 1; break; }
          __builtin_amdgcn_s_sleep(1);
        }
      }
    }
    __syncthreads();
    return flag[0] == 0;
  };
  // The slices pass through memory in register order (block kb of tile nt: 1 KB), 16 bytes per lane: as single words in the
  // layout of the replicas the agent-scope stores alone took 8 us with 256 workgroups.
  const int blocks4 = KB * NT * kWave;                     // 16-byte vectors of a slice of W_1
  const int small = W * D2P + W + D2P;                     // floats behind them (a multiple of 4)
  const int slice4 = blocks4 + small / 4;
  auto restart = [&]() -> bool {
    const auto* k = cold();
    const int n = k->n_workers;
    f32x4_t* const mine = reinterpret_cast<f32x4_t*>(k->exchange) + (size_t)me * slice4;
    f32x4_t* const means = reinterpret_cast<f32x4_t*>(k->exchange) + (size_t)members * slice4;    // [P][slice4]
    auto rsrc = [&](f32x4_t* base) __attribute__((always_inline)) {
      return __builtin_amdgcn_make_buffer_rsrc(base, 0, slice4 * 16, 0x00020000);
    };
    {
      const __amdgpu_buffer_rsrc_t to = rsrc(mine);
#pragma unroll
      for (int kbi = 0; kbi < KBI; ++kbi)
        if (block(kbi) < KB) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const f32x4_t v = {w1[kbi][nt][0], w1[kbi][nt][1], w1[kbi][nt][2], w1[kbi][nt][3]};
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), to,
                                                   ((block(kbi) * NT + nt) * kWave + lane) * 16, 0, kAgentScope);
          }
        }
      for (int e = tid; e < small / 4; e += kTT)
        __builtin_amdgcn_raw_buffer_store_b128(reinterpret_cast<const u32x4_t*>(w2)[e], to, (blocks4 + e) * 16, 0, kAgentScope);
    }
    ++restarts;
    if (!meet(flags, restarts)) return false;
    // this worker's share of the vectors of slice j, in the order of the restart kernels
    const int per = (slice4 + n - 1) / n, lo = min(slice4, i * per), hi = min(slice4, lo + per);
    const bool quarters = n >= 8 && k->m_pad / 4 < 65536;
    const int n_per = quarters ? (n + 3) / 4 : n;
    const int split = quarters && n > 16 ? 4 : 1;          // wide sums: a quarter per group of threads
    const int cols = kTT / split;
    f32x4_t* part = reinterpret_cast<f32x4_t*>(red);       // [4][cols]
    const __amdgpu_buffer_rsrc_t out = rsrc(means + (size_t)j * slice4);
    const __amdgpu_buffer_rsrc_t all = __builtin_amdgcn_make_buffer_rsrc(k->exchange, 0, members * slice4 * 16, 0x00020000);
    const int first = j * slice4 * 16, stride = p.P * slice4 * 16;
    for (int c0 = lo; c0 < hi; c0 += cols) {
      const int q = tid / cols, c = c0 + tid - q * cols;
      const int i0 = split == 4 ? min(n, q * n_per) : 0, i1 = split == 4 ? min(n, i0 + n_per) : n;
      f32x4_t total = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f}, sum = total;
      int left = n_per;
      bool begun = false;
      if (c < hi) {
        for (int r0 = i0; r0 < i1; r0 += 16) {
          u32x4_t v[16];
#pragma unroll
          for (int u = 0; u < 16; ++u)
            if (r0 + u < i1)
              v[u] = __builtin_amdgcn_raw_buffer_load_b128(all, first + c * 16 + (r0 + u) * stride, 0, kAgentScope);
#pragma unroll
          for (int u = 0; u < 16; ++u)
            if (r0 + u < i1) {
              sum += __builtin_bit_cast(f32x4_t, v[u]);
              if (--left == 0) {
                total = begun ? total + sum : sum;
                begun = true;
                sum = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
                left = n_per;
              }
            }
        }
        if (left != n_per) total = begun ? total + sum : sum;
      }
      if (split == 4) {
        part[tid] = total;
        __syncthreads();
        if (q == 0) total = ((total + part[cols + tid]) + part[2 * cols + tid]) + part[3 * cols + tid];
        __syncthreads();
      }
      if (q == 0 && c < hi) {
        const f32x4_t mean = total / (float)n;
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, mean), out, c * 16, 0, kAgentScope);
      }
    }
    if (!meet(flags + 8 * flag_stride, restarts)) return false;
#pragma unroll
    for (int kbi = 0; kbi < KBI; ++kbi)
      if (block(kbi) < KB) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const f32x4_t v = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
              out, ((block(kbi) * NT + nt) * kWave + lane) * 16, 0, kAgentScope));
#pragma unroll
          for (int q = 0; q < 4; ++q) w1[kbi][nt][q] = v[q];
        }
      }
    for (int e = tid; e < small / 4; e += kTT)
      reinterpret_cast<u32x4_t*>(w2)[e] = __builtin_amdgcn_raw_buffer_load_b128(out, (blocks4 + e) * 16, 0, kAgentScope);
    __syncthreads();
    return true;
  };
  int to_restart = p.interval > 0 ? p.interval - (int)(p.t0 % (uint64_t)p.interval) : 0;

  // Partial-logit exchange: E floats per member.  Small teams: every member reads all P partials, G groups of
  // members in parallel (group g = members [g PG, (g + 1) PG) in order), then the groups in order.  Large ones (kTwoHopFloats)
  // in two hops: member j adds the P partials of its share of the floats, publishes the sums, and everybody
  // reads E sums: 2 E floats per member instead of P E.
  const int E = B * d2;
  const bool two_hops = two_hop_exchange(p.P, E);
  // The first hop goes by groups of lanes of a wavefront that add the partials of one float of the share, each every hop_groups-th
  // member: a member's share is small where the team is large, and one thread per float would ask for P / 8 rounds of partials in
  // turn.  A group's lanes take consecutive floats (16 lanes of 16 members each instead: 8 x (784-256-10) 10.6 -> 12.1 us per iteration).
  // Against a thread per float: 4 x (784-1024-10) 17.2 -> 12.5 us, 1 x (256-4096-10) 29.9 -> 8.7, 8 x (784-256-10) 11.2 -> 10.6.
  const int G = two_hops ? 1 : max(1, min(p.P, kPollers / E));
  const int PG = (p.P + G - 1) / G;
  // this thread's first float, and the members it adds (with several groups a thread has one float at most)
  const int item_g = G > 1 ? tid / E : 0, item_e = tid - item_g * E;
  const bool has_item = !drawer && item_g < G;
  const int j_lo = item_g * PG, j_hi = min(p.P, j_lo + PG);
  unsigned polls = 0;
  // sum of what `from[first]`, `from[first + stride]`, .. (count) hold once they carry `number`
  auto polled_sum = [&](const unsigned long long* from, int first, int stride, int count, unsigned number)
      __attribute__((always_inline)) {
    float sum = 0.0f;
    for (int u0 = 0; u0 < count; u0 += 8) {
      unsigned long long v[8];
      unsigned missing = (1u << min(8, count - u0)) - 1u;
      const unsigned asked = missing;
      for (;;) {                                           // only what is still missing is asked for again
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if ((missing >> u) & 1u)
            v[u] = __hip_atomic_load(at(from, 8u * (uint32_t)(first + (u0 + u) * stride)), __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (((missing >> u) & 1u) && (unsigned)(v[u] >> 32) == number) missing &= ~(1u << u);
        if (missing == 0) break;
        if (gave_up(abort_flag, polls, p.spin_limit)) { flag[0] = 1; break; }
        __builtin_amdgcn_s_sleep(1);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if ((asked >> u) & 1u) sum += __uint_as_float((unsigned)v[u]);
    }
    return sum;
  };
  // the same with every float to a place of its own: to[u to_stride] = from[first + u stride]
  auto polled_copy = [&](float* to, int to_stride, const unsigned long long* from, int first, int stride, int count, unsigned number)
      __attribute__((always_inline)) {
    unsigned long long v[8];
    unsigned missing = (1u << count) - 1u;
    for (;;) {
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if ((missing >> u) & 1u)
          v[u] = __hip_atomic_load(at(from, 8u * (uint32_t)(first + u * stride)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (((missing >> u) & 1u) && (unsigned)(v[u] >> 32) == number) missing &= ~(1u << u);
      if (missing == 0) break;
      if (gave_up(abort_flag, polls, p.spin_limit)) { flag[0] = 1; break; }
      __builtin_amdgcn_s_sleep(1);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (u < count) to[u * to_stride] = __uint_as_float((unsigned)v[u]);
  };

  for (int s = 1; s <= my_k; ++s) {
    // opaque copies: LDS addresses built from the lane indices are recomputed every iteration
    // instead of being hoisted out of the loop into dozens of registers
    asm volatile("" : "+v"(n16), "+v"(q4));
    int nb = KB;                                           // opaque: compared again, not kept as a mask per block
    asm volatile("" : "+s"(nb));
    const unsigned number = base + (unsigned)s;
    // (a) forward slice: contraction index of MFMA step q is k = 16 kb + 4 q4 + q
    {
      f32x4_t acc[MT][NT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
      // the A fragments of row block kbi+1 are read from LDS while block kbi is multiplied; the
      // scheduling fence keeps the compiler from hoisting every block's reads (and their
      // registers) to the top
      auto load_a = [&](int kbi, f32x4_t (&a)[MT]) __attribute__((always_inline)) {
        const float* xp = X + (size_t)(wave + kTW * (kbi >> 1)) * XB;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const int r = mt * 16 + n16;
          a[mt] = *reinterpret_cast<const f32x4_t*>(xp + r * 32 + 4 * x_chunk(r, 4 * (kbi & 1) + q4));
        }
      };
      f32x4_t a_cur[MT], a_nxt[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) a_cur[mt] = a_nxt[mt] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
      if (block(0) < nb) load_a(0, a_cur);
#pragma unroll
      for (int kbi = 0; kbi < KBI; ++kbi) {
        if (block(kbi) < nb) {                       // uniform
          if (kbi + 1 < KBI && block(kbi + 1) < nb) load_a(kbi + 1, a_nxt);
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
              for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = mfma16(a_cur[mt][q], w1[kbi][nt][q], acc[mt][nt]);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) a_cur[mt] = a_nxt[mt];
        }
      }
      auto share_out = [&](bool add) __attribute__((always_inline)) {
        float* to = red + (size_t)(add ? wave - kTW / 2 : wave) * MR * W;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              float* q = to + (mt * 16 + 4 * q4 + v) * W + nt * 16 + n16;
              *q = add ? *q + acc[mt][nt][v] : acc[mt][nt][v];
            }
      };
      if (shares == kTW || wave < kTW / 2) share_out(false);
      if (shares != kTW) {                                 // the upper wavefronts add theirs
        lds_barrier();
        if (wave >= kTW / 2) share_out(true);
      }
    }
    lds_barrier();
    for (int e = tid; e < MR * W; e += kTT) {
      const int b = e / W, n = e % W;
      float z = b1[n];
#pragma unroll
      for (int w = 0; w < kTW / 2; ++w) z += red[w * MR * W + e];      // shares in order
      if (shares == kTW) {
#pragma unroll
        for (int w = kTW / 2; w < kTW; ++w) z += red[w * MR * W + e];
      }
      h[e] = b < B ? act2_fwd(z, p.act) : 0.0f;
    }
    lds_barrier();
    // (b) this slice's contribution to the logits, one 16 x 16 block per wavefront on the matrix
    // cores: part[b][c] = sum_n h[b][n] W_2[n][c]
    unsigned long long* const set = p.part + ((number & 1) != 0 ? p.part_odd : 0u);
    unsigned long long* team_part = set + (size_t)i * p.P * E;
    for (int tile = wave; tile < MT * CT; tile += kTW) {
      const int mt = tile / CT, ct = tile - mt * CT;
      f32x4_t g = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int u = 0; u < NT * 4; ++u)
        g = mfma16(h[(mt * 16 + n16) * W + 4 * u + q4], w2[cls(4 * u + q4, ct * 16 + n16)], g);
      const int b0 = mt * 16 + 4 * q4, c = ct * 16 + n16;
      unsigned long long* to = team_part + j * E;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (b0 + v < B && c < d2)
          __hip_atomic_store(at(to, 8u * (uint32_t)((b0 + v) * d2 + c)),
                             ((unsigned long long)number << 32) | __float_as_uint(g[v]), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    }
    // (c) sum of the P partial blocks, polled until every float carries this iteration's number
    float* lgp = red;                                      // [G][E] group sums
    if (!drawer) {
      polls = 0;
      if (!two_hops) {
        if (has_item) {
          for (int e = item_e; e < E; e += kPollers) {       // one pass when E <= 448
            lgp[item_g * E + e] = polled_sum(team_part, j_lo * E + e, E, j_hi - j_lo, number);
            if (G > 1) break;
          }
        }
      } else {
        const auto* k = cold();
        const int share_lo = min(E, j * k->share), share_hi = min(E, share_lo + k->share), hop_groups = k->hop_groups;
        unsigned long long* sums = set + (size_t)(members + i) * E;
        const int items = kWave / hop_groups, l = lane / items;
        for (int e0 = share_lo + wave * items; e0 < share_hi; e0 += (kTW - 1) * items) {
          const int e = e0 + (lane & (items - 1));
          float sum = polled_sum(team_part, l * E + e, hop_groups * E,
                                 e < share_hi ? (p.P - l + hop_groups - 1) / hop_groups : 0, number);
          for (int o = items; o < kWave; o <<= 1) sum += __shfl_xor(sum, o);
          if (l == 0 && e < share_hi)
            __hip_atomic_store(at(sums, 8u * (uint32_t)e), ((unsigned long long)number << 32) | __float_as_uint(sum),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // Up to ten floats per thread (3072 to 4096 floats): in two rounds instead of ten.  8 x (256-128-48), 64 rows, 14.2 -> 13.3 us
        // per iteration; fewer floats lose more by the registers (8 x (256-128-20), 32 rows, 8.0 -> 8.5 us).
        if constexpr (CT == 1 || MT < 3) {
          for (int e = tid; e < E; e += kPollers) lgp[e] = polled_sum(sums, e, 0, 1, number);
        } else {
          for (int e0 = tid; e0 < E; e0 += 8 * kPollers)
            polled_copy(lgp + e0, kPollers, sums, e0, kPollers, min(8, (E - e0 + kPollers - 1) / kPollers), number);
        }
      }
    } else if (s < my_k) {
      // meanwhile: labels of iteration s + 1 and rows of iteration s + 2
      const int r = draw(s + 2, lane);
      if (lane < B) {
        ylab[((s + 1) & 1) * MR + lane] = lab_next;
        rows[(s & 1) * MR + lane] = r;
        lab_next = label(r);
      }
      touch_lines(r);
    }
    lds_barrier();
    if (flag[0] != 0) { aborted = true; break; }
    // (d) logits = b_2 + group sums in order; softmax cross-entropy head, 16 lanes per minibatch
    // row, lane l holding classes l, l + 16, ...
    {
      const int l16 = tid & 15;
      for (int b = tid >> 4; b < MR; b += kTT / 16) {
        if (b < B) {
          float z[CT];
          float mx = -INFINITY;
#pragma unroll
          for (int q = 0; q < CT; ++q) {
            const int c = l16 + 16 * q;
            z[q] = -INFINITY;
            if (c < d2) {
              float sum = b2[c];
              for (int g = 0; g < G; ++g) sum += lgp[(size_t)g * E + b * d2 + c];
              z[q] = sum;
              mx = fmaxf(mx, sum);
            }
          }
          mx = row16_max(mx);
          float ex[CT];
          float se = 0.0f;
#pragma unroll
          for (int q = 0; q < CT; ++q) {
            ex[q] = (l16 + 16 * q < d2) ? expf(z[q] - mx) : 0.0f;
            se += ex[q];
          }
          se = row16_sum(se);
          const float inv_se = __builtin_amdgcn_rcpf(se);    // 1 <= se <= 64; one ulp
          const int y = ylab[(s & 1) * MR + b];
          const bool y_ok = y >= 0 && y < d2;               // an out-of-range label selects nothing
          if (j == 0 && l16 == (y_ok ? (y & 15) : 0)) {
            const int yq = y_ok ? (y >> 4) : 0;
            float zy = 0.0f;
#pragma unroll
            for (int q = 0; q < CT; ++q) zy = y_ok && yq == q ? z[q] : zy;
            p.row_loss[(size_t)i * B + b] = (mx + logf(se)) - zy;
          }
#pragma unroll
          for (int q = 0; q < CT; ++q) {
            const int c = l16 + 16 * q;
            lg[cls(b, c)] = c < d2 ? (ex[q] * inv_se - (c == y ? 1.0f : 0.0f)) * inv_b : 0.0f;
          }
        } else {
          for (int c = l16; c < D2P; c += 16) lg[b * D2P + c] = 0.0f;
        }
      }
    }
    lds_barrier();
    // (e) delta_1 slice (needs the pre-update W_2)
    for (int e = tid; e < MR * W; e += kTT) {
      const int b = e / W, n = e % W;
      float sum = 0.0f;
      for (int c = 0; c < (CT == 1 ? D2P : d2); c += 4) {          // delta_2 is zero from d_2 on
        const f32x4_t d4 = *reinterpret_cast<const f32x4_t*>(lg + cls(b, c));
        const f32x4_t w4 = *reinterpret_cast<const f32x4_t*>(w2 + cls(n, c));
        sum = fmaf(d4.x, w4.x, sum); sum = fmaf(d4.y, w4.y, sum);
        sum = fmaf(d4.z, w4.z, sum); sum = fmaf(d4.w, w4.w, sum);
      }
      dl1[e] = sum * act2_bwd(h[e], p.act);
    }
    // dW_2 = h^T delta_2 (one 16 x 16 block per wavefront) and db_2 = column sums of delta_2 (a
    // product with a matrix of ones) on the matrix cores, kept in registers until every read of
    // the old W_2 above is done.  Rows b >= B of delta_2 are zero.
    static_assert(NT * CT <= kTW, "one block of dW_2 per wavefront");
    const bool has_w = wave < NT * CT;
    const int nt_w = wave / CT, ct_w = wave - nt_w * CT;
    const int ct_b = kTW - 1 - wave;                              // db_2 blocks go to the last wavefronts
    const bool has_b2 = ct_b < CT;
    f32x4_t gw = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f}, gb2 = gw;
    if (has_w) {
#pragma unroll
      for (int u = 0; u < MT * 4; ++u)
        gw = mfma16(h[(4 * u + q4) * W + nt_w * 16 + n16], lg[cls(4 * u + q4, ct_w * 16 + n16)], gw);
    }
    if (has_b2) {
#pragma unroll
      for (int u = 0; u < MT * 4; ++u) gb2 = mfma16(1.0f, lg[cls(4 * u + q4, ct_b * 16 + n16)], gb2);
    }
    lds_barrier();
    // (f) dW_1 slice and eq. (3) in registers: contraction index of MFMA step u is b = 4u + q4.  A block
    // that has been multiplied takes the next minibatch.
    {
      const RowStarts rs = row_starts(rows + ((s + 1) & 1) * MR);
      float dfr[MT * 4][NT];
#pragma unroll
      for (int u = 0; u < MT * 4; ++u)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) dfr[u][nt] = dl1[(4 * u + q4) * W + nt * 16 + n16];
      auto load_x = [&](int kbi, float (&a)[MT * 4]) __attribute__((always_inline)) {
        const float* xp = X + (size_t)(wave + kTW * (kbi >> 1)) * XB;
#pragma unroll
        for (int u = 0; u < MT * 4; ++u)
          a[u] = xp[(4 * u + q4) * 32 + 4 * x_chunk(4 * u + q4, 4 * (kbi & 1) + (n16 >> 2)) + (n16 & 3)];
      };
      float x_cur[MT * 4], x_nxt[MT * 4];
#pragma unroll
      for (int u = 0; u < MT * 4; ++u) x_cur[u] = x_nxt[u] = 0.0f;
      if (block(0) < nb) load_x(0, x_cur);
#pragma unroll
      for (int kbi = 0; kbi < KBI; ++kbi) {
        if (block(kbi) < nb) {                       // uniform
          if (kbi + 1 < KBI && block(kbi + 1) < nb) load_x(kbi + 1, x_nxt);
          f32x4_t g[NT], g2[NT];                           // two chains: rows 4u of even and of odd u
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) g[nt] = g2[nt] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int u = 0; u < MT * 4; u += 2)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
              g[nt] = mfma16(x_cur[u], dfr[u][nt], g[nt]);
              g2[nt] = mfma16(x_cur[u + 1], dfr[u + 1][nt], g2[nt]);
            }
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) g[nt] += g2[nt];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              float gv = g[nt][v];
              if constexpr (MOM) {
                gv = fmaf(p.mu, vw1[kbi][nt][v], gv);
                vw1[kbi][nt][v] = gv;
              }
              w1[kbi][nt][v] = fmaf(-p.lr, gv, w1[kbi][nt][v]);
            }
          __builtin_amdgcn_sched_barrier(0);               // the products above have taken the pair out of LDS
          if (s < my_k && ((kbi & 1) != 0 || block(kbi) == nb - 1)) request_pair(rs, wave + kTW * (kbi >> 1));
#pragma unroll
          for (int u = 0; u < MT * 4; ++u) x_cur[u] = x_nxt[u];
        }
      }
    }
    // (g) the small updates; their next readers are behind a barrier of the next iteration
    if (has_w) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int e = cls(nt_w * 16 + 4 * q4 + v, ct_w * 16 + n16);
        float g = gw[v];
        if constexpr (MOM) { g = fmaf(p.mu, vw2[e], g); vw2[e] = g; }
        w2[e] = fmaf(-p.lr, g, w2[e]);
      }
    }
    if (has_b2 && q4 == 0) {
      float g = gb2[0];
      if constexpr (MOM) { g = fmaf(p.mu, vb2[ct_b * 16 + n16], g); vb2[ct_b * 16 + n16] = g; }
      b2[ct_b * 16 + n16] = fmaf(-p.lr, g, b2[ct_b * 16 + n16]);
    }
    if (wave >= 2 && wave < 2 + NT) {                             // db_1 = column sums of delta_1
      const int nt_b = wave - 2;
      f32x4_t gb1 = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int u = 0; u < MT * 4; ++u) gb1 = mfma16(1.0f, dl1[(4 * u + q4) * W + nt_b * 16 + n16], gb1);
      if (q4 == 0) {
        float g = gb1[0];
        if constexpr (MOM) { g = fmaf(p.mu, vb1[nt_b * 16 + n16], g); vb1[nt_b * 16 + n16] = g; }
        b1[nt_b * 16 + n16] = fmaf(-p.lr, g, b1[nt_b * 16 + n16]);
      }
    }
    if (p.interval > 0 && --to_restart == 0) {
      to_restart = p.interval;
      if (s < my_k) {
        __syncthreads();                                   // the slice is complete
        if (!restart()) { aborted = true; break; }
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this wavefront's blocks have landed
  }

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // no request into LDS outlives the workgroup
  if (aborted) return;
  __syncthreads();
  // ---- write the slice back ------------------------------------------------------------------
  {
    const auto* k = cold();
    float* prm = k->params + (size_t)i * k->m_pad;
    each_w1([&](int kbi, int nt, int q, uint32_t off, bool ok) __attribute__((always_inline)) {
      if (ok) *at(prm, off) = w1[kbi][nt][q];
    });
    // every member holds the same b_2: the first one writes it
    const long b2_at = 4 * k->b2_off;
    each_small(w2, b1, b2, [&](float& l, uint32_t off, bool ok) __attribute__((always_inline)) {
      if (ok && (j == 0 || (long)off < b2_at)) *at(prm, off) = l;
    });
    if constexpr (MOM) {
      float* vel = k->vel + (size_t)i * k->m_pad;
      each_w1([&](int kbi, int nt, int q, uint32_t off, bool ok) __attribute__((always_inline)) {
        if (ok) *at(vel, off) = vw1[kbi][nt][q];
      });
      each_small(vw2, vb1, vb2, [&](float& l, uint32_t off, bool ok) __attribute__((always_inline)) {
        if (ok && (j == 0 || (long)off < b2_at)) *at(vel, off) = l;
      });
    }
  }
  if (j == 0) {
    if (tid < B) p.idx[(size_t)i * B + tid] = rows[(my_k & 1) * MR + tid];
    if (tid == 0) {
      *base_slot = base + (unsigned)my_k;                  // all members have taken part in the last exchange
      if (i == 0 && p.interval > 0) *restart_base = restarts;
    }
  }
}

// ---- host side --------------------------------------------------------------------------------
size_t fused2_lds_bytes(const Fused2Plan& pl) {
  const size_t MR = (size_t)pl.MT * 16, W = (size_t)pl.NT * 16;
  size_t floats = (size_t)((pl.KB + 1) / 2) * MR * 32 + pl.shares * MR * W + 2 * MR * W + MR * pl.d2p + W * pl.d2p + W + pl.d2p +
                  4 * MR + 4 + kWave;
  if (pl.momentum) floats += W * pl.d2p + W + pl.d2p;
  return floats * sizeof(float);
}

template <int KBI, int NT, int MT> static const void* fused2_symbol(int ct, bool mom) {
  if (ct == 1)
    return mom ? reinterpret_cast<const void*>(mlp2_epoch_kernel<KBI, NT, MT, 1, true>)
               : reinterpret_cast<const void*>(mlp2_epoch_kernel<KBI, NT, MT, 1, false>);
  return mom ? reinterpret_cast<const void*>(mlp2_epoch_kernel<KBI, NT, MT, 4, true>)
             : reinterpret_cast<const void*>(mlp2_epoch_kernel<KBI, NT, MT, 4, false>);
}

static const void* fused2_pick(int kbi, int nt, int mt, int ct, bool mom) {
#define PICK(K, N, M) if (kbi == K && nt == N && mt == M) return fused2_symbol<K, N, M>(ct, mom);
  PICK(2, 1, 1) PICK(2, 1, 2) PICK(2, 1, 3) PICK(2, 1, 4) PICK(2, 2, 1) PICK(2, 2, 2) PICK(2, 2, 3) PICK(2, 2, 4)
  PICK(4, 1, 1) PICK(4, 1, 2) PICK(4, 1, 3) PICK(4, 1, 4) PICK(4, 2, 1) PICK(4, 2, 2) PICK(4, 2, 3) PICK(4, 2, 4)
  PICK(8, 1, 1) PICK(8, 1, 2) PICK(8, 1, 3) PICK(8, 1, 4) PICK(8, 2, 1) PICK(8, 2, 2) PICK(8, 2, 3) PICK(8, 2, 4)
#undef PICK
  return nullptr;
}

// Shapes the epoch kernel is written for (whether the teams fit the device is the plan's question), with any hidden width: per
// iteration of the epoch kernel and of the chain, 2 x (100-1999-10), 16 rows, 7.3 and 27 us, 1 x (783-900-10), 16 rows, 12 and 28 us.
// Momentum on ragged inputs or hidden layers stays with the per-layer chain.
bool fused2_shape(int n_workers, int d0, int d1, int d2, int batch, bool momentum) {
  if (momentum && ((d0 & 3) != 0 || (d1 & 15) != 0)) return false;
  return d0 >= 1 && d0 <= 1024 && d1 >= 1 && d2 <= 64 && batch <= 64 &&
         (long)n_workers * ((d1 + 31L) / 32) <= kFused2MaxMembers;
}

// Slots of the partial-logit exchange for the finest split, in two sets, or (`spare`) in one where two hops allow it.  Half as
// many members that take one hop, in two sets, need no more.
size_t fused2_part_slots(int n_workers, int d1, int d2, int batch, bool spare) {
  const size_t team = ((size_t)d1 + 15) / 16, floats = (size_t)batch * d2;
  if (!two_hop_exchange((int)team, (int)floats)) return (size_t)n_workers * floats * 2 * team;
  return (size_t)n_workers * floats * (team + 1) * (spare ? 1 : 2);
}

// Floats that the restarts inside a launch pass through memory: a slice per member, and the averages.  0: no plan can
// have that many workgroups resident.
size_t fused2_exchange_floats(int n_workers, int d0, int d1, int d2) {
  const size_t kb = ((size_t)d0 + 15) / 16, d2p = d2 <= 16 ? 16 : 64;
  size_t most = 0;
  for (size_t nt = 1; nt <= 2; ++nt) {
    const size_t team = (d1 + 16 * nt - 1) / (16 * nt), slice = kb * nt * 256 + nt * 16 * (d2p + 1) + d2p;
    const size_t floats = ((size_t)n_workers + 1) * team * slice;
    if ((size_t)n_workers * team <= kFused2MaxMembers && floats * sizeof(float) < ((size_t)1 << 31) && floats > most)
      most = floats;
  }
  return most;
}

// Decides whether the epoch kernel applies and how the team is shaped.  It needs every
// workgroup of the grid resident at once (checked against the occupancy the runtime reports), spread over the XCDs.  Narrow
// slices first: 20 x (784-192-10), 32 rows, teams of 12 spread 11.4 us per iteration, teams of 6 on an XCD each 15.7.
bool fused2_plan(int n_workers, int d0, int d1, int d2, int batch, bool momentum, Fused2Plan* pl) {
  if (!fused2_shape(n_workers, d0, d1, d2, batch, momentum)) return false;
  pl->momentum = momentum ? 1 : 0;
  pl->MT = (batch + 15) / 16;
  pl->KB = (d0 + 15) / 16;
  const int kbi_need = 2 * (((pl->KB + 1) / 2 + kTW - 1) / kTW);
  pl->KBI = kbi_need <= 2 ? 2 : kbi_need <= 4 ? 4 : 8;
  pl->d2p = d2 <= 16 ? 16 : 64;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return false;
  for (int nt = 1; nt <= 2; ++nt) {
    pl->NT = nt;
    pl->P = (d1 + 16 * nt - 1) / (16 * nt);
    // partial pre-activations of two wavefronts in one place, one barrier more, where the minibatch leaves no room
    pl->shares = kTW;
    if (fused2_lds_bytes(*pl) > 160 * 1024) pl->shares = kTW / 2;
    const size_t lds_bytes = fused2_lds_bytes(*pl);
    if (lds_bytes > 160 * 1024) continue;
    const void* sym = fused2_pick(pl->KBI, pl->NT, pl->MT, pl->d2p / 16, momentum);
    if (sym == nullptr) return false;
    if (hipFuncSetAttribute(sym, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes) != hipSuccess)
      return false;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, sym, kTT, lds_bytes) != hipSuccess)
      return false;
    const long places = (long)per_cu * (cus / 8);
    if (xcd_workgroups(n_workers, pl->P, false) > places) continue;
    pl->pinned_fits = xcd_workgroups(n_workers, pl->P, true) <= places;
    return true;
  }
  return false;
}

hipError_t launch_fused2(const Fused2Plan& pl, Fused2Args args, bool pinned, hipStream_t s) {
  const void* sym = fused2_pick(pl.KBI, pl.NT, pl.MT, pl.d2p / 16, pl.momentum != 0);
  if (sym == nullptr) return hipErrorInvalidValue;
  if ((pl.momentum != 0) != (args.vel != nullptr)) return hipErrorInvalidValue;
  args.P = pl.P;
  args.shares = pl.shares;
  args.pinned = pinned ? 1 : 0;
  const unsigned floats = (unsigned)(args.batch * args.d2);
  const bool two_hops = two_hop_exchange(pl.P, (int)floats);
  args.part_odd = args.spare_part && two_hops ? 0 : (unsigned)args.n_workers * (pl.P + (two_hops ? 1 : 0)) * floats;
  args.share = (args.batch * args.d2 + pl.P - 1) / pl.P;
  args.hop_groups = 1;
  while (args.hop_groups < 32 && 8 * args.hop_groups < pl.P) args.hop_groups *= 2;
  void* kargs[] = {&args};
  // Plain launch: fused2_plan has checked that the whole grid fits on an otherwise idle device at
  // once, and a team member that never shows up (other work holding compute units) ends in the
  // kernel's bounded wait and the abort flag, not in a hang.
  const int teams = pinned ? (args.n_workers + 7) / 8 * 8 : args.n_workers;
  return hipLaunchKernel(sym, dim3((unsigned)(teams * pl.P)), dim3(kTT), kargs, fused2_lds_bytes(pl), s);
}

}  // namespace prsgd
