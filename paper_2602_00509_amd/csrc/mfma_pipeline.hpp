// Software-pipelined NT bf16 GEMM main loop on v_mfma_f32_16x16x32_bf16, shared by the grouped FFN
// and the gate.  See the comments of ffn.hip for the pipeline; this header only holds the loop.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace probe {

constexpr int FBK = 64;  // k per step
#define PROBE_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

template <int N>
__device__ __forceinline__ void wait_vm_lgkm0() {  // s_waitcnt vmcnt(N) lgkmcnt(0), N < 64
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}

// ---- shared main loop -----------------------------------------------------------------
// 8 waves as 2 (rows) x 4 (columns).  The A tile has 64*MI rows; the B tile has PL planes of
// 128*NI rows each (plane p, column c at B-tile row p*128*NI + c).  The calling wave accumulates
//   acc[i][j] += sum_p  A[32*MI*wm + 16*i .. +16, :] * B_p[32*NI*wn + 16*j .. +16, :]^T
// (PL = 1: a plain GEMM; PL = 3: one logical weight held as three bf16 planes).
// rA / rB are buffer descriptors of the tile's first A row / of the weight matrix; voff[j] is
// this lane's byte offset for DMA instruction j (MI instructions for A, then BW for B); k0 is
// the first k of this call's K range and K its length (a multiple of 64).
// AROUND: the first k-step is number k_start, the walk goes round to k_start - 1.
// NST = LDS stages (2 or 3); a DMA batch is issued NST k-steps ahead of its use.
//
// What bounds it: matrix cores under the chip's power limit, and next to them the way of the weights from HBM.  With all
// k offsets pinned to 0 (every load an L2 hit) the previous form of this loop ran at 1.40 instead of 1.18 PFLOP/s on the
// 8-expert prefill, with only the weights' offsets pinned at 1.35; releasing the weights' part of a stage early
// (EARLY below) took that case from 1.18 to 1.27, and 36 slots of 512 rows from 1.08 to 1.20 PFLOP/s.  Releasing them
// half-way through the k-step instead costs 3 %, together with half of the activations 5 %; issuing
// the activations' DMA in one burst instead of spread over the last steps costs 3 %.
//
// Why 16x16x32 and not 32x32x16: the chip is power-limited under matrix work, and per flop the 16x16x32 form
// reads and writes half as many accumulator bits (each accumulator is touched once per 32 k instead of once per
// 16) for twice the operand reads.  A loop of nothing but MFMAs on N(0,1) x N(0,0.02) operands in registers runs at
// 1.79 PFLOP/s with 32x32x16 and at 2.05 PFLOP/s with 16x16x32 (2.01 when every row of accumulators starts over at
// column 0 instead of running back and forth, which keeps one operand of every consecutive pair the same).
//
// Accumulator layout.  The B fragment is the MFMA's row operand, so with PERM = false registers 0..3 of lane l
// hold output row (l % 16) of the 16-row A fragment and the four consecutive output columns 4(l / 16) .. +3 of the
// 16-column B fragment.  With PERM = true, position p of B fragment 2q + f is fed B row 32q + 8(p / 4) + 4f + p % 4, so
// acc[i][2q] and acc[i][2q + 1] together hold the EIGHT consecutive columns 32q + 8(l / 16) .. +7: a 16-byte bf16
// store per lane and 64 contiguous bytes per row and store instruction.
//
// DRAW: thread 0 of the workgroup draws the next ticket of a work queue (atomic add of 1 on *draw_counter) at the
// start of the second-to-last k-step, which issues no DMA and ends with a wait for everything in flight, and
// leaves it in *draw_slot (LDS) before that step's barrier; after the loop every thread can read it.  Returns
// whether that happened (it needs K >= 128).  After the barrier of the last k-step no wave reads the LDS stages.

// STEPWISE: a fragment's products of one k-step are summed in registers of their own and added to the accumulators by the
// vector units, so a chain of additions in the matrix cores is PL * 2 products of 32 long and not K / 32 of them.  Their error
// grows with the length of a chain almost linearly (7168 x 256 experts, probabilities against 64 bits: 1.7e-6 at chains of 56
// k-steps, 9.7e-7 at 28, 4.6e-7 at 7; stepwise 4.0e-7, 3.0e-7, 3.2e-7).  Four additions per MFMA row of a k-step: no
// time on the 128-token tile of the gate, 3 to 5 % on the 256-token tile.

// 16-byte chunk c of tile row r is stored at chunk position c ^ key(r), so that the sixteen rows of a fragment reading
// the same logical chunk cover all 64 banks exactly once: sixteen consecutive rows, or (PERM) the rows 8a + b + const,
// a and b = 0..3.
template <bool PERM>
__device__ __forceinline__ int lds_key(int row) {
  return PERM ? ((row >> 1) & 1) | (((row >> 3) & 3) << 1) : (row >> 1) & 7;
}

template <int MI, int NI, int PL, int NST, bool PERM = false, bool DRAW = false, bool AROUND = false,
          bool STEPWISE = false>
__device__ __forceinline__ bool gemm_mainloop(__amdgpu_buffer_rsrc_t rA, __amdgpu_buffer_rsrc_t rB,
                                              const int (&voff)[MI + NI * PL * 2], int k0, int K,
                                              u32x4* smem, int wv, int lane, f32x4 (&acc)[2 * MI][2 * NI],
                                              int32_t* draw_counter = nullptr, volatile int* draw_slot = nullptr,
                                              int k_start = 0) {
  constexpr int WN = 4, BROWS = 128 * NI * PL, AW = MI, BW = BROWS / 64, LPW = AW + BW, BM = 64 * MI;
  constexpr int BF = 2 * NI;              // B fragments of a plane
  constexpr int NB = BF * PL;             // B fragments per k32
  constexpr int kStage = (BM + BROWS) * 8;  // 16-byte units per stage
  static_assert(NST == 2 || NST == 3, "two or three stages");
  static_assert(NST * kStage * 16 <= 160 * 1024, "LDS budget");
  const int wm = wv / WN, wn = wv % WN;

  auto issue_one = [&](int st, int j, int kbytes) {
    if (j < AW)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rA, PROBE_LDS_PTR(smem + st * kStage + (wv * AW + j) * 64), 16,
                                               voff[j], kbytes, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rB, PROBE_LDS_PTR(smem + st * kStage + BM * 8 + (wv * BW + (j - AW)) * 64), 16, voff[j], kbytes, 0, 0);
  };
  const int KT = K / FBK;
  auto kbytes_of = [&](int kt) {
    int s = kt;
    if constexpr (AROUND) {
      s += k_start;
      s = s >= KT ? s - KT : s;
    }
    return (k0 + s * FBK) * 2;
  };
  auto issue_all = [&](int st, int kt) {
#pragma unroll
    for (int j = 0; j < LPW; ++j) issue_one(st, j, kbytes_of(kt));
  };
  const int arow = 32 * MI * wm + (lane & 15);
  const int brow = 32 * NI * wn + (PERM ? ((lane & 12) << 1) | (lane & 3) : (lane & 15));
  const int akey = lds_key<false>(arow), bkey = lds_key<PERM>(brow);
  // A k-step is STEPS = 4 * MI steps; a step multiplies one A fragment by all B fragments at one of the two k32 of the
  // step.  Fragments are taken in pairs: (2p, k32 0) (2p + 1, k32 0) (2p, k32 1) (2p + 1, k32 1).
  //   * A fragments live in a ring of W register sets: as soon as the MFMAs of a step are issued, its set is loaded with
  //     the fragment needed W steps later, so the LDS reads are spread evenly over the MFMAs.  (Reading the fragments of
  //     a quarter k-step at once, double-buffered, needs 20 more registers: the 320-row tile then spills in the loop.)
  //   * The B fragments of both k32 stay in registers for the whole k-step: those of k32 1 are read at its start, those
  //     of k32 0 of the next k-step during its last two steps.  The B part of a stage is therefore free after a fifth
  //     to a third of its k-step, and with EARLY the DMA of the weights due NST k-steps later starts there, behind a
  //     barrier of its own, instead of at the end: weights come from HBM and take longest to arrive.
  constexpr int STEPS = 4 * MI, W = MI == 5 ? 5 : (MI == 1 ? 2 : (MI == 3 ? 6 : 4)), BAR = STEPS - W + (W > 2 ? 1 : 0);
  constexpr bool EARLY = MI >= 3;
  constexpr int FREE_B = 4;  // EARLY: the step before which B's part of the stage is released
  static_assert(STEPS % W == 0, "ring positions repeat every k-step");
  static_assert(!EARLY || FREE_B < BAR, "B is released before A");
  constexpr auto frag_of = [](int t) { return 2 * (t / 4) + (t & 1); };
  constexpr auto k32_of = [](int t) { return (t >> 1) & 1; };
  auto read_a = [&](int st, int t) {
    return smem[st * kStage + (arow + 16 * frag_of(t)) * 8 + ((4 * k32_of(t) + (lane >> 4)) ^ akey)];
  };
  auto read_b = [&](int st, int kk, int r) {
    const int p = r / BF, j = r % BF;
    const int row = p * 128 * NI + (PERM ? 32 * (j >> 1) + 4 * (j & 1) : 16 * j);
    return smem[st * kStage + (BM + brow + row) * 8 + ((4 * kk + (lane >> 4)) ^ bkey)];
  };
  u32x4 a[W], b[2][NB];
  f32x4 part[2][BF];
  // plane slowest, so consecutive MFMAs hit different accumulators; columns run back and forth, so the MFMAs on either
  // side of a step's end share an operand.  The weight fragment is the row operand.
  auto mfma_step = [&](int t) {
    const int i = frag_of(t), kk = k32_of(t);
#pragma unroll
    for (int p = 0; p < PL; ++p)
#pragma unroll
      for (int c = 0; c < BF; ++c) {
        const int j = ((t + p) & 1) ? BF - 1 - c : c;
        if constexpr (STEPWISE)
          part[t & 1][j] = mfma_16x16x32(b[kk][p * BF + j], a[t % W],
                                         kk == 0 && p == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : part[t & 1][j]);
        else
          acc[i][j] = mfma_16x16x32(b[kk][p * BF + j], a[t % W], acc[i][j]);
      }
  };
  // STEPWISE: the sums of a fragment's k-step, complete with step t, go to the accumulators
  auto add_step = [&](int t) {
#pragma unroll
    for (int j = 0; j < BF; ++j) acc[frag_of(t)][j] += part[t & 1][j];
  };

  // prologue: NST batches in flight, wait for the first
  issue_all(0, 0);
  if (KT > 1) issue_all(1, 1);
  bool waited = false;
  if constexpr (NST == 3) {
    if (KT > 2) {
      issue_all(2, 2);
      wait_vm_lgkm0<2 * LPW>();
      waited = true;
    }
  }
  if (!waited) {
    if (KT > 1) wait_vm_lgkm0<LPW>(); else wait_vm_lgkm0<0>();
  }
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int r = 0; r < NB; ++r) b[0][r] = read_b(0, 0, r);
#pragma unroll
  for (int t = 0; t < W; ++t) a[t] = read_a(0, t);
  // One k-step on stage `cur`.  DMA: issue tile kt+NST into the stage being vacated.
  // YOUNGER: a batch younger than tile kt+1 is in flight at the barrier (it may stay in flight).
  // NEXT: tile kt+1 exists.
  // `hook` runs between the step's wait and its barrier (LDS writes made there are seen by every wave after it).
  auto k_step = [&](int kt, int cur, auto dma_c, auto younger_c, auto next_c, auto hook) {
    constexpr bool DMA = decltype(dma_c)::value, YOUNGER = decltype(younger_c)::value,
                   NEXT = decltype(next_c)::value;
    const int nxt = (cur + 1 == NST) ? 0 : cur + 1;
    const int kbytes = kbytes_of(kt + NST);
    // DMA instructions are spread over the steps after the barrier that releases their part of the stage
    constexpr int ASTEPS = STEPS - BAR, BSTEPS = EARLY ? BAR - FREE_B : ASTEPS;
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      if (t == 0) {
#pragma unroll
        for (int r = 0; r < NB; ++r) b[1][r] = read_b(cur, 1, r);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (DMA && EARLY && t == FREE_B) {  // b[1] was used by the last two steps: every B read of the stage has arrived
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (STEPWISE) {
        if (t > 0 && t % 4 == 0) add_step(t - 1);
      }
      if (t == BAR) {
        // every read of stage cur is issued: wait for them and for this wave's share of tile kt+1; what was issued
        // after that share may stay in flight
        wait_vm_lgkm0<(YOUNGER ? LPW : 0) + (DMA && EARLY ? BW : 0)>();
        hook();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if constexpr (NEXT) {
#pragma unroll
          for (int u = STEPS - W; u < BAR; ++u) a[u % W] = read_a(nxt, u + W - STEPS);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (NEXT) {
        if (t == STEPS - 2) {
#pragma unroll
          for (int r = 0; r < NB; ++r) b[0][r] = read_b(nxt, 0, r);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      mfma_step(t);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (STEPWISE) {  // one step late, when the matrix cores are done with them
        if (t % 4 == 3) add_step(t - 1);
      }
      if (t + W < STEPS) {
        a[t % W] = read_a(cur, t + W);
      } else if constexpr (NEXT) {
        if (t >= BAR) a[t % W] = read_a(nxt, t + W - STEPS);
      }
      if constexpr (DMA) {
        const int u = EARLY ? t - FREE_B : t - BAR;
#pragma unroll
        for (int j = 0; j < BW; ++j)
          if (u >= 0 && u < BSTEPS && j * BSTEPS / BW == u) issue_one(cur, AW + j, kbytes);
#pragma unroll
        for (int j = 0; j < AW; ++j)
          if (t >= BAR && j * ASTEPS / AW == t - BAR) issue_one(cur, j, kbytes);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (STEPWISE) add_step(STEPS - 1);
  };
  using T_ = std::integral_constant<bool, true>;
  using F_ = std::integral_constant<bool, false>;
  int kt = 0, cur = 0;
  auto advance = [&]() {
    ++kt;
    cur = (cur + 1 == NST) ? 0 : cur + 1;
  };
  auto none = []() {};
  bool drew = false;
  auto step_before_last = [&]() {
    if constexpr (DRAW) {
      int ticket = 0;
      if (threadIdx.x == 0) ticket = atomicAdd(draw_counter, 1);
      k_step(kt, cur, F_{}, F_{}, T_{}, [&]() {
        if (threadIdx.x == 0) *draw_slot = ticket;
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the write has landed before the barrier
      });
      drew = true;
    } else {
      k_step(kt, cur, F_{}, F_{}, T_{}, none);
    }
  };
  if constexpr (NST == 2) {
    while (kt + 2 < KT) {
      k_step(kt, cur, T_{}, F_{}, T_{}, none);
      advance();
    }
    if (kt + 1 < KT) {
      step_before_last();
      advance();
    }
  } else {
    while (kt + 3 < KT) {
      k_step(kt, cur, T_{}, T_{}, T_{}, none);
      advance();
    }
    if (kt + 2 < KT) {
      k_step(kt, cur, F_{}, T_{}, T_{}, none);
      advance();
    }
    if (kt + 1 < KT) {
      step_before_last();
      advance();
    }
  }
  k_step(kt, cur, F_{}, F_{}, F_{}, none);
  return drew;
}

// Raw buffer descriptor over [base, base + bytes): loads past the end return zero.
// base and bytes are the same for every lane; saying so (readfirstlane) keeps the compiler from wrapping each access in
// a loop over the distinct descriptors of the wave, which it does when a value came through LDS or a vector register.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, size_t bytes) {
  const uint64_t p = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(p));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(p >> 32));
  const int n = __builtin_amdgcn_readfirstlane(
      static_cast<int>(bytes > 0xffffffffull ? 0xffffffffu : static_cast<unsigned>(bytes)));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(static_cast<uint64_t>(hi) << 32 | lo), 0, n,
                                           0x00020000);
}

// Per-lane byte offsets of the DMA instructions of this wave: instruction j covers tile rows
// (wv*CNT + j)*8 .. +8; lane l reads row +l/8, the chunk that belongs at LDS position l%8.
// PERM as in gemm_mainloop for the weight tile, false for the activation tile.
template <int CNT, bool PERM = false, typename RowFn>
__device__ __forceinline__ void dma_offsets(int wv, int lane, int row_bytes, RowFn row_of, int* out) {
#pragma unroll
  for (int j = 0; j < CNT; ++j) {
    int row = (wv * CNT + j) * 8 + (lane >> 3);
    int c = (lane & 7) ^ lds_key<PERM>(row);
    out[j] = row_of(row) * row_bytes + c * 16;
  }
}

}  // namespace probe
