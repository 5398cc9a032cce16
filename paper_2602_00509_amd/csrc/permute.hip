// probe_permute: plan-driven grouping of (token, top-k position) pairs by weight slot.
//
// The sequential definition (walk the pairs in order, the j-th arrival of an expert goes to a
// replica by weighted round-robin, append to the slot's list) is reproduced exactly without
// atomics: a pair's destination row follows from (expert e, arrival rank j) alone.
//
//   1. hist     each workgroup counts the experts of its own contiguous block of 1024 pairs
//               (LDS counters)                                           -> blk_hist[U][E]
//   2. index    every workgroup sums the block histograms (its exclusive base = the blocks before it,
//               n_e = all blocks), derives the rows per replica in closed form and the prefix sum over
//               slots (workgroup 0 writes slot_counts, slot_offsets, n_local), ranks the pairs of its block among
//               equal experts (wave ballots, counts of the earlier waves) and computes slot and row
//               analytically                                             -> pair_row, row_pair
//   3. scatter  one thread per 16-byte chunk of a token row: read x once, write it to each of
//               the token's local rows                                   -> xp
// Up to 16384 pairs the index kernel counts all blocks itself (no step 1), and up to 4 MB of x it also copies the rows (no step 3); a
// batch of more than 262144 pairs runs step 2 as a one-workgroup scan kernel followed by the ranking kernel.
//
// Steps 1-2 touch only T*k integers; step 3 carries the HBM traffic (T*H*2 bytes read at
// most, n_local*H*2 written).
#include <algorithm>
#include <mutex>

#include "common.hpp"

namespace probe {

constexpr int kPermWaves = 4;                 // waves per workgroup of the separate ranking kernel
constexpr int kSegPairs = 256;                // pairs per wave segment there
constexpr int kSegIters = kSegPairs / kWave;  // 4 wave-wide iterations per segment
constexpr int kIndexThreads = 1024;           // threads of a workgroup with one pair each
constexpr int kIndexWaves = kIndexThreads / kWave;
constexpr int kRepLds = 2048;                 // replica-list entries staged in LDS by the index kernel
// Blocks up to which every workgroup counts all of them instead of reading histograms that a launch of its own made.  Index part of
// the call, histograms / own counts: 2 blocks (129 tokens, top-8 of 128) 6.3 / 4.7 us, 8 7.6 / 5.6, 16 7.7 / 6.5 (top-2 of 8: 7.8 /
// 8.0), 24 7.9 / 7.8, 32 7.9 / 8.5, 64 8.1 / 12.6.
constexpr int kSelfBlocks = 16;
// 16-byte pieces of x up to which it also copies the rows, several workgroups to a block: a piece per thread of one workgroup per
// CU.  A launch for the copy / by the index kernel: 256 tokens x 4096, top-8 of 128 7.0 / 6.2 us, 512 7.8 / 6.9, 1024 x 1024 10.0 /
// 8.8; but with more, where the workgroups that all count come in two rounds, 640 x 4096 8.5 / 9.6, 384 x 7168 7.2 / 8.8.
constexpr long kScatterPieces = 256 * kIndexThreads;
constexpr int kFusedBlocks = 256;             // up to this many blocks (262144 pairs) step 2 is one launch

__device__ __forceinline__ uint64_t lanemask_lt() {
  int l = lane_id();
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}

// Lanes of the wave holding the same 8-bit key as this lane (inactive lanes excluded by
// passing valid = false; they get an empty mask).
__device__ __forceinline__ uint64_t match_key8(int key, bool valid) {
  uint64_t m = __ballot(valid);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    uint64_t bal = __ballot(valid && ((key >> b) & 1));
    m &= ((key >> b) & 1) ? bal : ~bal;
  }
  return valid ? m : 0ull;
}

// Step 1.  One pair per thread, four counters per expert (the lanes of a wave that hold a popular expert seldom meet).
__global__ __launch_bounds__(kIndexThreads) void permute_hist_kernel(
    const int32_t* __restrict__ topk_idx, int N, int E, int32_t* __restrict__ blk_hist) {
  __shared__ int32_t counts[4][PROBE_MAX_EXPERTS];
  const int tid = threadIdx.x;
  const long p = static_cast<long>(blockIdx.x) * kIndexThreads + tid;
  const int e = p < N ? topk_idx[p] : -1;
  counts[tid >> 8][tid & 255] = 0;
  __syncthreads();
  if (static_cast<unsigned>(e) < static_cast<unsigned>(E)) atomicAdd(&counts[tid & 3][e], 1);  // bad ids count nowhere
  __syncthreads();
  if (tid < E)
    blk_hist[static_cast<long>(blockIdx.x) * E + tid] = counts[0][tid] + counts[1][tid] + counts[2][tid] + counts[3][tid];
}

// Steps 2a / 2b for batches of more than kFusedBlocks blocks, where every workgroup summing all block
// histograms itself would cost more than a scan kernel in between (the work of step 2 grows with the square
// of the number of blocks).
// 2a.  One workgroup of 1024 threads: expert e = tid % 256 is scanned by four threads, each over a quarter
// of the blocks (sum pass, then a pass that writes the exclusive bases).
__global__ __launch_bounds__(1024) void permute_scan_kernel(
    int32_t* __restrict__ seg_hist /* in: counts, out: exclusive bases */, int U, int E,
    const int32_t* __restrict__ rep_off, const int32_t* __restrict__ rep_slot,
    const int32_t* __restrict__ rep_weight, int S, int32_t* __restrict__ slot_counts,
    int32_t* __restrict__ slot_offsets, int32_t* __restrict__ n_local) {
  __shared__ int32_t sc[PROBE_MAX_SLOTS];
  __shared__ int32_t part_tot[4][PROBE_MAX_EXPERTS];
  __shared__ int32_t wave_tot[4];
  const int tid = threadIdx.x;
  const int e = tid & 255, part = tid >> 8;
  const int chunk = (U + 3) / 4;
  const int u0 = min(part * chunk, U), u1 = min(u0 + chunk, U);
  for (int s = tid; s < S; s += 1024) sc[s] = 0;
  // this expert's replica range, its total weight and its first replica are fetched now, under
  // the histogram passes
  int lo = 0, hi = 0, P = 0, w_first = 0, s_first = -1;
  if (part == 0 && e < E) {
    lo = rep_off[e];
    hi = rep_off[e + 1];
    for (int i = lo; i < hi; ++i) P += rep_weight[i];
    if (hi > lo) {
      w_first = rep_weight[lo];
      s_first = rep_slot[lo];
    }
  }
  int tot = 0;
  if (e < E) {
    int u = u0;
    for (; u + 16 <= u1; u += 16) {  // sixteen independent loads in flight
      int c[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) c[i] = seg_hist[static_cast<long>(u + i) * E + e];
#pragma unroll
      for (int i = 0; i < 16; ++i) tot += c[i];
    }
    for (; u < u1; ++u) tot += seg_hist[static_cast<long>(u) * E + e];
  }
  part_tot[part][e] = tot;
  __syncthreads();
  if (e < E) {
    int run = 0;
    for (int q = 0; q < part; ++q) run += part_tot[q][e];
    int u = u0;
    for (; u + 16 <= u1; u += 16) {
      int c[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) c[i] = seg_hist[static_cast<long>(u + i) * E + e];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        seg_hist[static_cast<long>(u + i) * E + e] = run;
        run += c[i];
      }
    }
    for (; u < u1; ++u) {
      long i = static_cast<long>(u) * E + e;
      int c = seg_hist[i];
      seg_hist[i] = run;
      run += c;
    }
  }
  if (part == 0 && e < E) {
    const int n_e = part_tot[0][e] + part_tot[1][e] + part_tot[2][e] + part_tot[3][e];
    // rows each replica of this expert receives: floor(n/P) w_i + clamp(n mod P - c_{i-1}, 0, w_i)
    if (P > 0) {
      int full = n_e / P, rem = n_e - full * P, cum = 0;
      for (int i = lo; i < hi; ++i) {
        int wgt = i == lo ? w_first : rep_weight[i];
        int part_rows = min(max(rem - cum, 0), wgt);
        int slot = i == lo ? s_first : rep_slot[i];
        if (slot >= 0 && slot < S) sc[slot] = full * wgt + part_rows;
        cum += wgt;
      }
    }
  }
  __syncthreads();
  // exclusive prefix sum over S <= 1024 slots: 4 consecutive slots per thread, first 256 threads
  int v[4] = {0, 0, 0, 0}, local = 0, incl = 0;
  if (tid < 256) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int s = tid * 4 + i;
      v[i] = s < S ? sc[s] : 0;
      local += v[i];
    }
    incl = local;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      int o = __shfl_up(incl, d, kWave);
      if (lane_id() >= d) incl += o;
    }
    if (lane_id() == kWave - 1) wave_tot[tid / kWave] = incl;
  }
  __syncthreads();
  if (tid < 256) {
    int wave_base = 0;
    for (int i = 0; i < tid / kWave; ++i) wave_base += wave_tot[i];
    int excl = wave_base + incl - local;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int s = tid * 4 + i;
      if (s < S) {
        slot_counts[s] = v[i];
        slot_offsets[s] = excl;
      }
      excl += v[i];
    }
    if (tid == 255) {
      slot_offsets[S] = excl;
      n_local[0] = excl;
    }
  }
}

// 2b.  Ranks and rows of a block from the exclusive bases and slot offsets written by 2a.
__global__ __launch_bounds__(kPermWaves* kWave) void permute_index_kernel(
    const int32_t* __restrict__ topk_idx, int N, int E, const int32_t* __restrict__ blk_base,
    const int32_t* __restrict__ rep_off, const int32_t* __restrict__ rep_slot,
    const int32_t* __restrict__ rep_weight, const int32_t* __restrict__ slot_offsets, int S,
    int32_t* __restrict__ pair_row, int32_t* __restrict__ row_pair) {
  __shared__ int32_t cnt_mem[kPermWaves][PROBE_MAX_EXPERTS];
  __shared__ int32_t e_lo[PROBE_MAX_EXPERTS], e_hi[PROBE_MAX_EXPERTS], e_P[PROBE_MAX_EXPERTS];
  __shared__ int32_t s_off[PROBE_MAX_SLOTS + 1];
  __shared__ int32_t s_rw[kRepLds], s_rs[kRepLds];
  int w = threadIdx.x / kWave, lane = lane_id();
  volatile int32_t* cnt_w = cnt_mem[w];  // volatile: keep every lane's read before the leader's update
  long base = (static_cast<long>(blockIdx.x) * kPermWaves + w) * kSegPairs;
  // every global load that depends on nothing is issued first, so that their latencies overlap:
  // this wave's pairs, the block's bases, the size of the replica list
  int seg_e[kSegIters];
#pragma unroll
  for (int it = 0; it < kSegIters; ++it) {
    long p = base + it * kWave + lane;
    seg_e[it] = p < N ? topk_idx[p] : -1;
  }
  int start[PROBE_MAX_EXPERTS / kWave];
#pragma unroll
  for (int i = 0; i < PROBE_MAX_EXPERTS / kWave; ++i) {
    int e = lane + i * kWave;
    start[i] = e < E ? blk_base[static_cast<long>(blockIdx.x) * E + e] : 0;
  }
  const int R = rep_off[E];
  // the plan, once per workgroup: replica lists (in LDS when they fit), replica range and total
  // weight of every expert, slot offsets
  const bool staged = R <= kRepLds;
  if (staged)
    for (int i = threadIdx.x; i < R; i += kPermWaves * kWave) {
      s_rw[i] = rep_weight[i];
      s_rs[i] = rep_slot[i];
    }
  const int32_t* rw = staged ? s_rw : rep_weight;  // flat pointers: LDS or global
  const int32_t* rs = staged ? s_rs : rep_slot;
  for (int e = threadIdx.x; e < E; e += kPermWaves * kWave) {
    e_lo[e] = rep_off[e];
    e_hi[e] = rep_off[e + 1];
  }
  for (int i = threadIdx.x; i <= S; i += kPermWaves * kWave) s_off[i] = slot_offsets[i];
  // counts of this wave's own segment (the same walk as in step 1)
  for (int e = lane; e < E; e += kWave) cnt_w[e] = 0;
#pragma unroll
  for (int it = 0; it < kSegIters; ++it) {
    int e = seg_e[it];
    bool valid = static_cast<unsigned>(e) < static_cast<unsigned>(E);
    uint64_t m = match_key8(e, valid);
    if (valid && (m & lanemask_lt()) == 0) cnt_w[e] += __popcll(m);
  }
  __syncthreads();
  // total weight of every expert, from the staged list when there is one
  for (int e = threadIdx.x; e < E; e += kPermWaves * kWave) {
    int P = 0;
    for (int i = e_lo[e]; i < e_hi[e]; ++i) P += rw[i];
    e_P[e] = P;
  }
  // arrival rank at the start of this wave's segment: block base + counts of the earlier waves
#pragma unroll
  for (int i = 0; i < PROBE_MAX_EXPERTS / kWave; ++i) {
    int e = lane + i * kWave;
    if (e < E)
      for (int q = 0; q < w; ++q) start[i] += cnt_mem[q][e];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PROBE_MAX_EXPERTS / kWave; ++i) {
    int e = lane + i * kWave;
    if (e < E) cnt_w[e] = start[i];
  }
  int n_loc = s_off[S];
#pragma unroll
  for (int it = 0; it < kSegIters; ++it) {
    long p = base + it * kWave + lane;
    int e = seg_e[it];
    bool valid = static_cast<unsigned>(e) < static_cast<unsigned>(E);
    uint64_t m = match_key8(e, valid);
    if (p < N && !valid) {  // expert id out of range: the pair is computed nowhere on this GPU
      pair_row[p] = -1;
      if (p >= n_loc) row_pair[p] = -1;
    }
    if (valid) {
      int before = __popcll(m & lanemask_lt());
      int j = cnt_w[e] + before;                       // arrival rank of this pair for expert e
      int lo = e_lo[e], hi = e_hi[e], P = e_P[e];
      int row = -1;
      if (P > 0) {
        int full = j / P, u = j - full * P, cum = 0;
        for (int i = lo; i < hi; ++i) {
          int wgt = rw[i];
          if (u < cum + wgt) {
            int slot = rs[i];
            if (slot >= 0 && slot < S) row = s_off[slot] + full * wgt + (u - cum);
            if (row >= N) row = -1;  // only an inconsistent plan (two replicas in one slot) gets here
            break;
          }
          cum += wgt;
        }
      }
      pair_row[p] = row;
      if (row >= 0) row_pair[row] = static_cast<int32_t>(p);
      if (p >= n_loc) row_pair[p] = -1;
    }
    // all lanes of a key have read the counter above; the key's first lane now advances it
    if (valid && (m & lanemask_lt()) == 0) cnt_w[e] += __popcll(m);
  }
}

// Steps 1-2 of a block of 1024 pairs, one pair per thread: ranks within a wave by ballots, ranks between the sixteen waves and
// the blocks by counts in LDS.  Every workgroup derives the slot counts and offsets from the totals n_e (redundantly,
// workgroup 0 writes them out).  What bounds it is a chain of latencies: ids and plan offsets, the replica lists behind
// them, four barriers.  With 256 threads that walked four pairs each one after another, the call without the copy took 8.2 us
// for 128 tokens, top-8 of 128 experts (now 4.4), 13.9 for 1000 (5.6), 14.1 for 8192 (8.1), 19.8 for 30000 (12.2).
//   COUNT_SELF  the workgroup counts all blocks itself: no histogram launch in front of it (4 to 6 us), but every workgroup
//               reads all ids
//   otherwise   it sums the block histograms of permute_hist_kernel
//   SCATTER     several workgroups to a block (blockIdx.x): each derives all of it and copies its share of the block's token rows
//               to their rows of xp, taken from LDS; the first writes the index outputs
struct IndexOut {
  int32_t *slot_counts, *slot_offsets, *n_local, *pair_row, *row_pair;
};

template <bool COUNT_SELF, bool SCATTER>
__global__ __launch_bounds__(kIndexThreads) void permute_block_kernel(
    const int32_t* __restrict__ topk_idx, int N, int E, const int32_t* __restrict__ blk_hist, int U,
    const int32_t* __restrict__ rep_off, const int32_t* __restrict__ rep_slot,
    const int32_t* __restrict__ rep_weight, int S, IndexOut out, const u32x4* __restrict__ x, int k,
    int chunks_per_row, u32x4* __restrict__ xp) {
  __shared__ int32_t cnt[kIndexWaves][PROBE_MAX_EXPERTS];   // counts of a wave's pairs, then arrival rank at its start
  __shared__ int32_t other[2][4][PROBE_MAX_EXPERTS];        // [0] blocks before this one, [1] this one and those behind it
  __shared__ int32_t e_lo[PROBE_MAX_EXPERTS], e_hi[PROBE_MAX_EXPERTS], e_P[PROBE_MAX_EXPERTS];
  __shared__ int32_t s_off[PROBE_MAX_SLOTS + 1], sc[PROBE_MAX_SLOTS];
  __shared__ int32_t s_rw[kRepLds], s_rs[kRepLds];
  __shared__ int32_t wave_tot[kIndexWaves];
  __shared__ int32_t row_of[SCATTER ? kIndexThreads : 1];
  const int tid = threadIdx.x, w = tid / kWave, lane = lane_id();
  const int b = blockIdx.y;
  const bool writer = blockIdx.x == 0;  // of the block's index outputs
  const long p = static_cast<long>(b) * kIndexThreads + tid;
  // loads that depend on nothing first
  const int my_e = p < N ? topk_idx[p] : -1;
  const int R = rep_off[E];
  int my_lo = 0, my_hi = 0;
  if (tid < E) {
    my_lo = rep_off[tid];
    my_hi = rep_off[tid + 1];
  }
  const int group = tid >> 8, ge = tid & 255;  // four groups of 256 threads
#pragma unroll
  for (int i = 0; i < PROBE_MAX_EXPERTS / kWave; ++i) cnt[w][lane + i * kWave] = 0;
  if (tid < S) sc[tid] = 0;
  if constexpr (COUNT_SELF) {
    if (U > 1) {
      // four counters per expert, so that the lanes of a wave that hold a popular expert seldom meet
      other[0][group][ge] = other[1][group][ge] = 0;
      __syncthreads();
      constexpr int kBatch = 8;  // blocks whose loads are in flight together
      for (int u0 = 0; u0 < U; u0 += kBatch) {
        int id[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
          const long at = static_cast<long>(u0 + q) * kIndexThreads + tid;
          id[q] = at < N ? topk_idx[at] : -1;
        }
#pragma unroll
        for (int q = 0; q < kBatch; ++q)
          if (static_cast<unsigned>(id[q]) < static_cast<unsigned>(E)) atomicAdd(&other[u0 + q < b ? 0 : 1][tid & 3][id[q]], 1);
      }
    }
  } else {
    int before = 0, rest = 0;
    constexpr int kBatch = 16;  // blocks of a group whose loads are in flight together
    if (ge < E)
      for (int u0 = group; u0 < U; u0 += 4 * kBatch) {
        int c[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
          const int u = u0 + 4 * q;
          c[q] = u < U ? blk_hist[static_cast<long>(u) * E + ge] : 0;
        }
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
          const bool is_before = u0 + 4 * q < b;
          before += is_before ? c[q] : 0;
          rest += is_before ? 0 : c[q];
        }
      }
    other[0][group][ge] = before;
    other[1][group][ge] = rest;
  }
  const bool staged = R <= kRepLds;
  if (staged)
    for (int i = tid; i < R; i += kIndexThreads) {
      s_rw[i] = rep_weight[i];
      s_rs[i] = rep_slot[i];
    }
  const int32_t* rw = staged ? s_rw : rep_weight;  // flat pointers: LDS or global
  const int32_t* rs = staged ? s_rs : rep_slot;
  // rank among the equal experts of the wave; its first lane leaves the count (a wave's own row: no barrier since the clearing)
  const bool valid = static_cast<unsigned>(my_e) < static_cast<unsigned>(E);  // bad ids count nowhere
  const uint64_t m = match_key8(my_e, valid);
  const int rank = __popcll(m & lanemask_lt());
  if (valid && rank == 0) cnt[w][my_e] = __popcll(m);
  __syncthreads();
  if (tid < E) {
    // rows each replica receives: floor(n/P) w_i + clamp(n mod P - c_{i-1}, 0, w_i)
    int n_e = 0, P = 0;
    if (COUNT_SELF && U <= 1) {
#pragma unroll
      for (int q = 0; q < kIndexWaves; ++q) n_e += cnt[q][tid];
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) n_e += other[0][q][tid] + other[1][q][tid];
    }
    for (int i = my_lo; i < my_hi; ++i) P += rw[i];
    e_lo[tid] = my_lo;
    e_hi[tid] = my_hi;
    e_P[tid] = P;
    if (P > 0) {
      int full = n_e / P, rem = n_e - full * P, cum = 0;
      for (int i = my_lo; i < my_hi; ++i) {
        const int wgt = rw[i];
        const int part_rows = min(max(rem - cum, 0), wgt);
        const int slot = rs[i];
        if (slot >= 0 && slot < S) sc[slot] = full * wgt + part_rows;
        cum += wgt;
      }
    }
  }
  if (COUNT_SELF && U <= 1) __syncthreads();  // the counts were read above
  if (group == 1) {
    // arrival rank at the start of each wave's pairs: the blocks before this one + the earlier waves
    int run = 0;
    if (!(COUNT_SELF && U <= 1)) {
#pragma unroll
      for (int q = 0; q < 4; ++q) run += other[0][q][ge];
    }
    int c[kIndexWaves];
#pragma unroll
    for (int q = 0; q < kIndexWaves; ++q) c[q] = cnt[q][ge];
#pragma unroll
    for (int q = 0; q < kIndexWaves; ++q) {
      cnt[q][ge] = run;
      run += c[q];
    }
  }
  __syncthreads();
  // exclusive prefix sum over the slots, one per thread
  const int rows = tid < S ? sc[tid] : 0;
  int incl = rows;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int o = __shfl_up(incl, d, kWave);
    if (lane >= d) incl += o;
  }
  int excl = incl - rows;
  if (S > kWave) {
    if (lane == kWave - 1) wave_tot[w] = incl;
    __syncthreads();
    for (int i = 0; i < w; ++i) excl += wave_tot[i];
  }
  if (tid < S) {
    s_off[tid] = excl;
    if (tid == S - 1) s_off[S] = excl + rows;
    if (writer && b == 0) {
      out.slot_counts[tid] = rows;
      out.slot_offsets[tid] = excl;
      if (tid == S - 1) {
        out.slot_offsets[S] = excl + rows;
        out.n_local[0] = excl + rows;
      }
    }
  }
  __syncthreads();
  int row = -1;
  if (valid) {
    const int j = cnt[w][my_e] + rank;                     // arrival rank of this pair for expert e
    const int lo = e_lo[my_e], hi = e_hi[my_e], P = e_P[my_e];
    if (P > 0) {
      int full = j / P, u = j - full * P, cum = 0;
      for (int i = lo; i < hi; ++i) {
        const int wgt = rw[i];
        if (u < cum + wgt) {
          const int slot = rs[i];
          if (slot >= 0 && slot < S) row = s_off[slot] + full * wgt + (u - cum);
          if (row >= N) row = -1;  // only an inconsistent plan (two replicas in one slot) gets here
          break;
        }
        cum += wgt;
      }
    }
  }
  if (p < N && writer) {  // an expert id out of range: the pair is computed nowhere on this GPU
    out.pair_row[p] = row;
    if (row >= 0) out.row_pair[row] = static_cast<int32_t>(p);
    if (p >= s_off[S]) out.row_pair[p] = -1;
  }
  if constexpr (SCATTER) {
    row_of[tid] = row;
    __syncthreads();
    // the tokens of this block: whole ones, see the launch
    const unsigned first = static_cast<unsigned>(b) * kIndexThreads / k;
    const unsigned tokens = min(N - b * kIndexThreads, kIndexThreads) / k;
    const unsigned cpr = chunks_per_row, total = tokens * cpr;  // below 2^31
    const u32x4* xb = x + static_cast<size_t>(first) * cpr;
    for (unsigned c = blockIdx.x * kIndexThreads + tid; c < total; c += gridDim.x * kIndexThreads) {
      const unsigned t = c / cpr, col = c - t * cpr;
      bool any = false;
      for (int q = 0; q < k; ++q) any |= row_of[t * k + q] >= 0;
      if (!any) continue;
      const u32x4 v = __builtin_nontemporal_load(&xb[c]);
      for (int q = 0; q < k; ++q) {
        const int r = row_of[t * k + q];
        if (r >= 0) __builtin_nontemporal_store(v, &xp[static_cast<size_t>(r) * cpr + col]);
      }
    }
  }
}

// Step 3.
template <int K>
__global__ __launch_bounds__(256) void permute_scatter_kernel(const u32x4* __restrict__ x,
                                                              const int32_t* __restrict__ pair_row,
                                                              long total_chunks, int chunks_per_row,
                                                              u32x4* __restrict__ xp) {
  long gid = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (gid >= total_chunks) return;
  int t = static_cast<int>(gid / chunks_per_row);
  int c = static_cast<int>(gid - static_cast<long>(t) * chunks_per_row);
  int rows[K];
  bool any = false;
#pragma unroll
  for (int s = 0; s < K; ++s) {
    rows[s] = pair_row[static_cast<long>(t) * K + s];
    any |= rows[s] >= 0;
  }
  if (!any) return;
  u32x4 v = __builtin_nontemporal_load(&x[gid]);
#pragma unroll
  for (int s = 0; s < K; ++s)
    if (rows[s] >= 0) __builtin_nontemporal_store(v, &xp[static_cast<long>(rows[s]) * chunks_per_row + c]);
}

static int num_blocks(long N) {
  const long per = static_cast<long>(kSegPairs) * kPermWaves;
  return static_cast<int>((N + per - 1) / per);
}

}  // namespace probe

extern "C" size_t probe_permute_workspace_bytes(int T, int E, int k, int S) {
  (void)S;
  if (T < 0 || E <= 0 || k <= 0) return 0;
  long N = static_cast<long>(T) * k;
  int U = probe::num_blocks(N);
  return probe::align_up(static_cast<size_t>(U > 0 ? U : 1) * E * sizeof(int32_t), 256);
}

namespace probe {

// Shared body of probe_permute (block histograms in the caller's workspace) and
// probe_permute_static (block histograms in the library's own static scratch array).
static int permute_impl(const char* name, const int32_t* topk_idx, const probe_plan* plan, const void* x_bf16,
                        int T, int H, int E, int k, int32_t* slot_counts, int32_t* slot_offsets,
                        int32_t* row_pair, int32_t* pair_row, void* xp_bf16, int32_t* n_local, int32_t* seg,
                        hipStream_t st) {
  const int S = plan->num_slots;
  int N = T * k;
  int U = num_blocks(N);
  const IndexOut out = {slot_counts, slot_offsets, n_local, pair_row, row_pair};
  const int cpr = H / 8;
  const u32x4* x = static_cast<const u32x4*>(x_bf16);
  u32x4* xp = static_cast<u32x4*>(xp_bf16);
  const long total = static_cast<long>(T) * cpr;
  // blocks of whole tokens only (at most 1024)
  if (U >= 1 && U <= kSelfBlocks && xp != nullptr && (U == 1 || kIndexThreads % k == 0) && total <= kScatterPieces) {
    const long pieces = std::min<long>(T, kIndexThreads / k) * cpr;  // of a block
    const unsigned shares = static_cast<unsigned>((pieces + kIndexThreads - 1) / kIndexThreads);
    hipLaunchKernelGGL((permute_block_kernel<true, true>), dim3(shares, U), dim3(kIndexThreads), 0, st, topk_idx, N, E,
                       nullptr, U, plan->rep_off, plan->rep_slot, plan->rep_weight, S, out, x, k, cpr, xp);
    return check_launch(name);
  }
  if (U <= kSelfBlocks) {
    hipLaunchKernelGGL((permute_block_kernel<true, false>), dim3(1, std::max(U, 1)), dim3(kIndexThreads), 0, st, topk_idx, N, E,
                       nullptr, U, plan->rep_off, plan->rep_slot, plan->rep_weight, S, out, nullptr, k, 0, nullptr);
  } else {
    hipLaunchKernelGGL(permute_hist_kernel, dim3(U), dim3(kIndexThreads), 0, st, topk_idx, N, E,
                       seg);
    if (U <= kFusedBlocks) {
      hipLaunchKernelGGL((permute_block_kernel<false, false>), dim3(1, U), dim3(kIndexThreads), 0, st, topk_idx, N, E, seg, U,
                         plan->rep_off, plan->rep_slot, plan->rep_weight, S, out, nullptr, k, 0, nullptr);
    } else {
      hipLaunchKernelGGL(permute_scan_kernel, dim3(1), dim3(1024), 0, st, seg, U, E, plan->rep_off,
                         plan->rep_slot, plan->rep_weight, S, slot_counts, slot_offsets, n_local);
      hipLaunchKernelGGL(permute_index_kernel, dim3(U), dim3(kPermWaves * kWave), 0, st, topk_idx, N, E,
                         seg, plan->rep_off, plan->rep_slot, plan->rep_weight, slot_offsets, S, pair_row, row_pair);
    }
  }
  if (U > 0 && xp_bf16 != nullptr) {  // xp == NULL: the caller gathers rows on load instead
    unsigned grid = static_cast<unsigned>((total + 255) / 256);
#define PROBE_SCATTER_CASE(K) \
  case K: hipLaunchKernelGGL(permute_scatter_kernel<K>, dim3(grid), dim3(256), 0, st, x, pair_row, total, cpr, xp); break;
    switch (k) {
      PROBE_SCATTER_CASE(1) PROBE_SCATTER_CASE(2) PROBE_SCATTER_CASE(3) PROBE_SCATTER_CASE(4)
      PROBE_SCATTER_CASE(5) PROBE_SCATTER_CASE(6) PROBE_SCATTER_CASE(7) PROBE_SCATTER_CASE(8)
    }
#undef PROBE_SCATTER_CASE
  }
  return check_launch(name);
}

// Argument checks common to both entry points (everything but the scratch memory).
static int permute_check(const char* name, const int32_t* topk_idx, const probe_plan* plan, const void* x_bf16,
                         int T, int H, int E, int k, int32_t* slot_counts, int32_t* slot_offsets,
                         int32_t* row_pair, int32_t* pair_row, void* xp_bf16, int32_t* n_local) {
  PROBE_REQUIRE(T >= 0 && H > 0 && E > 0 && k > 0, PROBE_EINVAL, "%s: bad dims T=%d H=%d E=%d k=%d", name, T, H,
                E, k);
  PROBE_REQUIRE(plan != nullptr, PROBE_EINVAL, "%s: plan is NULL", name);
  int S = plan->num_slots;
  PROBE_REQUIRE(S >= 1, PROBE_EINVAL, "%s: plan->num_slots=%d", name, S);
  PROBE_REQUIRE(E <= PROBE_MAX_EXPERTS && k <= PROBE_MAX_TOPK && S <= PROBE_MAX_SLOTS && H % 8 == 0,
                PROBE_EUNSUPPORTED, "%s: needs E <= %d, k <= %d, S <= %d, H %% 8 == 0 (E=%d k=%d S=%d H=%d)", name,
                PROBE_MAX_EXPERTS, PROBE_MAX_TOPK, PROBE_MAX_SLOTS, E, k, S, H);
  PROBE_REQUIRE(static_cast<long>(T) * k < (1l << 31), PROBE_EUNSUPPORTED, "%s: T*k >= 2^31", name);
  PROBE_REQUIRE(plan->rep_off && plan->rep_slot && plan->rep_weight, PROBE_EINVAL, "%s: plan array is NULL", name);
  PROBE_REQUIRE(slot_counts && slot_offsets && n_local, PROBE_EINVAL, "%s: null output", name);
  PROBE_REQUIRE(T == 0 || (topk_idx && row_pair && pair_row && (xp_bf16 == nullptr || x_bf16)), PROBE_EINVAL,
                "%s: null pointer", name);
  PROBE_REQUIRE(aligned16(x_bf16) && aligned16(xp_bf16), PROBE_EALIGN, "%s: x/xp must be 16-byte aligned", name);
  return PROBE_OK;
}

}  // namespace probe

extern "C" int probe_permute(const int32_t* topk_idx, const probe_plan* plan, const void* x_bf16,
                             int T, int H, int E, int k, int32_t* slot_counts,
                             int32_t* slot_offsets, int32_t* row_pair, int32_t* pair_row,
                             void* xp_bf16, int32_t* n_local, void* workspace,
                             size_t workspace_bytes, void* stream) {
  using namespace probe;
  int rc = permute_check("probe_permute", topk_idx, plan, x_bf16, T, H, E, k, slot_counts, slot_offsets, row_pair,
                         pair_row, xp_bf16, n_local);
  if (rc != PROBE_OK) return rc;
  PROBE_REQUIRE(workspace && workspace_bytes >= probe_permute_workspace_bytes(T, E, k, plan->num_slots),
                PROBE_EWORKSPACE, "probe_permute: workspace too small (%zu < %zu)", workspace_bytes,
                probe_permute_workspace_bytes(T, E, k, plan->num_slots));
  return permute_impl("probe_permute", topk_idx, plan, x_bf16, T, H, E, k, slot_counts, slot_offsets, row_pair,
                      pair_row, xp_bf16, n_local, static_cast<int32_t*>(workspace),
                      static_cast<hipStream_t>(stream));
}

// ---- probe_permute_static: the same call for callers that cannot allocate ------------------
// The block histograms live in a file-scope device array instead of a caller-supplied workspace.
// Each GPU the library runs on holds its own copy of the array at its own address until the process
// ends; the address is looked up once per device (hipGetSymbolAddress, no allocation) and passed to
// the kernels like any workspace pointer.  The histogram kernel writes every entry the later kernels
// read, so nothing has to be cleared between calls.
namespace probe {

constexpr size_t kStaticScratchBytes = PROBE_PERMUTE_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) int32_t scratch[kStaticScratchBytes / sizeof(int32_t)];

static int static_scratch(int32_t** out) {
  static std::mutex mu;
  static int32_t* ptr_of[64] = {nullptr};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    set_error("probe_permute_static: no current device");
    return PROBE_EHIP;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (ptr_of[dev] == nullptr) {
    void* p = nullptr;
    hipError_t err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (err != hipSuccess || p == nullptr) {
      set_error("probe_permute_static: cannot locate the scratch array on device %d: %s", dev,
                hipGetErrorString(err));
      return PROBE_EHIP;
    }
    ptr_of[dev] = static_cast<int32_t*>(p);
  }
  *out = ptr_of[dev];
  return PROBE_OK;
}

}  // namespace probe

extern "C" size_t probe_permute_static_max_pairs(int E) {
  if (E <= 0 || E > PROBE_MAX_EXPERTS) return 0;
  const size_t blocks = probe::kStaticScratchBytes / (static_cast<size_t>(E) * sizeof(int32_t));
  return blocks * probe::kSegPairs * probe::kPermWaves;
}

extern "C" int probe_permute_static(const int32_t* topk_idx, const probe_plan* plan, const void* x_bf16, int T,
                                    int H, int E, int k, int32_t* slot_counts, int32_t* slot_offsets,
                                    int32_t* row_pair, int32_t* pair_row, void* xp_bf16, int32_t* n_local,
                                    void* stream) {
  using namespace probe;
  int rc = permute_check("probe_permute_static", topk_idx, plan, x_bf16, T, H, E, k, slot_counts, slot_offsets,
                         row_pair, pair_row, xp_bf16, n_local);
  if (rc != PROBE_OK) return rc;
  const size_t need = probe_permute_workspace_bytes(T, E, k, plan->num_slots);
  PROBE_REQUIRE(need <= kStaticScratchBytes, PROBE_EUNSUPPORTED,
                "probe_permute_static: T*k = %ld pairs with E = %d need %zu bytes of block histograms, the static "
                "scratch holds %zu (at most %zu pairs at this E); use probe_permute with a workspace",
                static_cast<long>(T) * k, E, need, kStaticScratchBytes, probe_permute_static_max_pairs(E));
  int32_t* seg = nullptr;
  rc = static_scratch(&seg);
  if (rc != PROBE_OK) return rc;
  return permute_impl("probe_permute_static", topk_idx, plan, x_bf16, T, H, E, k, slot_counts, slot_offsets,
                      row_pair, pair_row, xp_bf16, n_local, seg, static_cast<hipStream_t>(stream));
}
