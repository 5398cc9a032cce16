// probe_plan_greedy: the greedy balance-optimal planner (Sec. 4.3, Algorithm 1) as one workgroup.
//
// Input is the all-gathered prediction n_hat[R][E] (tokens that originate on rank rs and are predicted
// for expert e); output is the placement change (Delta^in / Delta^out per rank), the assignment
// n[rs][e][rt] and, for one rank, the plan in the layout probe_permute consumes - all in device
// memory, so that predict -> plan -> permute needs no host round trip (Sec. 2.3).
//
// The paper runs its solver as a single-block kernel with serial iterative updates (Sec. 5); the
// same shape fits here: the loop is inherently sequential (each move changes the bottleneck), and
// what one iteration touches is small once the per-rank aggregates are kept incrementally:
//   LDS   ner[r][e]   tokens of expert e processed on rank r
//         pos[r][e]   the origins of those tokens, one bit each
//         n[e][rs][rt]  the assignment, expert-major: a move rewrites one R x R slab.  It lies in LDS where it fits
//                     (kPlanLdsBytes: every R <= 11, 16 ranks up to 135 experts), otherwise in the workspace.
//   registers of wave 0, one rank per lane:
//         comp        sum over experts with ner > 0 of (ner + n0)          (compute term)
//         vin, vout   tokens received from / sent to other ranks            (network term)
//         load        tokens processed on the rank
//         and its latency, budget counts and invalid partners
// What bounds it is latency: an iteration is a chain of dependent steps.  One wave makes it, so that nothing of it needs a
// barrier; the move's effect on every rank follows from one column and one row of the expert's slab (the tokens that
// origins without a copy give up, and dst's own tokens coming home), reductions and the prefix over the origins run over the
// sixteen lanes of a DPP row, and whether an expert has anything to move is one mask.  8 ranks, 128 experts, 3 replicas: with 256
// threads, the new slab in LDS and four barriers per move this call and probe_plan_dispatch took 56 to 65 us, now 28 to 31; 16
// ranks of 256 experts 180 to 196 and 104 to 117.
// Per iteration only SelectHeavyExpert looks at every expert (up to four per lane, arg-max over the wave).
// All arithmetic is integer, so the plan is bit-identical to the sequential definition.
//
// Cost model (a reading; the paper names the terms but not their constants):
//   L_r = g_den * comp[r] + 2 * g_num * max(vin[r], vout[r])
// with eta_g(n) = n / (n + n0) inside comp (Sec. 3.2) and g_num / g_den = network time per token over
// compute time per token (Sec. 3.3).
#include <limits.h>

#include <mutex>

#include "common.hpp"

namespace probe {

constexpr int kPlanMaxRanks = 16;
constexpr int kPlanMaxReplicas = 8;
constexpr int kPlanMaxMoves = 64;

struct PlannerArgs {
  int R, E, E_loc, rank, max_replicas, budget, k_max;
  long long eps, n0, g_num, g_den;
};

__device__ __forceinline__ long long comp_term(long long tokens, long long n0) { return tokens > 0 ? tokens + n0 : 0; }

// LDS that the assignment may take; ner and pos (6 R E bytes) and the rest of the kernel's state (2 KB) come on top.  The most is 12
// ranks of 240 experts: 139200 bytes of assignment and 17280 of ner and pos.
constexpr int kPlanLdsBytes = 136 * 1024;
// Words between the slabs of two experts.  In LDS one more than R * R, so that threads that look at the same entry of
// neighbouring experts are on different banks.
__host__ __device__ constexpr int plan_slab_stride(int R, bool in_lds) { return R * R + (in_lds ? 1 : 0); }
static bool plan_fits_lds(int R, int E) { return E * plan_slab_stride(R, true) * 4 <= kPlanLdsBytes; }
__host__ __device__ constexpr int plan_pos_words(int R, int E) { return (R * E + 1) / 2; }
static size_t plan_lds_bytes(int R, int E, bool in_lds) {
  return (static_cast<size_t>(R) * E + plan_pos_words(R, E) + (in_lds ? E * plan_slab_stride(R, true) : 0)) * sizeof(int32_t);
}

// Reductions over the sixteen lanes of a DPP row; every lane gets the result.  All lanes of the wave take part.
template <int N>
__device__ __forceinline__ long long row_ror64(long long v) {
  const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x120 | N, 0xf, 0xf, false));
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(v >> 32), 0x120 | N, 0xf, 0xf, false);
  return static_cast<long long>(static_cast<unsigned long long>(static_cast<unsigned>(hi)) << 32 | lo);
}
template <typename Op>
__device__ __forceinline__ long long row_reduce64(long long v, Op op) {
  v = op(v, row_ror64<8>(v));
  v = op(v, row_ror64<4>(v));
  v = op(v, row_ror64<2>(v));
  return op(v, row_ror64<1>(v));
}
__device__ __forceinline__ long long row_sum64(long long v) { return row_reduce64(v, [](long long a, long long b) { return a + b; }); }
__device__ __forceinline__ long long row_max64(long long v) { return row_reduce64(v, [](long long a, long long b) { return max(a, b); }); }
__device__ __forceinline__ long long row_min64(long long v) { return row_reduce64(v, [](long long a, long long b) { return min(a, b); }); }

// Exclusive prefix sum over the sixteen lanes of a DPP row.
template <int N>
__device__ __forceinline__ long long row_shr64(long long v) {  // lane - N of the row, 0 before its first lane
  const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x110 | N, 0xf, 0xf, true));
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(v >> 32), 0x110 | N, 0xf, 0xf, true);
  return static_cast<long long>(static_cast<unsigned long long>(static_cast<unsigned>(hi)) << 32 | lo);
}
__device__ __forceinline__ long long row_prefix64(long long v) {
  long long s = v;
  s += row_shr64<1>(s);
  s += row_shr64<2>(s);
  s += row_shr64<4>(s);
  s += row_shr64<8>(s);
  return s - v;
}
// The value of the lane on the other side in a swap of rows (16) or halves (32) and this lane's own, combined; every row gets
// the same result.
template <typename Op>
__device__ __forceinline__ long long cross_rows64(long long v, Op op) {
  unsigned lo = static_cast<unsigned>(v), hi = static_cast<unsigned>(v >> 32);
  auto join = [](unsigned l, unsigned h) { return static_cast<long long>(static_cast<unsigned long long>(h) << 32 | l); };
  const auto l16 = __builtin_amdgcn_permlane16_swap(lo, lo, false, false), h16 = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  v = op(join(l16[0], h16[0]), join(l16[1], h16[1]));
  lo = static_cast<unsigned>(v);
  hi = static_cast<unsigned>(v >> 32);
  const auto l32 = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), h32 = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  return op(join(l32[0], h32[0]), join(l32[1], h32[1]));
}
__device__ __forceinline__ long long wave_max64(long long v) {
  return cross_rows64(row_max64(v), [](long long a, long long b) { return max(a, b); });
}
__device__ __forceinline__ long long read_lane64(long long v, int lane) {
  const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(v), lane));
  const int hi = __builtin_amdgcn_readlane(static_cast<int>(v >> 32), lane);
  return static_cast<long long>(static_cast<unsigned long long>(static_cast<unsigned>(hi)) << 32 | lo);
}

template <bool IN_LDS>
__global__ __launch_bounds__(256) void plan_greedy_kernel(const int32_t* __restrict__ n_hat, PlannerArgs a,
                                                          int32_t* n_workspace,  // [E][R][R]
                                                          int32_t* __restrict__ rep_off, int32_t* __restrict__ rep_slot,
                                                          int32_t* __restrict__ rep_weight,
                                                          int32_t* __restrict__ slot_expert,
                                                          int32_t* __restrict__ delta_in, int32_t* __restrict__ delta_out,
                                                          int32_t* __restrict__ moves, long long* __restrict__ stats,
                                                          int32_t* __restrict__ n_assign) {
  const int R = a.R, E = a.E, E_loc = a.E_loc, stride = plan_slab_stride(R, IN_LDS);
  extern __shared__ int32_t lds[];
  int32_t* const ner = lds;                                           // [R][E]
  uint16_t* const pos = reinterpret_cast<uint16_t*>(lds + R * E);     // [R][E]
  int32_t* const g_n = IN_LDS ? lds + R * E + plan_pos_words(R, E) : n_workspace;
  __shared__ uint32_t hostmask[PROBE_MAX_EXPERTS];
  __shared__ long long comp[kPlanMaxRanks], vin[kPlanMaxRanks], vout[kPlanMaxRanks], load[kPlanMaxRanks];
  __shared__ int32_t d_in[kPlanMaxRanks][kPlanMaxReplicas];
  __shared__ int32_t wave_tot[4];
  const int tid = threadIdx.x, lane = tid & 63;

  // ---- initial assignment: every token to the expert's home rank (baseline placement P')
  if (tid < kPlanMaxRanks)
    for (int i = 0; i < kPlanMaxReplicas; ++i) d_in[tid][i] = -1;
  if (tid < E) {
    const int e = tid, home = e / E_loc;
    int v[kPlanMaxRanks], tot = 0;
    uint32_t origins = 0;
#pragma unroll
    for (int rs = 0; rs < kPlanMaxRanks; ++rs) v[rs] = rs < R ? max(n_hat[rs * E + e], 0) : 0;
#pragma unroll
    for (int rs = 0; rs < kPlanMaxRanks; ++rs) {
      if (rs < R)
        for (int rt = 0; rt < R; ++rt) g_n[e * stride + rs * R + rt] = (rt == home) ? v[rs] : 0;
      tot = static_cast<int>(static_cast<unsigned>(tot) + static_cast<unsigned>(v[rs]));
      origins |= v[rs] > 0 ? 1u << rs : 0u;
    }
    for (int r = 0; r < R; ++r) {
      ner[r * E + e] = (r == home) ? tot : 0;
      pos[r * E + e] = static_cast<uint16_t>((r == home) ? origins : 0u);
    }
    hostmask[e] = 1u << home;
  }
  for (int i = tid; i < R * a.max_replicas; i += 256) delta_in[i] = -1;
  if (delta_out)
    for (int i = tid; i < R * a.budget; i += 256) delta_out[i] = -1;
  for (int i = tid; i < a.k_max * 3; i += 256) moves[i] = -1;
  __syncthreads();
  {  // aggregates: sixteen threads per rank, each over every sixteenth expert
    const int r = tid >> 4;
    long long s_comp = 0, s_vin = 0, s_vout = 0, s_load = 0;
    if (r < R) {
      for (int e = tid & 15; e < E; e += 16) {
        const int home = __ffs(hostmask[e]) - 1;
        const long long from_r = g_n[e * stride + r * R + home];
        if (home == r) {
          long long tot = 0;  // in 64 bits: all origins of one expert
          for (int rs = 0; rs < R; ++rs) tot += g_n[e * stride + rs * R + r];
          s_load += tot;
          s_comp += comp_term(tot, a.n0);
          s_vin += tot - from_r;
        } else {
          s_vout += from_r;
        }
      }
    }
    s_comp = row_sum64(s_comp);
    s_vin = row_sum64(s_vin);
    s_vout = row_sum64(s_vout);
    s_load = row_sum64(s_load);
    if ((tid & 15) == 0) {
      comp[r] = s_comp;
      vin[r] = s_vin;
      vout[r] = s_vout;
      load[r] = s_load;
    }
  }
  __syncthreads();

  // ---- the loop of Algorithm 1, by one wave; the four rows of sixteen lanes hold the same ranks
  if (tid < kWave) {
    const int lr = lane & 15;  // this lane's rank
    const bool is_rank = lr < R;
    long long my_comp = comp[lr], my_vin = vin[lr], my_vout = vout[lr], my_load = load[lr];
    // lanes past the last rank have the lowest latency there is
    long long l = is_rank ? a.g_den * my_comp + 2 * a.g_num * max(my_vin, my_vout) : LLONG_MIN;
    const long long lat_before = row_max64(l);
    const long long total = row_sum64(my_load), avg = (total + R - 1) / R;
    const int cap_in = min(a.budget, a.max_replicas);
    uint32_t invalid = 0;  // partners with which this rank as a source is through
    int n_in = 0, n_out = 0, k = 0;
    for (int guard = 0; guard < kPlanMaxMoves + kPlanMaxRanks * kPlanMaxRanks + 1; ++guard) {
      // bottleneck rank and the least-loaded helper whose pair with it is still valid (ties: lower rank)
      const long long mx_old = row_max64(l);
      const int src = __ffsll(__ballot(l == mx_old)) - 1;
      const uint32_t barred = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(invalid), src)) | 1u << src;
      const bool free_pair = is_rank && !((barred >> lr) & 1u);
      const long long mn = row_min64(free_pair ? l : LLONG_MAX);
      const int dst = __ffsll(__ballot(free_pair && l == mn)) - 1;
      if (dst < 0) break;

      // dual-side budget check, and SelectHeavyExpert: most tokens on src among the experts src holds, dst does not, with
      // something to move (tokens of an origin without a copy); an empty selection is treated like an empty budget
      long long key = -1;
      const int out_src = __builtin_amdgcn_readlane(n_out, src), in_dst = __builtin_amdgcn_readlane(n_in, dst);
      if (out_src < a.budget && in_dst < cap_in) {
#pragma unroll
        for (int i = 0; i < PROBE_MAX_EXPERTS / kWave; ++i) {
          const int e = lane + i * kWave;
          if (e < E) {
            const uint32_t hm = hostmask[e], from = pos[src * E + e];
            const long long tokens = ner[src * E + e];
            if (((hm >> src) & 1u) && !((hm >> dst) & 1u) && (from & ~hm)) key = max(key, tokens << 9 | (511 - e));
          }
        }
        key = wave_max64(key);
      }
      if (key < 0) {
        if (lr == src) invalid |= 1u << dst;
        continue;
      }
      const int es = 511 - static_cast<int>(__builtin_amdgcn_readfirstlane(static_cast<int>(key)) & 511);

      // WaterFillingRebalance on the expert's slab: column src by origin, column dst by origin, row dst by rank
      int32_t* const slab = g_n + es * stride;
      const uint32_t hm = hostmask[es];
      const int at_src = is_rank ? slab[lr * R + src] : 0, at_dst = is_rank ? slab[lr * R + dst] : 0;
      const int own = is_rank ? slab[dst * R + lr] : 0;
      long long o_ner = 0;  // tokens of es on this lane's rank, in 64 bits
#pragma unroll
      for (int j = 0; j < kPlanMaxRanks / 4; ++j) {
        const int rs = 4 * j + (lane >> 4);
        o_ner += is_rank && rs < R ? slab[rs * R + lr] : 0;
      }
      o_ner = cross_rows64(o_ner, [](long long x, long long y) { return x + y; });
      // origins without a copy, ascending rank, until src is down to the mean: each gives what those before it leave
      const bool gives = is_rank && lr != dst && !((hm >> lr) & 1u);
      const long long before = row_prefix64(gives ? at_src : 0);
      const long long want = read_lane64(my_load, src) - __builtin_amdgcn_readlane(own, src) - avg - before;
      const int mv = gives ? static_cast<int>(max(min(static_cast<long long>(at_src), want), 0ll)) : 0;
      const long long moved = row_sum64(mv);
      const long long homed = row_sum64(lr != dst ? own : 0);  // dst's own tokens come home first
      // what the move does to this lane's rank.  An origin that gives tokens holds no copy, so it is neither src nor dst and sends
      // as much as before; dst stops sending its own.
      const long long leave = own + (lr == src ? moved : 0ll);
      const long long n_ner = lr == dst ? o_ner + homed + moved : o_ner - leave;
      const long long t_comp = my_comp - comp_term(o_ner, a.n0) + comp_term(n_ner, a.n0);
      const long long t_vin = my_vin + (lr == dst ? moved : -leave);
      const long long t_vout = my_vout - (lr == dst ? homed : 0ll);
      const long long t_load = my_load - o_ner + n_ner;
      const long long t_l = is_rank ? a.g_den * t_comp + 2 * a.g_num * max(t_vin, t_vout) : LLONG_MIN;
      const long long mx_new = row_max64(t_l);
      if (mx_old - mx_new <= a.eps || k >= a.k_max) break;  // converged, or the iteration budget is used up

      // accept the move
      const int kept = at_src - mv, taken = lr == dst ? static_cast<int>(homed + own) : at_dst + mv;
      const uint32_t on_src = static_cast<uint32_t>(__ballot(is_rank && lr != dst && kept > 0)) & 0xffffu;
      const uint32_t on_dst = static_cast<uint32_t>(__ballot(is_rank && taken > 0)) & 0xffffu;
      if (lane < R) {
        if (lr != dst) {
          slab[lr * R + src] = kept;
          slab[lr * R + dst] = taken;
        }
        slab[dst * R + lr] = lr == dst ? taken : 0;
        ner[lr * E + es] = static_cast<int>(n_ner);
        const uint32_t from = pos[lr * E + es] & ~(1u << dst);
        pos[lr * E + es] = static_cast<uint16_t>(lr == src ? on_src : (lr == dst ? on_dst : from));
      }
      if (lane == 0) {
        hostmask[es] = hm | 1u << dst;
        if (delta_out) delta_out[src * a.budget + out_src] = es;
        delta_in[dst * a.max_replicas + in_dst] = es;
        d_in[dst][in_dst] = es;
        moves[3 * k] = es;
        moves[3 * k + 1] = src;
        moves[3 * k + 2] = dst;
      }
      my_comp = t_comp;
      my_vin = t_vin;
      my_vout = t_vout;
      my_load = is_rank ? t_load : 0;
      l = t_l;
      n_out += lr == src ? 1 : 0;
      n_in += lr == dst ? 1 : 0;
      k += 1;
      // the wave's stores are seen by its loads of the next round
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    }
    const long long mx = row_max64(l), ml = row_max64(is_rank ? my_load : 0);
    if (lane == 0) {
      stats[0] = lat_before;
      stats[1] = mx;
      stats[2] = ml;
      stats[3] = k;
    }
  }
  __syncthreads();

  // ---- outputs
  const int rank = a.rank, S = E_loc + a.max_replicas;
  for (int s = tid; s < S; s += 256) {
    int e = -1;
    if (s < E_loc) {
      e = rank * E_loc + s;
      if (e >= E) e = -1;
    } else {
      e = d_in[rank][s - E_loc];
    }
    slot_expert[s] = e;
  }
  // the plan as `rank` sees it: one replica per holding rank in ascending rank order, weights = planned tokens
  const int cnt = tid < E ? __popc(hostmask[tid]) : 0;
  int incl = cnt;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    int o = __shfl_up(incl, d, kWave);
    if (lane >= d) incl += o;
  }
  if (lane == kWave - 1) wave_tot[tid >> 6] = incl;
  __syncthreads();
  int at = incl - cnt;
  for (int i = 0; i < (tid >> 6); ++i) at += wave_tot[i];
  if (tid < E) {
    const int e = tid, home = e / E_loc;
    const uint32_t hm = hostmask[e];
    rep_off[e] = at;
    long long planned = 0;
    int home_pos = at;
    for (int r = 0; r < R; ++r) {
      if (!((hm >> r) & 1u)) continue;
      int slot = -1;
      if (r == rank) {
        if (r == home) {
          slot = e - r * E_loc;
        } else {
          for (int i = 0; i < a.max_replicas; ++i)
            if (d_in[r][i] == e) slot = E_loc + i;
        }
      }
      if (r == home) home_pos = at;
      rep_slot[at] = slot;
      rep_weight[at] = ner[r * E + e];
      planned += ner[r * E + e];
      at += 1;
    }
    if (planned == 0) rep_weight[home_pos] = 1;  // nothing predicted: unforeseen tokens go home
    if (e == E - 1) rep_off[E] = at;
  }
  if (n_assign) {
    for (int i = tid; i < E * R; i += 256) {
      const int e = i / R, rt = i % R;
      for (int rs = 0; rs < R; ++rs) n_assign[static_cast<long>(rs) * E * R + i] = g_n[e * stride + rs * R + rt];
    }
  }
}

// More than 64 KB of dynamic LDS has to be opted into once per device.
constexpr int kPlanLdsMost = kPlanLdsBytes + 18 * 1024;  // 12 ranks, 240 experts: 156480 bytes
static int plan_prepare() {
  static std::mutex mu;
  static bool done[64] = {false};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    set_error("probe_plan_greedy: no current device");
    return PROBE_EHIP;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (done[dev]) return PROBE_OK;
  hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(plan_greedy_kernel<true>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kPlanLdsMost);
  if (err != hipSuccess) {
    set_error("probe_plan_greedy: cannot reserve %d bytes of LDS: %s", kPlanLdsMost, hipGetErrorString(err));
    return PROBE_EHIP;
  }
  done[dev] = true;
  return PROBE_OK;
}

// The plan as source rank `rank` applies it to its own tokens: one slot per (destination rank, expert
// copy), numbered by rank first and expert second.  One workgroup; thread e finds the ranks that hold
// expert e (home + the replicas listed in delta_in); per rank, wave ballots and per-wave totals give the
// number of lower experts held there (the slot inside the rank) and the rank's slot count; a block scan
// of the copies per expert gives rep_off.
__global__ __launch_bounds__(256) void plan_dispatch_kernel(const int32_t* __restrict__ n_assign,
                                                            const int32_t* __restrict__ delta_in, int R, int E,
                                                            int E_loc, int max_replicas, int rank,
                                                            int32_t* __restrict__ rep_off,
                                                            int32_t* __restrict__ rep_slot,
                                                            int32_t* __restrict__ rep_weight,
                                                            int32_t* __restrict__ rank_off,
                                                            int32_t* __restrict__ slot_expert) {
  __shared__ int32_t wave_tot[4];
  __shared__ int32_t wave_cnt[kPlanMaxRanks][4];
  __shared__ int32_t r_off[kPlanMaxRanks + 1];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, e = tid;
  uint32_t hm = 0;
  if (e < E) {
    hm = 1u << (e / E_loc);
    for (int r = 0; r < R; ++r)
      for (int i = 0; i < max_replicas; ++i)
        if (delta_in[r * max_replicas + i] == e) hm |= 1u << r;
  }
  const uint64_t lower = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  int within[kPlanMaxRanks];  // experts below e, in this wave, held by rank r
#pragma unroll
  for (int r = 0; r < kPlanMaxRanks; ++r) {
    const uint64_t m = __ballot((hm >> r) & 1u);
    within[r] = __popcll(m & lower);
    if (lane == 0) wave_cnt[r][wv] = __popcll(m);
  }
  const int cnt = __popc(hm);
  int incl = cnt;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    int o = __shfl_up(incl, d, kWave);
    if (lane >= d) incl += o;
  }
  if (lane == kWave - 1) wave_tot[wv] = incl;
  __syncthreads();
  if (tid == 0) {
    int run = 0;
    for (int r = 0; r < R; ++r) {
      r_off[r] = run;
      rank_off[r] = run;
      run += wave_cnt[r][0] + wave_cnt[r][1] + wave_cnt[r][2] + wave_cnt[r][3];
    }
    r_off[R] = run;
    rank_off[R] = run;
  }
  __syncthreads();
  for (int i = r_off[R] + tid; i < E + R * max_replicas; i += 256) slot_expert[i] = -1;  // slots not in use
  int pos = incl - cnt;
  for (int i = 0; i < wv; ++i) pos += wave_tot[i];
  if (e < E) {
    const int home = e / E_loc;
    rep_off[e] = pos;
    long long planned = 0;
    int home_pos = pos, own_pos = -1;
#pragma unroll
    for (int r = 0; r < kPlanMaxRanks; ++r) {
      if (r < R && ((hm >> r) & 1u)) {
        int slot = r_off[r] + within[r];
        for (int i = 0; i < wv; ++i) slot += wave_cnt[r][i];
        const int w = n_assign[(static_cast<long>(rank) * E + e) * R + r];
        if (r == home) home_pos = pos;
        if (r == rank) own_pos = pos;
        rep_slot[pos] = slot;
        rep_weight[pos] = w;
        slot_expert[slot] = e;
        planned += w;
        pos += 1;
      }
    }
    // nothing predicted from this origin: an unforeseen token stays here if a copy is here, else goes home
    if (planned == 0) rep_weight[own_pos >= 0 ? own_pos : home_pos] = 1;
    if (e == E - 1) rep_off[E] = pos;
  }
}

}  // namespace probe

extern "C" int probe_plan_dispatch(const int32_t* n_assign, const int32_t* delta_in, int R, int E, int E_loc,
                                   int max_replicas, int rank, int32_t* rep_off, int32_t* rep_slot,
                                   int32_t* rep_weight, int32_t* rank_off, int32_t* slot_expert, void* stream) {
  using namespace probe;
  PROBE_REQUIRE(R >= 1 && E >= 1 && E_loc >= 1 && static_cast<long>(E_loc) * R >= E && rank >= 0 && rank < R &&
                    max_replicas >= 0,
                PROBE_EINVAL, "probe_plan_dispatch: bad dims R=%d E=%d E_loc=%d rank=%d max_replicas=%d", R, E, E_loc,
                rank, max_replicas);
  PROBE_REQUIRE(R <= kPlanMaxRanks && E <= PROBE_MAX_EXPERTS && max_replicas <= kPlanMaxReplicas, PROBE_EUNSUPPORTED,
                "probe_plan_dispatch: needs R <= %d, E <= %d, max_replicas <= %d", kPlanMaxRanks, PROBE_MAX_EXPERTS,
                kPlanMaxReplicas);
  PROBE_REQUIRE(n_assign && (delta_in || max_replicas == 0) && rep_off && rep_slot && rep_weight && rank_off &&
                    slot_expert,
                PROBE_EINVAL, "probe_plan_dispatch: null pointer");
  hipLaunchKernelGGL(plan_dispatch_kernel, dim3(1), dim3(256), 0, static_cast<hipStream_t>(stream), n_assign,
                     delta_in, R, E, E_loc, max_replicas, rank, rep_off, rep_slot, rep_weight, rank_off, slot_expert);
  return check_launch("probe_plan_dispatch");
}

extern "C" size_t probe_plan_greedy_workspace_bytes(int R, int E) {
  if (R <= 0 || E <= 0) return 0;
  return probe::align_up(static_cast<size_t>(E) * R * R * sizeof(int32_t), 256);
}

extern "C" int probe_plan_greedy(const int32_t* n_hat, int R, int E, int E_loc, int rank,
                                 const probe_planner_params* params, int32_t* rep_off, int32_t* rep_slot,
                                 int32_t* rep_weight, int32_t* slot_expert, int32_t* delta_in,
                                 int32_t* delta_out, int32_t* moves, int64_t* stats, int32_t* n_assign,
                                 void* workspace, size_t workspace_bytes, void* stream) {
  using namespace probe;
  PROBE_REQUIRE(params != nullptr, PROBE_EINVAL, "probe_plan_greedy: params is NULL");
  PROBE_REQUIRE(R >= 1 && E >= 1 && E_loc >= 1 && static_cast<long>(E_loc) * R >= E && rank >= 0 && rank < R,
                PROBE_EINVAL, "probe_plan_greedy: bad dims R=%d E=%d E_loc=%d rank=%d", R, E, E_loc, rank);
  PROBE_REQUIRE(params->max_replicas >= 0 && params->budget >= 0 && params->k_max >= 0 && params->g_den >= 1 &&
                    params->g_num >= 0 && params->n0 >= 0,
                PROBE_EINVAL, "probe_plan_greedy: bad parameters");
  PROBE_REQUIRE(R <= kPlanMaxRanks && E <= PROBE_MAX_EXPERTS && params->max_replicas <= kPlanMaxReplicas &&
                    params->budget <= kPlanMaxReplicas && params->k_max <= kPlanMaxMoves,
                PROBE_EUNSUPPORTED,
                "probe_plan_greedy: needs R <= %d, E <= %d, max_replicas <= %d, budget <= %d, k_max <= %d",
                kPlanMaxRanks, PROBE_MAX_EXPERTS, kPlanMaxReplicas, kPlanMaxReplicas, kPlanMaxMoves);
  PROBE_REQUIRE(n_hat && rep_off && rep_slot && rep_weight && slot_expert && stats &&
                    (delta_in || params->max_replicas == 0) && (moves || params->k_max == 0),
                PROBE_EINVAL, "probe_plan_greedy: null pointer");
  PROBE_REQUIRE(workspace && workspace_bytes >= probe_plan_greedy_workspace_bytes(R, E), PROBE_EWORKSPACE,
                "probe_plan_greedy: workspace too small (%zu < %zu)", workspace_bytes,
                probe_plan_greedy_workspace_bytes(R, E));
  PlannerArgs a;
  a.R = R; a.E = E; a.E_loc = E_loc; a.rank = rank;
  a.max_replicas = params->max_replicas; a.budget = params->budget; a.k_max = params->k_max;
  a.eps = params->eps; a.n0 = params->n0; a.g_num = params->g_num; a.g_den = params->g_den;
  const bool in_lds = plan_fits_lds(R, E);
  if (in_lds) {
    int rc = plan_prepare();
    if (rc != PROBE_OK) return rc;
  }
  const size_t lds = plan_lds_bytes(R, E, in_lds);
  hipLaunchKernelGGL(in_lds ? plan_greedy_kernel<true> : plan_greedy_kernel<false>, dim3(1), dim3(256), lds,
                     static_cast<hipStream_t>(stream), n_hat, a, static_cast<int32_t*>(workspace), rep_off, rep_slot,
                     rep_weight, slot_expert, delta_in, delta_out, moves, reinterpret_cast<long long*>(stats), n_assign);
  return check_launch("probe_plan_greedy");
}
