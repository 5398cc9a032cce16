// probe_grouped_ffn: grouped SwiGLU expert FFN on the bf16 matrix cores.
//
//   0. schedule  turn slot_offsets into a table of row tiles (slot, first row, height), on device
//   1. gemm1     h[r, f] = silu(xp[r] . W1[f]) * (xp[r] . W3[f])        (K = H)
//   2. gemm2     y[r, n] = h[r] . W2[n]                                  (K = F)
//
// Both GEMMs are "NT": activations [rows, K] and weights [out, K] are K-contiguous, which is
// the 8-consecutive-k-per-lane operand layout of v_mfma_f32_16x16x32_bf16, so an MFMA operand
// is one 16-byte LDS read.
//
// One workgroup = 8 waves (2 x 4) computes a 256 x 256 output tile (320, 192, 128 or 64 rows x 256
// where a slot's row count is not a multiple of 256) in steps of 64 k:
//   * global -> LDS goes through buffer_load ... lds (no register staging).  The per-lane
//     offset is fixed for the whole K loop; the k position travels in a scalar offset.
//   * two LDS stages of up to 72 KB (three smaller ones for the 128- and 64-row tiles).  Rows are
//     128 bytes; 16-byte chunk c of row r is stored at chunk position c ^ key(r), one key for the activation and one
//     for the weight tile (lds_key), so that the sixteen rows of a fragment reading the same logical chunk cover all 64
//     banks exactly once.
//   * the fragment reads are spread over the MFMAs of a k-step.  A barrier after its first steps releases the
//     weights' part of the stage, one before its last steps the activations' part; the DMA instructions that
//     prefetch tile k+2 follow each of them, spread over MFMAs (mfma_pipeline.hpp).
//
// In gemm1 a workgroup's 256 weight rows are 128 gate rows plus the 128 matching up rows,
// arranged so that each lane holds gate and up of the same output element; SwiGLU is applied
// on the accumulators.  Ragged row counts: a tile row past the slot's last row lies past the end
// of the activation tile's buffer descriptor, so its loads return zeros, and its stores are
// dropped the same way; the row space is never padded.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "common.hpp"
#include "mfma_pipeline.hpp"

namespace probe {

constexpr int FBN = 256;
// LDS: tiles of 192 rows and more run two stages (72 KB each for the 320-row tile); the short
// tiles (128 / 64 rows) are bound by load latency rather than by the matrix cores and run three
// stages of 48 / 40 KB, which gives every DMA batch two k-steps to land.
constexpr int kFfnLdsBytes = 3 * (128 + 256) * 128;  // 144 KB
static_assert(kFfnLdsBytes >= 2 * (320 + 256) * 128, "two stages of the tallest tile");
// Narrow column blocks leave room for three stages up to 256 rows.  More (six at 64 rows) measured the same.
constexpr int ffn_stages(int mi, int ni) { return ni == 1 ? (mi == 5 ? 2 : 3) : (mi >= 3 ? 2 : 3); }
static_assert(kFfnLdsBytes >= 3 * (256 + 128) * 128 && kFfnLdsBytes >= 2 * (320 + 128) * 128, "stages of the narrow tiles");


// ---- 0. schedule ----------------------------------------------------------------------
// The table is one 32-byte header (first word = number of tiles) followed by one 32-byte TileEntry
// per row tile, which holds everything a workgroup needs to start loading: first row, number
// of valid rows from there to the end of the slot, tile height (320, 256, 192, 128 or 64) and
// the slot's two weight pointers.
//
// How a slot is cut.  Every tile streams 256 weight rows per k-step whatever its height, so a
// short tile costs far more than its share of rows (64 rows take almost half the time of 256).
// A slot of M rows, u = ceil(M / 64), becomes a tiles of 320 and b tiles of 256 with 5a + 4b = u
// and a as large as possible: b = 4u mod 5, which exists whenever 4b <= u (every u >= 12).  The
// six values of u without such a cut end in one short tile, chosen by measured tile cost:
//   u = 1, 2, 3: one tile of 64u rows;  6: 256 + 128;  7: 320 + 128;  11: 320 + 256 + 128.
// Inside a slot the 320s come first, then the 256s, then the short tile.
//
// Order of the table.  Slots are taken by descending row count (ties: lower slot first) and a
// slot's tiles stay together: the workgroups that run side by side then share a slot's weight
// slices in L2 and the long slots start early; the single short tiles (slots of up to 192 rows, or up to the height of the tiles where that is
// less) are spread evenly over the table, so that tiles that wait for weights run beside tiles that keep the matrix cores busy.  Two or three
// tiles of 64 rows of a slot stay together: spread apart they took up to 1.04 of the time in 16 calls of up to 256 items, on average 1.01.
//
// Where gemm1 has more items than CUs, but few enough tall tiles (more than 192 rows) that all of theirs start at once, the
// tiles stand by descending height instead: a tall item that begins second is then the end of the launch.  768 tokens,
// top-4 of 128 experts, 18 slots of 2880 x 2880: gemm1 116 -> 87 us, the layer 262 -> 235; 1500 tokens, 36 slots of 7168 x 2048
// 863 -> 809 us, 2000 tokens of the first 355 -> 333.  With more tall tiles they hold each other up (clock) and the short
// ones all come after them: 16384 tokens x 64 slots 3212 -> 3290 us, 2000 tokens of an 8-expert model 1338 -> 1390.  With no
// second round the order only moves items between XCDs (700 tokens, 33 slots of 2048 x 1024: 167 -> 172 us).  A cut without tall tiles keeps
// the slots in order: sorted by height, 24 calls each of more than 256 items took 1.028 (tiles of 192 rows; 0.95 to 1.12), 1.013 (128) and 1.006 (64)
// of the time.
struct alignas(16) TileEntry {
  int32_t row0, rows, height, slot;
  const void* w13;
  const void* w2;
};
static_assert(sizeof(TileEntry) == 32, "one 32-byte record per tile");
// Table header, 128 bytes: word 0 = number of tiles; words 1 and 2 = whether gemm1 and gemm2 take narrow column blocks; words 8..15
// and 16..23 = the work-queue tickets of gemm1 and gemm2 (one counter per XCD), set by the schedule kernel of the same call.
constexpr int kTableHeaderInts = 32, kNarrow1 = 1, kNarrow2 = 2, kQueue1 = 8, kQueue2 = 16;

struct SlotCut {
  int n320, n256;   // the standard cut
  int n_cap, cap;   // or tiles of one height
  int tail;         // height of the one short tile (64, 128 or 192), 0 if there is none
  __device__ __forceinline__ int tiles() const { return n320 + n256 + n_cap + (tail ? 1 : 0); }
  // tallest first: 320, 256, 192, 128, 64 rows
  static __device__ __forceinline__ int height_class(int height) { return height == 320 ? 0 : 5 - (height >> 6); }
  // tiles of each height, twelve bits per class
  __device__ __forceinline__ unsigned long long classes() const {
    return static_cast<unsigned long long>(n320) + (static_cast<unsigned long long>(n256) << 12) +
           (n_cap ? static_cast<unsigned long long>(n_cap) << (12 * height_class(cap)) : 0ull) +
           (tail ? 1ull << (12 * height_class(tail)) : 0ull);
  }
};

// cap = 0: the standard cut; otherwise tiles of `cap` rows (256, 192, 128 or 64) and one shorter.
__device__ __forceinline__ SlotCut cut_slot(int m, int cap) {
  SlotCut c = {0, 0, 0, 0, 0};
  const int u = (m + 63) >> 6;
  if (u <= 0) return c;
  if (cap) {
    c.cap = cap;
    c.n_cap = cap == 256 ? u >> 2 : cap == 192 ? u / 3 : cap == 128 ? u >> 1 : u;
    c.tail = 64 * u - cap * c.n_cap;
    return c;
  }
  if (u <= 3) {
    c.tail = 64 * u;
    return c;
  }
  const int b = (4 * u) % 5;
  if (4 * b <= u) {
    c.n256 = b;
    c.n320 = (u - 4 * b) / 5;
  } else {  // u == 6, 7 or 11
    c.n320 = u == 6 ? 0 : 1;
    c.n256 = u == 7 ? 0 : 1;
    c.tail = 128;
  }
  return c;
}

// Height of the tiles and width of the items.  A call with few tiles leaves CUs without an item, or with a second one when most are
// through; shorter tiles, or column blocks half as wide (64 h columns, 128 y columns), make more items that last less long, and move more
// bytes in all.  The schedule kernel estimates the launches of both GEMMs for the standard cut and for tiles of at most 256, 192, 128 and 64
// rows, each with wide and with narrow items, and takes the shortest; another cut has to be 2 % better than the standard one.
//
// The estimate: an item lasts 0.85 ns x k-steps x (3 x its rows + 4 x its weight rows), and 0.3 us; items are dealt as if tallest first, one
// workgroup to a CU.  The launch lasts as long as ceil(n / CUs) times the shortest of its n tallest items, for every n, and, with more
// items than CUs, as their mean load of a CU and 0.6 of the shortest.  Fitted to 90 drawn FFN calls of 64 to 4096 tokens, each timed with all
// twenty cuts: of the 4.7 % that the best cut of each gains over the standard cut with the former rule for the width (a limit on wide
// items, and an estimate for the width alone) this finds 3.4 %, on the half it was not fitted to 3.2 of 4.3.  640 x 1344, 18 blocks
// of 64 rows 42 -> 29 us (64 rows), 2880 x 2880, 17 blocks 127 -> 107 (128 rows, narrow gemm2), 52 blocks 213 -> 195 (192 rows), 4672 x 832, 25
// blocks 128 -> 104 (128 rows, narrow).  With many items per CU the standard cut moves the fewest bytes and stays.
constexpr int kXcds = 8, kBlkM = 8, kBlkN = 4, kBlk = kBlkM * kBlkN;  // blocks of work items, see ffn_item_of
constexpr int kCuts = 5;                                              // heights: the standard cut, 256, 192, 128, 64
__device__ __forceinline__ int cut_cap(int cut) { return cut == 0 ? 0 : 320 - 64 * cut; }
constexpr int kCutParts = kWave / kCuts;                              // lanes that count the tiles of one cut
constexpr int kCutUnits = 4000;                                       // 64-row units up to which the classes' twelve bits hold any cut's tiles
constexpr float kItemCost = 350.f, kCutGain = 0.98f;

__device__ __forceinline__ int tiles_of(unsigned long long classes) {
  int n = 0;
#pragma unroll
  for (int c = 0; c < 5; ++c) n += static_cast<int>(classes >> (12 * c)) & 4095;
  return n;
}

// rows up to which a slot is a single short tile
__device__ __forceinline__ int single_tile_rows(int cap) { return cap ? min(cap, 192) : 192; }

__device__ __forceinline__ float launch_estimate(unsigned long long classes, int n_cols, int steps, int weight_rows, int cus) {
  const float per_cu = 1.f / static_cast<float>(cus);
  float longest = 0.f, sum = 0.f, item = 0.f;
  int n = 0;
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    const int k = (static_cast<int>(classes >> (12 * c)) & 4095) * n_cols;
    if (k == 0) continue;
    const int height = c == 0 ? 320 : 64 * (5 - c);
    item = static_cast<float>(3 * height + 4 * weight_rows) * static_cast<float>(steps) + kItemCost;
    n += k;
    sum += static_cast<float>(k) * item;
    longest = fmaxf(longest, ceilf(static_cast<float>(n) * per_cu) * item);
  }
  return n > cus ? fmaxf(longest, sum * per_cu + 0.6f * item) : longest;
}

// One slot, then one entry of the table per thread.  What bounds it is latency: two dependent rounds of loads and a chain of LDS
// phases.  With four slots per thread of 256 and 64-bit divisions per entry 36 slots took 10.8 us and 64 slots 13.5.
constexpr int kScheduleThreads = 1024, kScheduleWaves = kScheduleThreads / kWave;
static_assert(kScheduleThreads >= PROBE_MAX_SLOTS, "one slot per thread");

__global__ __launch_bounds__(kScheduleThreads) void ffn_schedule_kernel(const int32_t* __restrict__ slot_offsets,
                                                           const void* const* __restrict__ w13_ptrs,
                                                           const void* const* __restrict__ w2_ptrs,
                                                           int S, int max_tiles, int n_cols1, int n_cols2, int steps1, int steps2,
                                                           int cus, int32_t* __restrict__ table) {
  __shared__ alignas(16) int32_t rows_of[PROBE_MAX_SLOTS];
  __shared__ int32_t first_of[PROBE_MAX_SLOTS];
  __shared__ const void* w13_of[PROBE_MAX_SLOTS];
  __shared__ const void* w2_of[PROBE_MAX_SLOTS];
  __shared__ int32_t slot_at[PROBE_MAX_SLOTS];       // slot at each position of the sorted order
  __shared__ int32_t start[PROBE_MAX_SLOTS + 1];     // first tile of each position (exclusive prefix)
  __shared__ unsigned long long class_start[PROBE_MAX_SLOTS + 1];  // the same per tile height, twelve bits each
  __shared__ int32_t wave_tot[kScheduleWaves];
  __shared__ unsigned long long wave_classes[kScheduleWaves];
  __shared__ int32_t n_big;                          // slots of more rows than the single short tiles have
  __shared__ unsigned long long cut_classes[kCuts];  // tiles of each height with each cut
  __shared__ int32_t cut_units, cut_chosen, cut_narrow;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int m = -1;
  const void *w13 = nullptr, *w2 = nullptr;  // on their way until the tiles are counted
  if (tid < S) {
    const int first = slot_offsets[tid];
    m = max(slot_offsets[tid + 1] - first, 0);
    w13 = w13_ptrs[tid];
    w2 = w2_ptrs[tid];
    first_of[tid] = first;
  }
  rows_of[tid] = m;  // entries past S are -1: they come before nobody
  if (tid == 0) n_big = cut_units = cut_chosen = cut_narrow = 0;
  if (tid < kCuts) cut_classes[tid] = 0;
  __syncthreads();
  // position of a slot = number of slots that come before it
  if (tid < S) {
    int pos = 0;
    for (int u0 = 0; u0 < S; u0 += 4) {
      const int4 r4 = *reinterpret_cast<const int4*>(&rows_of[u0]);
      const int ru[4] = {r4.x, r4.y, r4.z, r4.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) pos += (ru[j] > m || (ru[j] == m && u0 + j < tid)) ? 1 : 0;
    }
    slot_at[pos] = tid;
  }
  // Meanwhile the last wave chooses the cut.  Lane l counts the tiles of cut l % 5 in every twelfth slot, then lane
  // (cut, GEMM, width) estimates a launch.
  if (wv == kScheduleWaves - 1) {
    const int cut = lane % kCuts, part = lane / kCuts;
    if (part < kCutParts) {
      unsigned long long counts = 0;
      int units = 0;
      for (int u = part; u < S; u += kCutParts) {
        const int r = rows_of[u];
        counts += cut_slot(r, cut_cap(cut)).classes();
        units = min(units + min((r + 63) >> 6, kCutUnits + 1), kCutUnits + 1);
      }
      atomicAdd(&cut_classes[cut], counts);
      if (cut == 0) atomicAdd(&cut_units, units);
    }
    // the lanes read below what others of the wave have added; LDS operations of a wave are done in order, so this only binds the compiler
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (cut_units <= kCutUnits) {
      const int c = min(lane >> 2, kCuts - 1), second = (lane >> 1) & 1, narrow = lane & 1;
      const int n_cols = second ? (narrow ? (steps1 + 1) / 2 : n_cols2) : (narrow ? steps2 : n_cols1);  // columns of a k-step's 64: H, F
      const unsigned long long counts = cut_classes[c];
      const float t = launch_estimate(counts, n_cols, second ? steps2 : steps1, 256 >> narrow, cus);
      const float other = __shfl_xor(t, 1, kWave), best = fminf(t, other);      // the better width of this GEMM
      const float both = best + __shfl_xor(best, 2, kWave);                     // both GEMMs with this cut
      const bool fits = c == 0 || tiles_of(counts) <= max_tiles;
      const float standard = __shfl(both, 0, kWave);
      const float mine = c == 0 ? kCutGain * standard : fits ? both : 3.0e38f;
      float least = mine;
#pragma unroll
      for (int d = 4; d < kWave; d <<= 1) least = fminf(least, __shfl_xor(least, d, kWave));
      const unsigned long long at = __ballot(lane < 4 * kCuts && mine == least);
      const int chosen = __builtin_ctzll(at) >> 2;
      const unsigned widths = static_cast<unsigned>(__ballot(narrow && t < other) >> (4 * chosen));
      if (lane == 0) {
        cut_chosen = chosen;
        cut_narrow = ((widths >> 1) & 1) | ((widths >> 2) & 2);
      }
    }
  }
  __syncthreads();
  const int cap = cut_cap(__builtin_amdgcn_readfirstlane(cut_chosen));
  const int big_here = __popcll(__ballot(m > single_tile_rows(cap)));
  if (lane == 0 && big_here) atomicAdd(&n_big, big_here);
  // exclusive prefix of tiles over the positions
  const SlotCut my_cut = tid < S ? cut_slot(rows_of[slot_at[tid]], cap) : SlotCut{0, 0, 0, 0, 0};
  const int tiles = my_cut.tiles();
  const unsigned long long classes = my_cut.classes();
  int incl = tiles;
  unsigned long long c_incl = classes;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int o = __shfl_up(incl, d, kWave);
    const unsigned long long co = __shfl_up(c_incl, d, kWave);
    if (lane >= d) {
      incl += o;
      c_incl += co;
    }
  }
  if (S > kWave) {
    if (lane == kWave - 1) {
      wave_tot[wv] = incl;
      wave_classes[wv] = c_incl;
    }
    __syncthreads();
    for (int i = 0; i < wv; ++i) {
      incl += wave_tot[i];
      c_incl += wave_classes[i];
    }
  }
  if (tid < S) {
    w13_of[tid] = w13;
    w2_of[tid] = w2;
    start[tid] = incl - tiles;
    class_start[tid] = c_incl - classes;
    if (tid == S - 1) {
      start[S] = incl;
      class_start[S] = c_incl;
    }
  }
  __syncthreads();
  // the same in all lanes: in scalar registers, so that what follows is branched over where it is not wanted
  const int total = __builtin_amdgcn_readfirstlane(min(start[S], max_tiles));
  const unsigned long long heights = class_start[S];
  const unsigned long long all_classes =
      static_cast<unsigned long long>(static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(heights >> 32)))) << 32 |
      static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(heights)));
  // taller than 192 rows; beyond 4095 tiles the twelve-bit fields run into each other and are not looked at
  const int n_tall = static_cast<int>(all_classes & 4095) + static_cast<int>((all_classes >> 12) & 4095);
  const bool narrow1 = (cut_narrow & 1) != 0, narrow2 = (cut_narrow & 2) != 0;
  const int cols1 = narrow1 ? steps2 : n_cols1;
  const bool tall_first = (cap == 0 || cap > 192) && start[S] <= min(max_tiles, 4095) && n_tall * cols1 <= cus &&
                          static_cast<long>(start[S]) * cols1 > cus;
  if (tid < kTableHeaderInts) {
    // the queues' tickets: the first ones go without a draw, to the workgroups in order
    int v = tid >= kQueue1 && tid < kQueue2 + kXcds ? (cus + kXcds - 1 - tid % kXcds) / kXcds : 0;
    if (tid == 0) v = total;
    if (tid == kNarrow1) v = narrow1;
    if (tid == kNarrow2) v = narrow2;
    table[tid] = v;
  }
  TileEntry* entries = reinterpret_cast<TileEntry*>(table + kTableHeaderInts);
  // positions [0, n_big) hold the slots of more rows: tiles [0, nb) are theirs, the ns single short tiles follow
  const int nb = min(start[n_big], total), ns = total - nb;
  const bool small = total < (1 << 16);  // products of two of them in 32 bits
  for (int p = tid; p < total; p += kScheduleThreads) {
    // entry p of the table: the short tiles are spread evenly over the table
    int before, until;
    if (small) {
      before = static_cast<int>(static_cast<unsigned>(p) * static_cast<unsigned>(ns) / static_cast<unsigned>(total));
      until = static_cast<int>(static_cast<unsigned>(p + 1) * static_cast<unsigned>(ns) / static_cast<unsigned>(total));
    } else {
      before = static_cast<int>(static_cast<long>(p) * ns / total);
      until = static_cast<int>(static_cast<long>(p + 1) * ns / total);
    }
    const bool is_short = until > before;
    const int t = tall_first ? p : (is_short ? nb + before : p - before);
    int lo = 0, hi = S;  // last position with start[position] <= t
    while (hi - lo > 1) {
      int mid = (lo + hi) >> 1;
      if (start[mid] <= t) lo = mid; else hi = mid;
    }
    const int slot = slot_at[lo], first = first_of[slot];
    const SlotCut c = cut_slot(rows_of[slot], cap);
    int i = t - start[lo], row0 = first, height;
    if (i < c.n320) {
      row0 += i * 320;
      height = 320;
    } else if ((i -= c.n320) < c.n256) {
      row0 += c.n320 * 320 + i * 256;
      height = 256;
    } else if ((i -= c.n256) < c.n_cap) {
      row0 += i * c.cap;
      height = c.cap;
    } else {
      i = 0;
      row0 += c.n320 * 320 + c.n256 * 256 + c.n_cap * c.cap;
      height = c.tail;
    }
    int at = p;
    if (tall_first) {  // taller tiles first: the tiles of its height in the slots before it, and all taller ones
      const int cls = SlotCut::height_class(height);
      at = i + static_cast<int>((class_start[lo] >> (12 * cls)) & 4095);
      for (int q = 0; q < cls; ++q) at += static_cast<int>((class_start[S] >> (12 * q)) & 4095);
    }
    TileEntry e;
    e.row0 = row0;
    e.rows = first + rows_of[slot] - row0;
    e.height = height;
    e.slot = slot;
    e.w13 = w13_of[slot];
    e.w2 = w2_of[slot];
    entries[at] = e;
  }
}

template <int MI, int NI>
__device__ __forceinline__ void zero_acc(f32x4 (&acc)[2 * MI][2 * NI]) {
#pragma unroll
  for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
    for (int j = 0; j < 2 * NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
}


// ---- workgroup -> (row tile, column block) -----------------------------------------------
// Workgroups are dealt to the 8 XCDs round-robin by their linear id, and each XCD has its own
// L2.  The launch is one-dimensional; workgroup L is the (L / 8)-th of XCD L % 8.  Work items
// are numbered so that the 32 workgroups an XCD runs side by side form a compact 8 x 4 block
// (8 consecutive row tiles x 4 consecutive column blocks): per k-step they pull 12 distinct
// operand slices through that L2 instead of 18 for a 16 x 2 strip.  Blocks at the edges are smaller and
// no number is left out: with 384 numbers for the 230 items of 10 tiles x 23 columns every third draw of the
// queue named none.
__device__ __forceinline__ bool ffn_item_of(int q, int n_tiles, int n_cols, int& tile, int& col) {
  if (q >= n_tiles * n_cols) return false;
  // tile groups slowest, then the column groups of a tile group, then the tiles of a block
  const int tg = q / (kBlkM * n_cols), in_group = q - tg * kBlkM * n_cols;
  const int rows = min(kBlkM, n_tiles - tg * kBlkM);  // tiles of the group
  const int cg = in_group / (rows * kBlkN), in_block = in_group - cg * rows * kBlkN;
  const int width = min(kBlkN, n_cols - cg * kBlkN);
  const int t = in_block / width;
  tile = tg * kBlkM + t;
  col = cg * kBlkN + in_block - t * width;
  return true;
}

// Item number of ticket t of XCD x: chunks of 32 items are dealt to the XCDs round-robin; fewer items than that makes for all
// eight are dealt in eight even chunks.
__device__ __forceinline__ int ffn_item_number(int t, int x, int n_items) {
  if (n_items > kXcds * kBlk) return ((t / kBlk) * kXcds + x) * kBlk + t % kBlk;
  const int chunk = (n_items + kXcds - 1) / kXcds;
  return t < chunk ? x * chunk + t : n_items;
}

// Work queue of the persistent launch (one workgroup per CU).  Chunks of 32 items are dealt to the XCDs
// round-robin as above (chunk b belongs to XCD b % 8), but which workgroup runs which item is decided at
// run time: a workgroup draws tickets from the counter of the XCD it runs on, so the 32 workgroups of an XCD
// still walk one block side by side; when its own XCD's chunks are used up it looks at all eight counters and
// draws from the next one that has tickets left.  Counters only grow and nobody waits for anybody: a draw that
// names no item means a counter that the next look leaves out, so every workgroup ends after at most 8 of them.
// What bounds a call of a few items per CU is the way in and out.  The first item is nobody's to draw: workgroup L takes ticket L / 8 of
// XCD L % 8, and the counters begin behind those (schedule kernel).  At the end one look at the counters (1 us) takes the place of a draw
// from each, which at one to two items per CU was 4 to 20 us of a call: 704 x 1408 with 44 row tiles 72.8 -> 49.1 us, 1024 x 2304 with
// 15 68 -> 59, 768 tokens of 2880 x 2880 150 -> 141; calls of many items gain up to 1 %.  One workgroup per item, without the queue,
// is not faster any more at any size (4096 x 14336, 160 wide items of gemm2 718 -> 693).
struct WorkQueue {
  int32_t* counters;  // [8], set by the schedule kernel
  int victim;         // the XCD whose counter is drawn from
  __device__ __forceinline__ void init(int32_t* c) { counters = c; }
  // The workgroup's first item; false if there is none (and no other for it either: fewer items than workgroups).
  __device__ __forceinline__ bool first(int n_tiles, int n_cols, int& tile, int& col) {
    victim = __builtin_amdgcn_s_getreg((20 << 0) | (0 << 6) | (3 << 11)) & (kXcds - 1);  // XCC_ID
    return ffn_item_of(ffn_item_number(blockIdx.x / kXcds, blockIdx.x % kXcds, n_tiles * n_cols), n_tiles, n_cols, tile, col);
  }
  // All threads of the workgroup call this together; slot is two ints of static LDS.  used_up: the victim is known to be used up.
  __device__ __forceinline__ bool next(bool used_up, int n_tiles, int n_cols, volatile int* slot, int& tile, int& col) {
    const int n_items = n_tiles * n_cols;
    __syncthreads();  // the previous item is finished by every wave (LDS stages, slot)
    if (threadIdx.x < kWave) {
      const int lane = threadIdx.x;
      int q = n_items;
      while (true) {
        if (!used_up) {
          int t = 0;
          if (lane == 0) t = atomicAdd(&counters[victim], 1);
          q = ffn_item_number(__builtin_amdgcn_readfirstlane(t), victim, n_items);
          if (q < n_items) break;
        }
        const int drawn = __hip_atomic_load(&counters[lane & (kXcds - 1)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned left = static_cast<unsigned>(__ballot(ffn_item_number(drawn, lane & (kXcds - 1), n_items) < n_items)) & ((1u << kXcds) - 1);
        if (!left) break;
        const unsigned from = left * ((1u << kXcds) + 1) >> victim;  // bit i: counter (victim + i) % 8
        victim = (victim + __builtin_ctz(from)) & (kXcds - 1);
        used_up = false;
      }
      if (lane == 0) {
        slot[0] = q;
        slot[1] = victim;
      }
    }
    __syncthreads();
    victim = __builtin_amdgcn_readfirstlane(slot[1]);
    return ffn_item_of(__builtin_amdgcn_readfirstlane(slot[0]), n_tiles, n_cols, tile, col);
  }
  // The same when thread 0 has already drawn a ticket during the last k-steps of the previous item (gemm_mainloop,
  // DRAW) and every wave is past that loop's last barrier: no barrier is needed to read it, and none before the next
  // item's loads either, because no wave reads the LDS stages after that barrier.  Falls back to next() when the
  // ticket names no item.
  __device__ __forceinline__ bool next_drawn(bool drew, int n_tiles, int n_cols, volatile int* slot, int& tile,
                                             int& col) {
    if (drew && ffn_item_of(ffn_item_number(__builtin_amdgcn_readfirstlane(slot[0]), victim, n_tiles * n_cols), n_tiles, n_cols, tile, col)) return true;
    return next(drew, n_tiles, n_cols, slot, tile, col);
  }
};

// ---- 1. gemm1 + SwiGLU ----------------------------------------------------------------
// Where the activation rows of gemm1 come from: the permuted copy xp (row r of the row space), or,
// gathered on load, the token rows themselves: row r is x[row_pair[r] / k] (no xp is ever written).
struct RowSource {
  const bf16_t* base;         // xp, or x when gathering
  const int32_t* row_pair;    // nullptr = rows are stored in row-space order
  int k, n_tokens;
};

__device__ __forceinline__ float swiglu(float gate, float up) { return gate / (1.f + __expf(-gate)) * up; }

// NI = 32-row weight fragments per wave: 2 = a column block of 128 h columns (128 gate + 128 up weight
// rows per workgroup), 1 = 64 h columns (the skinny tiles of the decode schedule).  NST = LDS stages.
template <int MI, bool GATHER, int NI = 2, int NST = (MI >= 3 ? 2 : 3), bool DRAW = false, bool SPLIT = false>
__device__ __forceinline__ bool gemm1_tile(const RowSource& src, const bf16_t* __restrict__ w13,
                                           int row0, int rows, int n0, int n_end, int H, int F,
                                           bf16_t* __restrict__ hbuf, u32x4* smem, int32_t* draw_counter = nullptr,
                                           volatile int* draw_slot = nullptr, int k0 = 0, int klen = 0,
                                           float* partial = nullptr, int k_start = 0) {
  // SPLIT: only k0 .. k0 + klen - 1 of the contraction; the fp32 sums go to partial[row of the tile][gate F | up F].
  // rows = valid rows from row0 to the end of the slot (may exceed the tile height); columns n0 .. n_end - 1, which may be fewer
  // than a column block has
  constexpr int HALF = 16 * NI;  // h columns per wave; its 32*NI weight rows are HALF gate rows, then the HALF up rows
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wv / 4, wn = wv % 4;
  __amdgpu_buffer_rsrc_t rA =
      GATHER ? make_rsrc(src.base, static_cast<size_t>(src.n_tokens) * H * 2)
             : make_rsrc(src.base + static_cast<size_t>(row0) * H, static_cast<size_t>(rows) * H * 2);
  __amdgpu_buffer_rsrc_t rB = make_rsrc(w13, static_cast<size_t>(2) * F * H * 2);
  int voff[MI + 2 * NI];
  dma_offsets<MI>(wv, lane, H * 2,
                  [&](int r) {
                    // a tile row past the slot's last row gets an offset past the end of the descriptor: the
                    // load returns zeros, which also cost the matrix cores less than a copy of a real row
                    if (!GATHER) return r;
                    if (r >= rows) return src.n_tokens;
                    const int pair = src.row_pair[row0 + r];  // a valid row always names a pair
                    return min(max(pair, 0) / src.k, src.n_tokens - 1);
                  },
                  voff);
  // weight tile row j: wave column block q = j / (2 HALF), row r inside it.  NI = 2: HALF gate rows, then the HALF
  // up rows (B fragments 0, 1 / 2, 3 of the wave).  NI = 1: gate and up rows in alternating runs of four, which makes
  // the main loop's fragment 0 the sixteen gate rows and fragment 1 the up rows.
  dma_offsets<2 * NI, true>(wv, lane, H * 2,
                            [&](int j) {
                              const int q = j / (2 * HALF), r = j % (2 * HALF);
                              const bool up = NI == 2 ? r >= HALF : (r >> 2) & 1;
                              const int c = NI == 2 ? r % HALF : ((r >> 3) << 2) | (r & 3);
                              const int f = n0 + HALF * q + c;
                              if (f >= n_end) return 2 * F;  // past the descriptor: zeros without traffic, masked at the store
                              return up ? F + f : f;
                            },
                            voff + MI);
  f32x4 acc[2 * MI][2 * NI];
  zero_acc<MI, NI>(acc);
  const bool drew =
      gemm_mainloop<MI, NI, 1, NST, true, DRAW, NI == 1>(rA, rB, voff, SPLIT ? k0 : 0, SPLIT ? klen : H, smem, wv, lane,
                                                         acc, draw_counter, draw_slot, k_start);

  // NI = 2: acc[i][0..1] are eight consecutive gate columns of one output row, acc[i][2..3] the up columns (see
  // gemm_mainloop, PERM): one 16-byte store.  NI = 1: four of each, 8 bytes.  The stores go through a buffer
  // descriptor that ends with the tile's last valid row, so rows past it are dropped by the
  // bounds check instead of a branch.
  const int valid = min(rows, 64 * MI);
  __amdgpu_buffer_rsrc_t rH = make_rsrc(hbuf + static_cast<size_t>(row0) * F, static_cast<size_t>(valid) * F * 2);
  const int row_in = 32 * MI * wm + (lane & 15);
  const int cbase = n0 + HALF * wn + 4 * NI * (lane >> 4);
  if constexpr (SPLIT) {
    static_assert(NI == 1, "four columns per lane");
    __amdgpu_buffer_rsrc_t rP = make_rsrc(partial, static_cast<size_t>(valid) * 2 * F * 4);
    if (cbase < n_end) {
#pragma unroll
      for (int i = 0; i < 2 * MI; ++i) {
        const int off = ((row_in + 16 * i) * 2 * F + cbase) * 4;
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][0]), rP, off, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][1]), rP, off + F * 4, 0, 0);
      }
    }
    return drew;
  }
  if (cbase < n_end) {  // n_end % 8 == 0: a group of 4 * NI columns is in or out as a whole
#pragma unroll
    for (int i = 0; i < 2 * MI; ++i) {
      const int off = ((row_in + 16 * i) * F + cbase) * 2;
      uint32_t pk[2 * NI];
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        float hv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float gt = acc[i][j][e], up = acc[i][NI + j][e];
          hv[e] = swiglu(gt, up);
        }
        pk[2 * j] = pack_bf16x2(hv[0], hv[1]);
        pk[2 * j + 1] = pack_bf16x2(hv[2], hv[3]);
      }
      if constexpr (NI == 2)
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{pk[0], pk[1], pk[2], pk[3]}, rH, off, 0, 0);
      else
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{pk[0], pk[1]}, rH, off, 0, 0);
    }
  }
  return drew;
}

// one-dimensional launch over (row tile, column block) work items; a column block is 64 NI gate + 64 NI up weight rows
template <bool GATHER, int NI>
__device__ __forceinline__ void ffn_gemm1_items(const RowSource& src, const int32_t* __restrict__ table, int32_t* table_rw,
                                                int H, int F, bf16_t* __restrict__ hbuf, u32x4* smem,
                                                volatile int* ticket) {
  constexpr int COLS = 64 * NI;
  const int n_tiles = table[0], n_cols = (F + COLS - 1) / COLS;
  int tile, col;
  auto run = [&](int32_t* ctr) {
    const TileEntry e = reinterpret_cast<const TileEntry*>(table + kTableHeaderInts)[tile];
    const int n0 = col * COLS;
    const bf16_t* w13 = static_cast<const bf16_t*>(e.w13);
    if (e.height > 256)
      return gemm1_tile<5, GATHER, NI, ffn_stages(5, NI), true>(src, w13, e.row0, e.rows, n0, F, H, F, hbuf, smem, ctr, ticket);
    if (e.height > 192)
      return gemm1_tile<4, GATHER, NI, ffn_stages(4, NI), true>(src, w13, e.row0, e.rows, n0, F, H, F, hbuf, smem, ctr, ticket);
    if (e.height > 128)
      return gemm1_tile<3, GATHER, NI, ffn_stages(3, NI), true>(src, w13, e.row0, e.rows, n0, F, H, F, hbuf, smem, ctr, ticket);
    if (e.height > 64)
      return gemm1_tile<2, GATHER, NI, ffn_stages(2, NI), true>(src, w13, e.row0, e.rows, n0, F, H, F, hbuf, smem, ctr, ticket);
    return gemm1_tile<1, GATHER, NI, ffn_stages(1, NI), true>(src, w13, e.row0, e.rows, n0, F, H, F, hbuf, smem, ctr, ticket);
  };
  // the ticket of the next item is drawn while the last k-steps of this one run
  WorkQueue wq;
  wq.init(table_rw + kQueue1);
  bool more = wq.first(n_tiles, n_cols, tile, col);
  while (more) {
    const bool drew = run(wq.counters + wq.victim);
    more = wq.next_drawn(drew, n_tiles, n_cols, ticket, tile, col);
  }
}

template <bool GATHER>
__global__ __launch_bounds__(512, 2) void ffn_gemm1_kernel(RowSource src, const int32_t* __restrict__ table,
                                                           int32_t* table_rw, int H, int F,
                                                           bf16_t* __restrict__ hbuf) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ u32x4 smem[];
  __shared__ int ticket[2];
  if (table[kNarrow1])
    ffn_gemm1_items<GATHER, 1>(src, table, table_rw, H, F, hbuf, smem, ticket);
  else
    ffn_gemm1_items<GATHER, 2>(src, table, table_rw, H, F, hbuf, smem, ticket);
#endif
}

// ---- 2. gemm2 -------------------------------------------------------------------------
template <int MI, int NI = 2, int NST = (MI >= 3 ? 2 : 3), bool DRAW = false, bool SPLIT = false, bool LAST = false>
__device__ __forceinline__ bool gemm2_tile(const bf16_t* __restrict__ hbuf, const bf16_t* __restrict__ w2,
                                           int row0, int rows, int n0, int n_end, int H, int F,
                                           bf16_t* __restrict__ y, u32x4* smem, int32_t* draw_counter = nullptr,
                                           volatile int* draw_slot = nullptr, int k0 = 0, int klen = 0,
                                           float* partial = nullptr, int k_start = 0, int piece = 0, int pieces = 1,
                                           uint32_t* arrivals = nullptr, int item = 0) {
  // SPLIT: only k0 .. k0 + klen - 1 of the contraction, piece `piece` of `pieces`.  The fp32 sums go to partial[piece][row of
  // the tile][H]; LAST: the workgroup that counts as the last of its item adds them, otherwise ffn_skinny_add_kernel does.
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wv / 4, wn = wv % 4;
  __amdgpu_buffer_rsrc_t rA = make_rsrc(hbuf + static_cast<size_t>(row0) * F, static_cast<size_t>(rows) * F * 2);
  __amdgpu_buffer_rsrc_t rB = make_rsrc(w2, static_cast<size_t>(H) * F * 2);
  int voff[MI + 2 * NI];
  dma_offsets<MI>(wv, lane, F * 2, [&](int r) { return r; }, voff);  // rows past the slot read as zeros (out of range)
  dma_offsets<2 * NI, true>(wv, lane, F * 2, [&](int j) { return n0 + j < n_end ? n0 + j : H; }, voff + MI);
  f32x4 acc[2 * MI][2 * NI];
  zero_acc<MI, NI>(acc);
  const bool drew =
      gemm_mainloop<MI, NI, 1, NST, true, DRAW, NI == 1>(rA, rB, voff, SPLIT ? k0 : 0, SPLIT ? klen : F, smem, wv, lane,
                                                         acc, draw_counter, draw_slot, k_start);

  const int valid = min(rows, 64 * MI);  // rows past it are dropped by the descriptor's bounds check
  __amdgpu_buffer_rsrc_t rY = make_rsrc(y + static_cast<size_t>(row0) * H, static_cast<size_t>(valid) * H * 2);
  const int row_in = 32 * MI * wm + (lane & 15);
  if constexpr (SPLIT) {
    // Stores and loads of the last workgroup's sums at device scope (sc1): the pieces of an item run on different XCDs, whose L2s do not see one another.
    constexpr int kDeviceScope = 16, kScope = LAST ? kDeviceScope : 0;
    const size_t piece_floats = static_cast<size_t>(64 * MI) * H;
    auto offset_of = [&](int i, int q) { return ((row_in + 16 * i) * H + n0 + 32 * NI * wn + 32 * q + 8 * (lane >> 4)) * 4; };
    auto in_range = [&](int q) { return n0 + 32 * NI * wn + 32 * q + 8 * (lane >> 4) < n_end; };
    __amdgpu_buffer_rsrc_t rP = make_rsrc(partial + piece * piece_floats, static_cast<size_t>(valid) * H * 4);
#pragma unroll
    for (int i = 0; i < 2 * MI; ++i) {
#pragma unroll
      for (int q = 0; q < NI; ++q) {
        if (in_range(q)) {
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][2 * q]), rP, offset_of(i, q), 0, kScope);
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][2 * q + 1]), rP, offset_of(i, q) + 16, 0, kScope);
        }
      }
    }
    if constexpr (!LAST) return drew;
    // every wave's stores have arrived before the workgroup counts itself in: four items to a word, one byte each
    __shared__ int last;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0)
      last = static_cast<int>((atomicAdd(&arrivals[item >> 2], 1u << (8 * (item & 3))) >> (8 * (item & 3))) & 255u) == pieces - 1;
    __syncthreads();
    if (!last) return drew;
    // the sums in ascending order of the pieces, whichever came last
#pragma unroll
    for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
      for (int j = 0; j < 2 * NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int BATCH = 2;  // pieces whose loads are in flight together
    for (int p0 = 0; p0 < pieces; p0 += BATCH) {
      f32x4 v[BATCH][2 * MI][2 * NI];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        __amdgpu_buffer_rsrc_t rQ = make_rsrc(partial + min(p0 + u, pieces - 1) * piece_floats, static_cast<size_t>(valid) * H * 4);
#pragma unroll
        for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
          for (int q = 0; q < NI; ++q) {
            v[u][i][2 * q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rQ, offset_of(i, q), 0, kDeviceScope));
            v[u][i][2 * q + 1] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rQ, offset_of(i, q) + 16, 0, kDeviceScope));
          }
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u)
        if (p0 + u < pieces) {
#pragma unroll
          for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
            for (int j = 0; j < 2 * NI; ++j) acc[i][j] += v[u][i][j];
        }
    }
  }
#pragma unroll
  for (int i = 0; i < 2 * MI; ++i) {
#pragma unroll
    for (int q = 0; q < NI; ++q) {
      const int cbase = n0 + 32 * NI * wn + 32 * q + 8 * (lane >> 4);
      const int off = ((row_in + 16 * i) * H + cbase) * 2;
      if (cbase < n_end) {
        u32x4 pk;
        pk[0] = pack_bf16x2(acc[i][2 * q][0], acc[i][2 * q][1]);
        pk[1] = pack_bf16x2(acc[i][2 * q][2], acc[i][2 * q][3]);
        pk[2] = pack_bf16x2(acc[i][2 * q + 1][0], acc[i][2 * q + 1][1]);
        pk[3] = pack_bf16x2(acc[i][2 * q + 1][2], acc[i][2 * q + 1][3]);
        __builtin_amdgcn_raw_buffer_store_b128(pk, rY, off, 0, 0);
      }
    }
  }
  return drew;
}

// one-dimensional launch over (row tile, column block of 128 NI output columns) work items
template <int NI>
__device__ __forceinline__ void ffn_gemm2_items(const bf16_t* __restrict__ hbuf, const int32_t* __restrict__ table,
                                                int32_t* table_rw, int H, int F, bf16_t* __restrict__ y,
                                                u32x4* smem, volatile int* ticket) {
  constexpr int COLS = 128 * NI;
  const int n_tiles = table[0], n_cols = (H + COLS - 1) / COLS;
  int tile, col;
  auto run = [&](int32_t* ctr) {
    const TileEntry e = reinterpret_cast<const TileEntry*>(table + kTableHeaderInts)[tile];
    const int n0 = col * COLS;
    const bf16_t* w2 = static_cast<const bf16_t*>(e.w2);
    if (e.height > 256) return gemm2_tile<5, NI, ffn_stages(5, NI), true>(hbuf, w2, e.row0, e.rows, n0, H, H, F, y, smem, ctr, ticket);
    if (e.height > 192) return gemm2_tile<4, NI, ffn_stages(4, NI), true>(hbuf, w2, e.row0, e.rows, n0, H, H, F, y, smem, ctr, ticket);
    if (e.height > 128) return gemm2_tile<3, NI, ffn_stages(3, NI), true>(hbuf, w2, e.row0, e.rows, n0, H, H, F, y, smem, ctr, ticket);
    if (e.height > 64) return gemm2_tile<2, NI, ffn_stages(2, NI), true>(hbuf, w2, e.row0, e.rows, n0, H, H, F, y, smem, ctr, ticket);
    return gemm2_tile<1, NI, ffn_stages(1, NI), true>(hbuf, w2, e.row0, e.rows, n0, H, H, F, y, smem, ctr, ticket);
  };
  WorkQueue wq;
  wq.init(table_rw + kQueue2);
  bool more = wq.first(n_tiles, n_cols, tile, col);
  while (more) {
    const bool drew = run(wq.counters + wq.victim);
    more = wq.next_drawn(drew, n_tiles, n_cols, ticket, tile, col);
  }
}

__global__ __launch_bounds__(512, 2) void ffn_gemm2_kernel(const bf16_t* __restrict__ hbuf,
                                                           const int32_t* __restrict__ table, int32_t* table_rw,
                                                           int H, int F, bf16_t* __restrict__ y) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ u32x4 smem[];
  __shared__ int ticket[2];
  if (table[kNarrow2])
    ffn_gemm2_items<1>(hbuf, table, table_rw, H, F, y, smem, ticket);
  else
    ffn_gemm2_items<2>(hbuf, table, table_rw, H, F, y, smem, ticket);
#endif
}

// ---- decode schedule: skinny tiles -------------------------------------------------------------
// When every slot holds a few rows (a decode step: rows per slot of the order of ten), the grouped GEMM does
// almost no arithmetic per weight byte (the small-n end of eta_g(n), Sec. 3.2) and the call is a stream
// of every active slot's weights through the chip.  What matters then is that every CU pulls a distinct
// slice at all times, so the work is cut finer and kept resident: tiles of 64 rows x 64 h columns (gemm1:
// 64 gate + 64 up weight rows) or 64 rows x 128 output columns (gemm2), three LDS stages of 24 KB, two
// workgroups per CU (sixteen waves, 72 KB of LDS each), one work item per workgroup in slot order.  A
// slot with more than 64 rows is simply several row tiles: correct for any input, tuned for short slots.
constexpr int kSkinnyLdsBytes = 3 * (64 + 128) * 128;  // 72 KB
constexpr int kSkinnyCols1 = 64, kSkinnyCols2 = 128;   // h columns / y columns per work item

// Few tiles.  A call with one or two active slots (a single token; a shared expert) has fewer items than the chip has
// CUs, and an item streams its weights no faster than about 50 GB/s.  The contraction is then cut into pieces, as many
// as give every CU one item: each leaves its fp32 sums in the workspace, and they are added in ascending order.  The number
// of tiles is known on the device only.  A second kernel adds the pieces; the host decides whether the tiles can be few
// (skinny_may_split) and then launches it, and it ends at once if nothing was split.  Few pieces of few rows of gemm2 are added by the
// workgroup that counts as the last of its item instead, on counters that gemm1's launch clears (skinny_last_adds).
// One token, two experts of 4096 x 14336: FFN 194 -> 137 us (gemm2 104 -> 41, adding 5); 512 items instead of 256: 141,
// 1024: 161.  One slot of 75 rows, 7168 x 2048, which took the tall tiles before: 125 -> 43 us.
constexpr int kSkinnyItems = 256;
constexpr int kSkinnyMinSteps = 16;      // k-steps of a piece at least
// k-steps from which a contraction may be cut.  Shorter ones gain less over the adding kernel's launch (about 5 us), but some
// still do: uncut / cut one slot of 16 rows, 3072 x 1536 28.3 / 24.1 us; two of 2880 x 2880 47.5 / 41.2, four 52.4 / 52.3.
constexpr int kSkinnySplitSteps = 64;
// Where the last workgroup adds, pieces have 13 k-steps and more, and contractions of 32 to 63 are cut as well, into as many pieces as
// give 192 items.  That costs about as much as ten to sixteen k-steps, and the sums of many rows more.  In a hot loop (weights in
// the last-level cache; from HBM every cut below gains 3 to 16 us) uncut / cut: one slot of 64 rows of 2880 x 2880 (23 items of 45
// k-steps) 33.2 / 30.6 us, two 34.4 / 33.8, three of 16 rows 33.5 / 31.8; 64 rows of 4096 x 3968 (32 of 62) 42.6 / 37.0; but full
// tiles in 48 items of 56 k-steps 0.6 us slower, in 64 up to 2.8, in 92 (256 rows of 2880 x 2880) 41.9 / 44.3, in 96 (24 slots of 512 x
// 2112) 38.6 / 43.9; 80 items of 32 k-steps and 16 rows 0.7 slower, 72 of one row level.
constexpr int kSkinnyShortSteps = 32, kSkinnyLastMinSteps = 13, kSkinnyShortItems = 192;
constexpr int kSkinnyShortCut = 72;    // items that are cut at most; their rows x column blocks: 32 per k-step
constexpr int kSkinnyShortFull = 46;   // from 40 k-steps on: items that are cut whatever their rows
constexpr int kSkinnyFewItems = 512;     // items at capacity up to which tiles can be few
constexpr size_t kSkinnyPartialBytes = static_cast<size_t>(kSkinnyItems) * 64 * 128 * sizeof(float);
// Items that are cut number at most half of kSkinnyItems: a byte each counts the pieces that have arrived.  They lie in the tile table,
// which the decode schedule does not use and which is never shorter.
constexpr int kArrivalWords = kSkinnyItems / 2 / 4;
static_assert(kArrivalWords * sizeof(uint32_t) <= kTableHeaderInts * sizeof(int32_t) && kSkinnyItems <= 256, "bytes of the table header");

// most row tiles that max_rows rows in S slots can give: every tile has a row, every slot one tile that is not full
static int skinny_max_tiles(int S, int max_rows) {
  return std::min<long>(max_rows, (static_cast<long>(max_rows) + 63l * S) / 64);
}
// Whether the contraction of `steps` k-steps, over n_cols column blocks, may be cut: few items at capacity, and a cut
// that is still possible if every slot that probably holds rows does.  Most of the capacity is as a rule other ranks' (one
// token, eight experts, one of them local, 36 slots of 7168 x 2048: FFN 70.9 -> 36.7 us; eight slots of 7168 x 256, 421 of 3200
// rows local: 68.8 -> 45.2; all eight experts local: 127.1 / 125.4).  But with kSkinnyFullRows rows of capacity per slot nearly
// every slot holds one, and if an eighth of the capacity is local it fills a tile more per 512 rows.  Where that many tiles
// leave no second piece the launch of the adding kernel would be lost (12 slots of 5632 x 1408, 480 rows of capacity, five in
// each: 133.5 without, 137.2 with it; 32 slots of 6912 x 256, 401 rows under a Zipf law 92.2 / 99.9).
constexpr int kSkinnyFullRows = 8;
static bool skinny_may_split(int S, int max_rows, int n_cols, int steps) {  // if it holds, it holds for fewer rows too
  const long most = skinny_max_tiles(S, max_rows);
  if (steps < kSkinnySplitSteps || most * n_cols > kSkinnyFewItems) return false;
  const bool every_slot = max_rows >= static_cast<long>(kSkinnyFullRows) * S;
  return !every_slot || std::min<long>(most, S + (static_cast<long>(max_rows) + 511) / 512) * n_cols <= kSkinnyItems / 2;
}
// Whether gemm2's pieces are added by the last workgroup of an item and not by the adding kernel, which has a workgroup for every row.
// From 64 k-steps on, call by that kernel / by the last, hot loop: two pieces 63.6 / 60.3 us (three slots of 4096 x 4096, a row in
// each) and three 70 / 67 (two of 5120 x 4608) whatever the rows up to 32; four or five of a single tile 20.5 / 19.0 (one row of 1024 x
// 4608), 25.1 / 24.0 (16 rows of 2048 x 4608), 32 rows level, 48 one us slower; three or four tiles of 2048 x 4096 are 0.5 to
// 1 us slower, two of 3072 x 5120 one, and two of 2048 x 4096 0.5 faster.  Six: up to eight rows 0.2 to 0.9 faster in one tile, 0.5
// slower in two of 2048 x 5120.  Seven and eight: two tiles of 4096 x 14336 (one token, two experts) 128.9 / 126.8, but a single one
// of 4096 x 8192 0.4 slower, of 2048 x 8320 25.8 / 27.4.  16 pieces of one row of 1024 x 16384 25.8 / 29.8.
static bool skinny_last_adds(int S, int max_rows, int n_cols, int steps) {
  const long tiles = skinny_max_tiles(S, max_rows);
  if (steps < kSkinnyShortSteps || tiles * n_cols > kSkinnyFewItems) return false;
  if (steps < kSkinnySplitSteps) return true;
  // row tiles, and rows of each, if every slot that probably holds rows does
  const int likely = max_rows >= static_cast<long>(kSkinnyFullRows) * S ? S : 1, rows = max_rows / likely;
  const int pieces = std::min(kSkinnyItems / (likely * n_cols), steps / kSkinnyLastMinSteps);
  if (pieces > 8 || max_rows > 48) return false;
  if (pieces <= 3) return rows <= 32;
  if (pieces <= 5) return rows <= 32 && (likely == 1 || n_cols >= 32 || likely * n_cols <= 32);
  if (tiles > 1 && n_cols >= 24) return rows <= 16;
  return pieces == 6 ? rows <= 8 && (tiles == 1 || tiles * n_cols <= 16) : rows <= 4 && tiles * n_cols <= 8;
}
// k-steps per piece of a contraction of `steps`, `items` = row tiles x column blocks of `rows` rows; 0 if it is not cut.  LAST: the
// last workgroup adds, and `steps` may be below kSkinnySplitSteps.
template <bool LAST>
__device__ __forceinline__ int skinny_steps(int items, int rows, int n_cols, int steps) {
  if (items <= 0) return 0;
  int most = kSkinnyItems;
  if (LAST && steps < kSkinnySplitSteps) {
    most = kSkinnyShortItems;
    if (!(items <= kSkinnyShortCut && rows * n_cols <= kSkinnyShortSteps * steps) && !(items <= kSkinnyShortFull && steps >= 40)) return 0;
  }
  if (2 * items > most) return 0;  // before any division
  const int split = min(most / items, steps / (LAST ? kSkinnyLastMinSteps : kSkinnyMinSteps));
  return split > 1 ? (steps + split - 1) / split : 0;
}

// Column blocks of a row tile that are cut into two halves, `items` = row tiles x n_cols blocks of the usual width.  Two items to a CU stream at
// one rate wherever they are, but a number of items that leaves some CUs with two and some with one (or, further up, a last round that is nearly
// empty) makes the call as long as the fuller ones.  As many blocks are then halved as give 512 workgroups, or a multiple, one item each, the
// whole ones first, so that with up to 256 of them no CU gets two.  A half begins at the k-step of its block (skinny_start): every element's sum
// is made in the same order as without the cut, whatever else the call holds.  Columns dealt evenly to the 512 were up to 3 % faster still, but
// a block's start, and with it the low bits of its elements, then followed the number of tiles.  Narrower blocks alone lose: fewer weight rows
// in flight per workgroup (7 slots of 4096 x 1536, 168 items of gemm1 or 511 of a third of the width, 55.9 / 65.2 us; 224 items of 7168 x 2048
// 112 / 126), so only where the last round is at most that full.
// FFN calls, usual blocks / halved: 9, 10, 11 slots of 7168 x 2048 (288, 320, 352 items of gemm1) 164 / 147, 178 / 165, 186 / 175; 11 to 14 of
// 4096 x 1536 (264 to 336) 97 / 84, 99 / 88, 100 / 93, 104 / 99; gemm2 of 9, 10, 11 slots of 4096 x 14336 (288, 320, 352) 586 / 552, 631 / 603,
// 686 / 663.  Up to 376 items none of 150 calls is slower, whatever its rows; 384 1.04 to 0.97 x, 400 level.  The halves of a second round load
// the activation rows once more: 17 slots of 7168 x 2048 (544 items) gain 1.05 x with 6 rows each, 1.035 with 20, 1.02 with 36 and lose 0.6 %
// with 60; 576 to 608 of five shapes 1.02 to 1.05 x with 6, up to 1.02 with 28, 0.96 to 0.99 with 48; 528 items 1.01 to 1.08 x with any; 640
// 0.954 to 1.006 x with few.
// gemm2 of fewer than 40 k-steps: 264 to 324 items 1.01 to 1.1 x; columns dealt evenly lost from 336 on (6 and 7 slots of 7168 x 2048 107 / 110
// and 112 / 117), and nothing is halved there.
constexpr int kSkinnySlots = 512;  // workgroups that run at once, two to a CU
// items up to which a single round (of more than 256) is filled: gemm1 and gemm2 from kSkinnyHalvesSteps k-steps on, gemm2 of fewer
constexpr int kSkinnyHalves = 376, kSkinnyHalvesShort = 328, kSkinnyHalvesSteps = 40;
// k-steps from which blocks are halved: 15 tiles of 832 x 1472 (345 items of 13 k-steps), columns dealt evenly, 28.7 / 30.8 us, 18 of 1088 x 1216
// (342 of 17) 34.6 / 30.0
constexpr int kSkinnyHalvesMinSteps = 15;
// gemm1: items of a last round that is filled, with any rows and with up to kSkinnyHalvesRows per tile; rounds at most.  Only where no slot has
// several tiles (one_each, looked at up to 128 slots): those read their weights together, and a second round of such calls, routed under Zipf laws,
// lost 2 % on average (10 calls, 0.93 to 1.01 x) where single tiles gain (11 calls 1.017 x); single rounds gain with either (1.02 to 1.1 x of 127).
constexpr int kSkinnyHalvesLast = 16, kSkinnyHalvesLastFew = 96, kSkinnyHalvesRows = 32, kSkinnyHalvesRounds = 2;
template <bool GEMM1>
__device__ __forceinline__ int skinny_halved(int n_tiles, bool one_each, int rows, int n_cols, int steps) {
  const int items = n_tiles * n_cols, rounds = (items + kSkinnySlots - 1) / kSkinnySlots, last = items - kSkinnySlots * (rounds - 1);
  if (steps < kSkinnyHalvesMinSteps) return 0;
  const bool fill = rounds == 1 ? last > kSkinnySlots / 2 && last <= (GEMM1 || steps >= kSkinnyHalvesSteps ? kSkinnyHalves : kSkinnyHalvesShort)
                                : GEMM1 && rounds <= kSkinnyHalvesRounds && one_each &&
                                      last <= (rows <= kSkinnyHalvesRows * n_tiles ? kSkinnyHalvesLastFew : kSkinnyHalvesLast);
  return fill ? max(kSkinnySlots * rounds / n_tiles - n_cols, 0) : 0;  // fewer than n_cols: more than half of the places have an item
}

// Few rows in every slot and few items that are not cut: at most 64 items leave three of four CUs without one, and an item of 192 or 128
// weight rows is then bound by what one CU can have in flight and by the three stages that it fills before its first product.  Such a
// GEMM takes items a quarter as wide, one to a CU: 32 weight rows (16 gate and 16 up, or 32 columns of y), the eight waves an eighth of K
// each, weights and activations loaded straight to the registers that the matrix instructions read (nothing is shared between the
// waves, so LDS would only be a detour), and the eight sums added through LDS at the end.  Measured, per call, before / after: one slot of
// 1536 x 1536 19.2 / 12.9 us, two of 2048 x 768 18.3 / 12.2, one of 2880 x 2880 25.2 / 19.5, four of 3072 x 1024 34.1 / 20.8, five of
// 1024 x 768 with 25 rows 14.5 / 11.2.  From 65 to 99 items some CUs have two narrow items and some one, and it is level or loses up to 1 us
// (90 of 23 k-steps 17.5 / 18.3); from 100 to 128 nearly all have two, and up to four rows, whose loads are few beside the weights',
// gain again (110 of 32 k-steps 31.6 / 28.9, 120 of 63 51.3 / 46.4; 16 rows: 112 of 29 48.3 / 52.1).  More lose at once (160 of 32 k-steps 36.8 /
// 37.6).  Batches of four k-steps: two batches in turn lose 10 to 25 % (most waves have two to eight steps, and loads past them cost issue).
constexpr int kFewRows = 16, kFewRowsItems = 64;
constexpr int kFewerRows = 4, kFewerRowsItems[2] = {100, 128}, kFewerRowsSteps = 16;
constexpr int kFewRowsCols1 = 16, kFewRowsCols2 = 32;  // h columns / y columns per item
// The test for them is in instances of their own, which the host launches where the tiles at capacity make up to 128 items and hold up to
// kFewRows rows on average: in a call that turns out to have more rows or items it costs 0.2 to 0.4 us (code in front of the main loop:
// nine slots of 1024 x 1024 16.5 / 16.9).
constexpr int kFewRowsLikely = 128;
constexpr int kFewRowsUnroll = 4;
constexpr uint32_t kPast = 0xffffff00u;  // past every descriptor: zeros without traffic

// sums[wave][fragment][lane]: what this wave's eighth of K gives of two fragments (16 weight rows each) x 16 activation rows
template <typename WeightOff>
__device__ __forceinline__ void few_rows_products(__amdgpu_buffer_rsrc_t rA, bool a_in, uint32_t a_off, __amdgpu_buffer_rsrc_t rW, const WeightOff& w_off,
                                                  int K, f32x4 (*sums)[2][kWave]) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int steps = K / 32, per = (steps + 7) / 8, s0 = wv * per, s1 = min(s0 + per, steps);
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  for (int s = s0; s < s1; s += kFewRowsUnroll) {
    u32x4 a[kFewRowsUnroll], w[kFewRowsUnroll][2];
#pragma unroll
    for (int u = 0; u < kFewRowsUnroll; ++u) {
      const uint32_t k = (s + u) * 64u;  // bytes
      const bool in = s + u < s1;        // the wave's part
      w[u][0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rW, in ? w_off(0) + k : kPast, 0, 0));
      w[u][1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rW, in ? w_off(1) + k : kPast, 0, 0));
      a[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rA, in && a_in ? a_off + k : kPast, 0, 0));
    }
    __builtin_amdgcn_sched_barrier(0);  // all loads of the batch before the first product waits
#pragma unroll
    for (int u = 0; u < kFewRowsUnroll; ++u) {
      acc[0] = mfma_16x16x32(w[u][0], a[u], acc[0]);
      acc[1] = mfma_16x16x32(w[u][1], a[u], acc[1]);
    }
  }
  sums[wv][0][lane] = acc[0];
  sums[wv][1][lane] = acc[1];
  __syncthreads();
}

__device__ __forceinline__ f32x4 few_rows_sum(const f32x4 (*sums)[2][kWave], int f, int lane) {
  f32x4 v = sums[0][f][lane];
#pragma unroll
  for (int q = 1; q < 8; ++q) v += sums[q][f][lane];
  return v;
}

template <bool GATHER>
__device__ __forceinline__ void few_rows_gemm1(const RowSource& src, const bf16_t* __restrict__ w13, int row0, int rows, int n0, int H, int F,
                                               bf16_t* __restrict__ hbuf, f32x4 (*sums)[2][kWave]) {
  const int lane = threadIdx.x & 63, r = lane & 15, kq = 16 * (lane >> 4);
  const __amdgpu_buffer_rsrc_t rA = GATHER ? make_rsrc(src.base, static_cast<size_t>(src.n_tokens) * H * 2)
                                           : make_rsrc(src.base + static_cast<size_t>(row0) * H, static_cast<size_t>(rows) * H * 2);
  const __amdgpu_buffer_rsrc_t rW = make_rsrc(w13, static_cast<size_t>(2) * F * H * 2);
  int row = r;
  if (GATHER && r < rows) row = min(max(src.row_pair[row0 + r], 0) / src.k, src.n_tokens - 1);
  const uint32_t w0 = (n0 + r) * (H * 2u) + kq, up = F * (H * 2u);
  few_rows_products(rA, r < rows, row * (H * 2u) + kq, rW, [&](int f) { return w0 + (f ? up : 0); }, H, sums);
  // lane l of a fragment holds weight rows 4 (l / 16) .. + 3 of activation row l % 16
  if (threadIdx.x < kWave && r < rows) {
    const f32x4 gate = few_rows_sum(sums, 0, lane), upv = few_rows_sum(sums, 1, lane);
    *reinterpret_cast<u32x2*>(hbuf + static_cast<size_t>(row0 + r) * F + n0 + 4 * (lane >> 4)) =
        u32x2{pack_bf16x2(swiglu(gate[0], upv[0]), swiglu(gate[1], upv[1])), pack_bf16x2(swiglu(gate[2], upv[2]), swiglu(gate[3], upv[3]))};
  }
}

__device__ __forceinline__ void few_rows_gemm2(const bf16_t* __restrict__ hbuf, const bf16_t* __restrict__ w2, int row0, int rows, int n0, int H,
                                               int F, bf16_t* __restrict__ y, f32x4 (*sums)[2][kWave]) {
  const int lane = threadIdx.x & 63, r = lane & 15, kq = 16 * (lane >> 4);
  const __amdgpu_buffer_rsrc_t rA = make_rsrc(hbuf + static_cast<size_t>(row0) * F, static_cast<size_t>(rows) * F * 2);
  const __amdgpu_buffer_rsrc_t rW = make_rsrc(w2, static_cast<size_t>(H) * F * 2);
  const uint32_t w0 = (n0 + r) * (F * 2u) + kq, next = 16 * (F * 2u);
  few_rows_products(rA, r < rows, r * (F * 2u) + kq, rW, [&](int f) { return w0 + (f ? next : 0); }, F, sums);
  if (threadIdx.x < 2 * kWave && r < rows) {
    const int f = threadIdx.x >> 6;
    const f32x4 v = few_rows_sum(sums, f, lane);
    *reinterpret_cast<u32x2*>(y + static_cast<size_t>(row0 + r) * H + n0 + 16 * f + 4 * (lane >> 4)) =
        u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
  }
}

// Item number -> (slot, first row, rows to the end of the slot, weight pointer, piece of K) without a tile table: slots
// in their own order, ceil(M / 64) tiles each.  Every workgroup finds its own tile with one scan over the
// (at most 1024) slots, two per thread, so the decode schedule needs no schedule kernel in front of it.
// Returns false if the item number is past the last item (the launch is sized for the capacity).
struct SkinnyTile {
  int row0, rows;
  int n0, n_end;  // columns
  bool few;       // few rows: an item of few_rows_gemm1 / 2
  int tile, col, piece, pieces, piece_steps;
  bool spread;  // the items begin at different k-steps (skinny_start)
  const void* w;
};

// Inclusive sum over the lanes of a wave: inside each row of sixteen, then from the rows before.
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // lane 15 of rows 0 and 2 to rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // lane 31 to rows 2 and 3
  return v;
}

// REDUCE: `item` is a tile number (columns and piece are not looked at).  GEMM1: which of the two, columns of `cols` in n_cols blocks.
// FEW: items of few rows are possible.
template <bool REDUCE, bool LAST, bool GEMM1 = false, bool FEW = false>
__device__ __forceinline__ bool skinny_locate(const int32_t* __restrict__ slot_offsets,
                                              const void* const* __restrict__ w_ptrs, int S, int item, int cols,
                                              int n_cols, int steps, bool may_split, int few_items, SkinnyTile& out) {
  const int all_rows = slot_offsets[S] - slot_offsets[0];
  __shared__ int32_t wave_tot[8];
  __shared__ int32_t found_row0, found_rows;
  __shared__ const void* found_w;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // Up to 128 slots every wave scans them for itself, two to a lane, without LDS and barriers: what the scan costs stands before an item's
  // first load, 1.9 us of both kernels each in the middle (time stamps), and 0.6 to 1 us of a call less this way (8 slots of 512 x 1024
  // 15.9 -> 15.2 us, two of 2880 x 2880 38.3 -> 37.3, 16 of 7168 x 2048 level).
  const bool alone = S <= 2 * kWave;
  const int at = alone ? lane : tid;
  if (!alone && tid == 0) found_rows = 0;
  int first[2], m[2], t[2];
  const void* w[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int sl = 2 * at + i;
    first[i] = m[i] = 0;
    w[i] = nullptr;
    if (sl < S) {
      first[i] = slot_offsets[sl];
      m[i] = max(slot_offsets[sl + 1] - first[i], 0);
      if (!REDUCE) w[i] = w_ptrs[sl];
    }
    t[i] = (m[i] + 63) >> 6;
  }
  const int local = t[0] + t[1];
  int incl = wave_scan(local);
  int excl = incl - local, n_tiles = 0;
  if (alone) {
    n_tiles = __builtin_amdgcn_readlane(incl, kWave - 1);
  } else {
    if (lane == kWave - 1) wave_tot[wv] = incl;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      excl += i < wv ? wave_tot[i] : 0;
      n_tiles += wave_tot[i];
    }
    n_tiles = __builtin_amdgcn_readfirstlane(n_tiles);
  }
  // These integer divisions follow one another before an item's first load.  A call that is not cut makes one of them and not
  // all six: 60 slots of 704 x 2816 (2640 items of 11 k-steps), gemm1 93.7 -> 89.0 us.
  int tile = item;
  out.piece_steps = steps;
  out.pieces = 1;
  out.col = out.piece = 0;
  const int piece_steps = may_split ? skinny_steps<LAST>(n_tiles * n_cols, all_rows, n_cols, steps) : 0;
  if (piece_steps) {
    out.piece_steps = piece_steps;
    out.pieces = (steps + piece_steps - 1) / piece_steps;
  }
  if (!REDUCE) {
    const int n_items = n_tiles * n_cols, most = max(m[0], m[1]);
    out.few = FEW && alone && 4 * n_items <= few_items && !piece_steps &&
              (n_items <= kFewRowsItems ? !__ballot(most > kFewRows)
                                        : n_items >= kFewerRowsItems[0] && n_items <= kFewerRowsItems[1] && steps >= kFewerRowsSteps &&
                                              !__ballot(most > kFewerRows));
    constexpr int kWidth = GEMM1 ? kSkinnyCols1 : kSkinnyCols2, kFewWidth = GEMM1 ? kFewRowsCols1 : kFewRowsCols2;
    const int halved = out.few || piece_steps ? 0 : skinny_halved<GEMM1>(n_tiles, alone && !__ballot(most > 64), all_rows, n_cols, steps);
    const int whole = out.few ? cols / kFewWidth : n_cols - halved, wholes = n_tiles * whole;
    if (!halved || item < wholes) {
      tile = item / whole;
      out.col = item - tile * whole;
      out.n0 = out.col * (out.few ? kFewWidth : kWidth);
      out.n_end = min(out.n0 + kWidth, cols);
    } else {  // the whole blocks of all tiles, then the halves
      tile = (item - wholes) / (2 * halved);
      const int half = item - wholes - 2 * halved * tile;
      out.col = whole + (half >> 1);
      const int width = min(kWidth, cols - out.col * kWidth) >> 1;  // a last block of gemm2 may have 64 columns
      out.n0 = out.col * kWidth + (half & 1) * width;
      out.n_end = out.n0 + width;
    }
    if (piece_steps) {
      const int q = tile;
      tile = q / out.pieces;
      out.piece = q - tile * out.pieces;
    }
  }
  out.tile = tile;
  // rows * K * 2 bytes * (share of the items that run at once) against 6 MB, one and a half of an XCD's L2; with fewer than 16
  // columns, dealt out to 8 XCDs, an XCD has no two items with the same rows
  out.spread = n_cols < 16 ||
               static_cast<long>(all_rows) * steps <= 96l * max(n_tiles * n_cols * out.pieces, 2 * kSkinnyItems);
  if (alone) {
    out.row0 = out.rows = 0;
    out.w = nullptr;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const unsigned long long hit = __ballot(tile >= excl && tile < excl + t[i]);  // one lane for one i when the tile exists
      if (hit) {
        const int src = __builtin_ctzll(hit), r = (tile - __builtin_amdgcn_readlane(excl, src)) * 64;
        out.row0 = __builtin_amdgcn_readlane(first[i], src) + r;
        out.rows = __builtin_amdgcn_readlane(m[i], src) - r;
        if (!REDUCE) {
          const uint64_t p = reinterpret_cast<uint64_t>(w[i]);
          const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(p), src), hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(p >> 32), src);
          out.w = reinterpret_cast<const void*>(static_cast<uint64_t>(hi) << 32 | lo);
        }
      }
      excl += t[i];
    }
    return out.rows > 0;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if (tile >= excl && tile < excl + t[i]) {  // true for exactly one (thread, i) when the tile exists
      const int r = (tile - excl) * 64;
      found_row0 = first[i] + r;
      found_rows = m[i] - r;
      found_w = w[i];
    }
    excl += t[i];
  }
  __syncthreads();
  out.row0 = __builtin_amdgcn_readfirstlane(found_row0);
  out.rows = __builtin_amdgcn_readfirstlane(found_rows);
  if (!REDUCE) out.w = found_w;
  return out.rows > 0;
}

// where piece p of a tile leaves its sums: [tile][piece][64][ld] floats
__device__ __forceinline__ float* skinny_partial(float* partial, const SkinnyTile& e, int piece, int ld) {
  return partial + static_cast<size_t>(e.tile * e.pieces + piece) * 64 * ld;
}

// The k-step at which an item begins; it goes round to the one before.  Items that all walk K from 0 ask at any moment for the
// same 128 bytes of rows that lie 2H (or 2F) bytes apart, which for H = 4096 is the same few HBM channels: spread over K,
// gemm1 of one token (4096 x 14336) takes 83 instead of 91 us, of 14 slots of 4096 x 1536 71 instead of 75, gemm2 of 20 slots
// of 7168 x 2048 123 instead of 130.  By column only: the row tiles of a slot read its weights together, from the caches
// (197 tokens, 64 slots of 7168 x 2048: 675 us, spread by tile too 687, all from 0 682).  Where the step count is a multiple of
// 11 few starts are left, but such rows are no power of two apart (11264 x 5632: 815 us, a stride of 13 822).
// But items that begin together also share the activation rows, and once those of the items that run at once are more than
// an XCD's L2 keeps that counts for more: 64 slots of 7168 x 2048, 45 rows in each, FFN 1040 us spread, 979 with gemm1 from 0;
// 30 rows 988 / 961; ten slots of 4096 x 14336, 60 rows in each 702, 683 with gemm2 from 0.  18 slots of 4096 x 1536, 30 rows in
// each (4.4 MB) 136 / 140; one slot, 2000 rows of 7168 x 512 (8 columns) 77 / 81.
// The tall tiles keep to k = 0: there the items of an XCD share weights and rows in its L2, and started block by block prefill
// of 8192 tokens was 3 % slower.
__device__ __forceinline__ int skinny_start(const SkinnyTile& e, int klen) {
  return e.spread ? (e.col * 11) % (klen / FBK) : 0;
}

// CLEAR: the arrival counters are cleared for gemm2's launch
template <bool GATHER, bool CLEAR, bool FEW>
__global__ __launch_bounds__(512, 4) void ffn_gemm1_skinny_kernel(RowSource src,
                                                                  const int32_t* __restrict__ slot_offsets,
                                                                  const void* const* __restrict__ w13_ptrs, int S,
                                                                  int H, int F, int may_split, int few_items,
                                                                  bf16_t* __restrict__ hbuf, float* partial,
                                                                  uint32_t* __restrict__ arrivals) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ u32x4 smem[];
  if (CLEAR && blockIdx.x == 0 && threadIdx.x < kArrivalWords) arrivals[threadIdx.x] = 0;
  SkinnyTile e;
  if (!skinny_locate<false, false, true, FEW>(slot_offsets, w13_ptrs, S, blockIdx.x, F, (F + kSkinnyCols1 - 1) / kSkinnyCols1, H / FBK,
                                               may_split, few_items, e))
    return;
  const bf16_t* w = static_cast<const bf16_t*>(e.w);
  if (FEW && e.few) {
    few_rows_gemm1<GATHER>(src, w, e.row0, e.rows, e.n0, H, F, hbuf, reinterpret_cast<f32x4(*)[2][kWave]>(smem));
    return;
  }
  if (e.pieces == 1) {
    gemm1_tile<1, GATHER, 1, 3>(src, w, e.row0, e.rows, e.n0, e.n_end, H, F, hbuf, smem, nullptr, nullptr, 0, 0,
                                nullptr, skinny_start(e, H));
  } else {
    const int k0 = e.piece * e.piece_steps * FBK;
    gemm1_tile<1, GATHER, 1, 3, false, true>(src, w, e.row0, e.rows, e.n0, e.n_end, H, F, hbuf, smem, nullptr,
                                             nullptr, k0, min(H - k0, e.piece_steps * FBK),
                                             skinny_partial(partial, e, e.piece, 2 * F),
                                             skinny_start(e, min(H - k0, e.piece_steps * FBK)));
  }
#endif
}

template <bool LAST, bool FEW>
__global__ __launch_bounds__(512, 4) void ffn_gemm2_skinny_kernel(const bf16_t* __restrict__ hbuf,
                                                                  const int32_t* __restrict__ slot_offsets,
                                                                  const void* const* __restrict__ w2_ptrs, int S,
                                                                  int H, int F, int may_split, int few_items,
                                                                  bf16_t* __restrict__ y, float* partial,
                                                                  uint32_t* arrivals) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ u32x4 smem[];
  SkinnyTile e;
  if (!skinny_locate<false, LAST, false, FEW>(slot_offsets, w2_ptrs, S, blockIdx.x, H, (H + kSkinnyCols2 - 1) / kSkinnyCols2, F / FBK,
                                       may_split, few_items, e))
    return;
  const bf16_t* w = static_cast<const bf16_t*>(e.w);
  if (FEW && e.few) {
    few_rows_gemm2(hbuf, w, e.row0, e.rows, e.n0, H, F, y, reinterpret_cast<f32x4(*)[2][kWave]>(smem));
    return;
  }
  if (e.pieces == 1) {
    gemm2_tile<1, 1, 3>(hbuf, w, e.row0, e.rows, e.n0, e.n_end, H, F, y, smem, nullptr, nullptr, 0, 0, nullptr,
                        skinny_start(e, F));
  } else {
    const int k0 = e.piece * e.piece_steps * FBK;
    const int n_cols = (H + kSkinnyCols2 - 1) / kSkinnyCols2, klen = min(F - k0, e.piece_steps * FBK);
    gemm2_tile<1, 1, 3, false, true, LAST>(hbuf, w, e.row0, e.rows, e.n0, e.n_end, H, F, y, smem, nullptr, nullptr, k0, klen,
                                     skinny_partial(partial, e, 0, H), skinny_start(e, klen), e.piece, e.pieces, arrivals,
                                     e.tile * n_cols + e.col);
  }
#endif
}

// The adding kernel: workgroup b adds the pieces of row b % 64 of tile b / 64, four columns per thread at a time.
// SWIGLU: partial rows are [gate F | up F] and the result is h; otherwise [H] and the result is y.
template <bool SWIGLU>
__global__ __launch_bounds__(512) void ffn_skinny_add_kernel(const float* __restrict__ partial,
                                                             const int32_t* __restrict__ slot_offsets, int S,
                                                             int n_cols, int steps, int out_cols,
                                                             bf16_t* __restrict__ out) {
  SkinnyTile e;
  const int row = blockIdx.x & 63;
  if (!skinny_locate<true, false>(slot_offsets, nullptr, S, blockIdx.x >> 6, out_cols, n_cols, steps, true, 0, e)) return;
  if (e.pieces == 1 || row >= e.rows) return;
  const int ld = SWIGLU ? 2 * out_cols : out_cols;
  const float* base = partial + static_cast<size_t>(e.tile * e.pieces) * 64 * ld + static_cast<size_t>(row) * ld;
  const size_t piece = static_cast<size_t>(64) * ld;
  for (int c = threadIdx.x * 4; c < out_cols; c += 512 * 4) {
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
    constexpr int BATCH = 8;  // pieces whose loads are in flight together
    for (int p0 = 0; p0 < e.pieces; p0 += BATCH) {
      f32x4 va[BATCH], vb[BATCH];
#pragma unroll
      for (int q = 0; q < BATCH; ++q) {
        const float* src = base + min(p0 + q, e.pieces - 1) * piece + c;
        va[q] = *reinterpret_cast<const f32x4*>(src);
        if constexpr (SWIGLU) vb[q] = *reinterpret_cast<const f32x4*>(src + out_cols);
      }
#pragma unroll
      for (int q = 0; q < BATCH; ++q)
        if (p0 + q < e.pieces) {
          a += va[q];
          if constexpr (SWIGLU) b += vb[q];
        }
    }
    if constexpr (SWIGLU) {
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] = swiglu(a[j], b[j]);
    }
    *reinterpret_cast<u32x2*>(out + static_cast<size_t>(e.row0 + row) * out_cols + c) =
        u32x2{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3])};
  }
}

struct FfnShape {
  bool skinny;  // the decode schedule
  int max_tiles, cut_tiles;  // tiles at most: with the standard cut, with any
  size_t h_bytes, table_bytes;
  size_t partial_bytes;  // room that cutting the contraction takes; not demanded: without it the call runs uncut
};

// The decode schedule is chosen on the host from the capacity of the row space alone (the row counts live
// on the device): at most 64 rows per slot (fewer where blocks are many) on average even if every pair were local, or so few items
// that 64-row tiles give gemm1 at most two to a CU (a shared expert's single slot).  gemm2 may then have many more and still
// gains, up to kSkinnyFewItems2.  One slot, tall tiles / this schedule: 454 rows of 7168 x 2048 176 / 84 us, 4000 of 7168 x 512
// 200 / 144, 15000 of 4096 x 128 145 / 122, 16000 of 32768 x 64 (64256 items of gemm2) 959 / 743, 32000 of it (128256) 1208 / 1501.
// Many slots of many column blocks have several items per CU with either schedule, and then a weight that two 64-row tiles of a slot stream
// twice costs more than the schedule kernel: from more than 1024 blocks on (S x F / 64) the line lies lower.  This schedule / tall tiles:
// 4096 x 14336, 10 slots (2240 blocks), 36 rows of capacity per slot 625 / 642 us, 40 732 / 658, 43 697 / 652, 59 799 / 703; 64 slots of
// 7168 x 2048 (2048) 32 643 / 650, 40 816 / 807, 50 743 / 708, 58 694 / 664 and 709 / 714; 36 slots (1152) 46 357 / 368, 50 428 / 434, 54 406 / 397,
// 62 436 / 413; but 18 slots of 2880 x 2880 (810) 52 133 / 133, 61 115 / 110, of 4096 x 1536 (432) 62 95 / 115.
// What the other path costs per item counts for more the shorter H is.  Calls between the lines with rows routed under Zipf laws, a hundredth to
// all of them local, tall tiles against this schedule, geometric mean: H below 768 0.99 x (31 calls, 0.81 to 1.18), to 1151 0.97 x (30, 0.63 to
// 1.33), to 1535 1.06 x (27), to 2240 1.15 x (69), above 1.14 x (145, 0.86 to 1.74).  Most are lost where few of the capacity's rows are local (39 of 64 slots of 7168 x 2048
// with 490 rows of 2880: 583 / 621 us), which the host cannot know.
constexpr int kSkinnyRowsPerSlot = 64;
constexpr int kSkinnyBlocks[2] = {1024, 1536}, kSkinnyRowsOfMore[2] = {52, 40};
constexpr int kSkinnyWide = 1152;  // H from which the line lies lower
static int skinny_rows_per_slot(int S, int H, int F) {
  if (H < kSkinnyWide) return kSkinnyRowsPerSlot;
  const long blocks = static_cast<long>(S) * ((F + kSkinnyCols1 - 1) / kSkinnyCols1);
  return blocks > kSkinnyBlocks[1] ? kSkinnyRowsOfMore[1] : blocks > kSkinnyBlocks[0] ? kSkinnyRowsOfMore[0] : kSkinnyRowsPerSlot;
}
constexpr int kSkinnyFewItems2 = 65536;
static_assert(kSkinnyFewItems2 * 512ll < (1ll << 32), "threads of one launch");

static FfnShape ffn_shape(int S, int H, int F, int max_rows) {
  FfnShape s;
  const bool short_slots = static_cast<long>(max_rows) <= static_cast<long>(skinny_rows_per_slot(S, H, F)) * S;
  const long tiles = static_cast<long>(max_rows) / 64 + S;
  s.skinny = short_slots || (tiles * ((F + kSkinnyCols1 - 1) / kSkinnyCols1) <= kSkinnyFewItems &&
                             tiles * ((H + kSkinnyCols2 - 1) / kSkinnyCols2) <= kSkinnyFewItems2);
  s.max_tiles = s.skinny ? max_rows / 64 + S : max_rows / 256 + S;
  s.cut_tiles = max_rows / 64 + S;
  const int table_tiles = short_slots ? max_rows / 64 + S : max_rows / 256 + S;
  s.h_bytes = align_up(static_cast<size_t>(max_rows > 0 ? max_rows : 1) * F * sizeof(bf16_t), 256);
  s.table_bytes = align_up(kTableHeaderInts * sizeof(int32_t) + static_cast<size_t>(table_tiles) * sizeof(TileEntry), 256);
  s.partial_bytes = s.skinny ? kSkinnyPartialBytes : 0;
  return s;
}

// What the workspace query returns: the most that any call of up to max_rows rows can use, so that a workspace sized for the
// largest batch serves every smaller one, at its full speed, and the query does not fall as max_rows grows.  h grows with
// the rows, and what may be cut at all may be at one row.  The tile table has room for every cut that the schedule kernel looks at: the
// standard one always, others up to kCutUnits tiles (six slots of 111 to 557 rows of 704 x 1024 take 16 tiles, 30.9 us; with room for 12
// tiles, which is what the standard cut and the decode schedule need, nine and 35.2).
static size_t ffn_query_bytes(int S, int H, int F, int max_rows) {
  const FfnShape s = ffn_shape(S, H, F, max_rows);
  const size_t table = kTableHeaderInts * sizeof(int32_t) + static_cast<size_t>(std::min(s.cut_tiles, kCutUnits)) * sizeof(TileEntry);
  size_t bytes = s.h_bytes + std::max(align_up(table, 256), s.table_bytes);
  if (max_rows > 0 && (skinny_may_split(S, 1, (F + kSkinnyCols1 - 1) / kSkinnyCols1, H / FBK) ||
                       skinny_last_adds(S, 1, (H + kSkinnyCols2 - 1) / kSkinnyCols2, F / FBK) ||
                       skinny_may_split(S, 1, (H + kSkinnyCols2 - 1) / kSkinnyCols2, F / FBK)))
    bytes += kSkinnyPartialBytes;
  return bytes;
}

// The GEMM kernels use 144 KB of dynamic LDS, which has to be opted into once per device.  *cus receives
// the device's CU count (the size of the persistent launch).
static int ffn_prepare(int* cus) {
  static std::mutex mu;
  static bool done[64] = {false};
  static int cu_count[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    set_error("probe_grouped_ffn: no current device");
    return PROBE_EHIP;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (done[dev]) {
    *cus = cu_count[dev];
    return PROBE_OK;
  }
  if (hipDeviceGetAttribute(&cu_count[dev], hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cu_count[dev] <= 0) {
    set_error("probe_grouped_ffn: cannot read the CU count of device %d", dev);
    return PROBE_EHIP;
  }
  *cus = cu_count[dev];
  hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(ffn_gemm1_kernel<false>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kFfnLdsBytes);
  if (err == hipSuccess)
    err = hipFuncSetAttribute(reinterpret_cast<const void*>(ffn_gemm1_kernel<true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, kFfnLdsBytes);
  if (err == hipSuccess)
    err = hipFuncSetAttribute(reinterpret_cast<const void*>(ffn_gemm2_kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, kFfnLdsBytes);
  const void* skinny[] = {reinterpret_cast<const void*>(ffn_gemm1_skinny_kernel<false, false, false>),
                          reinterpret_cast<const void*>(ffn_gemm1_skinny_kernel<false, false, true>),
                          reinterpret_cast<const void*>(ffn_gemm1_skinny_kernel<false, true, false>),
                          reinterpret_cast<const void*>(ffn_gemm1_skinny_kernel<false, true, true>),
                          reinterpret_cast<const void*>(ffn_gemm1_skinny_kernel<true, false, false>),
                          reinterpret_cast<const void*>(ffn_gemm1_skinny_kernel<true, false, true>),
                          reinterpret_cast<const void*>(ffn_gemm1_skinny_kernel<true, true, false>),
                          reinterpret_cast<const void*>(ffn_gemm1_skinny_kernel<true, true, true>),
                          reinterpret_cast<const void*>(ffn_gemm2_skinny_kernel<false, false>),
                          reinterpret_cast<const void*>(ffn_gemm2_skinny_kernel<false, true>),
                          reinterpret_cast<const void*>(ffn_gemm2_skinny_kernel<true, false>),
                          reinterpret_cast<const void*>(ffn_gemm2_skinny_kernel<true, true>)};
  for (const void* kernel : skinny)
    if (err == hipSuccess) err = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kSkinnyLdsBytes);
  if (err != hipSuccess) {
    set_error("probe_grouped_ffn: cannot reserve %d bytes of LDS: %s", kFfnLdsBytes, hipGetErrorString(err));
    return PROBE_EHIP;
  }
  done[dev] = true;
  return PROBE_OK;
}

}  // namespace probe

extern "C" size_t probe_grouped_ffn_workspace_bytes(int S, int H, int F, int max_rows) {
  if (S <= 0 || F <= 0 || max_rows < 0) return 0;
  return probe::ffn_query_bytes(S, H, F, max_rows);
}

namespace probe {

// Shared body of probe_grouped_ffn (row_pair == nullptr: activations from xp) and
// probe_grouped_ffn_gather (activations gathered from the token rows through row_pair).
static int ffn_impl(const char* name, const void* act_bf16, const int32_t* row_pair, int k, int T,
                    const int32_t* slot_offsets, const void* const* w13_ptrs, const void* const* w2_ptrs, int S,
                    int H, int F, int max_rows, void* y_bf16, void* workspace, size_t workspace_bytes,
                    void* stream) {
  PROBE_REQUIRE(S >= 1 && H > 0 && F > 0 && max_rows >= 0, PROBE_EINVAL,
                "%s: bad dims S=%d H=%d F=%d max_rows=%d", name, S, H, F, max_rows);
  PROBE_REQUIRE(S <= PROBE_MAX_SLOTS && H % 64 == 0 && F % 64 == 0, PROBE_EUNSUPPORTED,
                "%s: needs S <= %d, H %% 64 == 0, F %% 64 == 0 (S=%d H=%d F=%d)", name, PROBE_MAX_SLOTS, S, H, F);
  PROBE_REQUIRE(static_cast<size_t>(2) * F * H * 2 <= 0x7fffffffull, PROBE_EUNSUPPORTED,
                "%s: one expert's w13 must stay below 2 GiB (H=%d F=%d)", name, H, F);
  PROBE_REQUIRE(H <= (1 << 21) && F <= (1 << 21), PROBE_EUNSUPPORTED,
                "%s: H and F must not exceed 2^21 (32-bit byte offsets inside a row tile)", name);
  const bool gather = row_pair != nullptr;
  if (gather) {
    PROBE_REQUIRE(k >= 1 && k <= PROBE_MAX_TOPK && T >= 0, PROBE_EINVAL, "%s: bad k=%d or T=%d", name, k, T);
    PROBE_REQUIRE(static_cast<size_t>(T) * H * 2 <= 0x7fffffffull, PROBE_EUNSUPPORTED,
                  "%s: x must stay below 2 GiB (T=%d H=%d)", name, T, H);
  }
  if (max_rows == 0 || (gather && T == 0)) return PROBE_OK;
  PROBE_REQUIRE(act_bf16 && slot_offsets && w13_ptrs && w2_ptrs && y_bf16, PROBE_EINVAL, "%s: null pointer", name);
  PROBE_REQUIRE(aligned16(act_bf16) && aligned16(y_bf16), PROBE_EALIGN,
                "%s: activations and y must be 16-byte aligned", name);
  FfnShape sh = ffn_shape(S, H, F, max_rows);
  PROBE_REQUIRE(workspace && aligned16(workspace) && workspace_bytes >= sh.h_bytes + sh.table_bytes,
                PROBE_EWORKSPACE, "%s: workspace too small or misaligned (%zu < %zu)", name, workspace_bytes,
                sh.h_bytes + sh.table_bytes);
  PROBE_REQUIRE(static_cast<long>(sh.max_tiles + 8) * ((F + 127) / 128 + 4) < (1l << 30) &&
                    static_cast<long>(sh.max_tiles + 8) * ((H + 255) / 256 + 4) < (1l << 30),
                PROBE_EUNSUPPORTED, "%s: max_rows too large (%d)", name, max_rows);
  int cus = 0;
  int rc = ffn_prepare(&cus);
  if (rc != PROBE_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  bf16_t* hbuf = static_cast<bf16_t*>(workspace);
  int32_t* table = reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + sh.h_bytes);
  RowSource src;
  src.base = static_cast<const bf16_t*>(act_bf16);
  src.row_pair = row_pair;
  src.k = gather ? k : 1;
  src.n_tokens = gather ? T : 0;
  if (sh.skinny) {
    float* partial = reinterpret_cast<float*>(static_cast<char*>(workspace) + sh.h_bytes + sh.table_bytes);
    bf16_t* y = static_cast<bf16_t*>(y_bf16);
    const int tiles = skinny_max_tiles(S, max_rows);
    const int n1 = (F + kSkinnyCols1 - 1) / kSkinnyCols1, n2 = (H + kSkinnyCols2 - 1) / kSkinnyCols2;
    const bool room = workspace_bytes >= sh.h_bytes + sh.table_bytes + sh.partial_bytes;
    const bool split1 = room && skinny_may_split(S, max_rows, n1, H / FBK);
    const bool last_adds = room && skinny_last_adds(S, max_rows, n2, F / FBK);
    const bool split2 = last_adds || (room && skinny_may_split(S, max_rows, n2, F / FBK));
    uint32_t* arrivals = last_adds ? reinterpret_cast<uint32_t*>(table) : nullptr;
    // a split call has at most kSkinnyItems items, one that is not split tiles * n
    // and one whose blocks may be halved at most whole rounds of kSkinnySlots
    auto items = [](long n, bool split, int rounds, int steps) {
      if (split) n = std::max<long>(n, kSkinnyItems);
      return steps >= kSkinnyHalvesMinSteps && n > kSkinnySlots / 2 && n < kSkinnySlots * rounds ? (n + kSkinnySlots - 1) / kSkinnySlots * kSkinnySlots : n;
    };
    // Items of few rows are a quarter as wide; 0: none.  A grid for kFewRowsItems of them is enough unless 100 to 128 are likely.
    auto few_items = [S, max_rows](long n, int steps) {
      if (S > 2 * kWave || n > kFewRowsLikely || max_rows > static_cast<long>(kFewRows) * S) return 0l;
      return n >= kFewerRowsItems[0] && n <= kFewerRowsItems[1] && steps >= kFewerRowsSteps ? 4 * n : std::min<long>(4 * n, 4 * kFewRowsItems);
    };
    const long few1 = few_items(tiles * n1, H / FBK), few2 = few_items(tiles * n2, F / FBK);
    const dim3 g1(std::max(items(tiles * n1, split1, kSkinnyHalvesRounds, H / FBK), few1)), g2(std::max(items(tiles * n2, split2, 1, F / FBK), few2));
    // tiles that can be split at all: two pieces or more need kSkinnyItems / 2 items or fewer
    const int add1 = split1 ? std::min(tiles, kSkinnyItems / 2 / n1) : 0;
    const int add2 = split2 && !last_adds ? std::min(tiles, kSkinnyItems / 2 / n2) : 0;
    auto gemm1 = [&](auto gathers, auto clears, auto few) {
      hipLaunchKernelGGL((ffn_gemm1_skinny_kernel<gathers.value, clears.value, few.value>), g1, dim3(512), kSkinnyLdsBytes, st, src, slot_offsets,
                         w13_ptrs, S, H, F, split1, static_cast<int>(few1), hbuf, partial, arrivals);
    };
    auto gemm2 = [&](auto last, auto few) {
      hipLaunchKernelGGL((ffn_gemm2_skinny_kernel<last.value, few.value>), g2, dim3(512), kSkinnyLdsBytes, st, hbuf, slot_offsets, w2_ptrs, S, H, F,
                         split2, static_cast<int>(few2), y, partial, arrivals);
    };
    auto either = [](bool v, auto&& f) { v ? f(std::true_type()) : f(std::false_type()); };
    either(gather, [&](auto g) { either(last_adds, [&](auto c) { either(few1 > 0, [&](auto few) { gemm1(g, c, few); }); }); });
    if (add1 > 0)
      hipLaunchKernelGGL(ffn_skinny_add_kernel<true>, dim3(add1 * 64), dim3(512), 0, st, partial, slot_offsets, S, n1,
                         H / FBK, F, hbuf);
    // A call that is not cut takes the instance whose loads of the row total lie in front of the scan (two slots of 832 x 768 14.05 -> 13.9).
    either(last_adds || !split2, [&](auto l) { either(few2 > 0, [&](auto few) { gemm2(l, few); }); });
    if (add2 > 0)
      hipLaunchKernelGGL(ffn_skinny_add_kernel<false>, dim3(add2 * 64), dim3(512), 0, st, partial, slot_offsets, S, n2,
                         F / FBK, H, y);
    return check_launch(name);
  }
  const int n1 = (F + 127) / 128, n2 = (H + FBN - 1) / FBN;
  const dim3 grid(cus);  // persistent: one workgroup per CU, items drawn from the work queue
  // the room of the table decides how many tiles a cut may make: the standard one always fits, a workspace of the query's size holds any
  const size_t room = (workspace_bytes - sh.h_bytes - kTableHeaderInts * sizeof(int32_t)) / sizeof(TileEntry);
  const int max_tiles = static_cast<int>(std::min<size_t>(sh.cut_tiles, room));
  hipLaunchKernelGGL(ffn_schedule_kernel, dim3(1), dim3(kScheduleThreads), 0, st, slot_offsets, w13_ptrs, w2_ptrs, S,
                     max_tiles, n1, n2, H / FBK, F / FBK, cus, table);
  if (gather)
    hipLaunchKernelGGL(ffn_gemm1_kernel<true>, grid, dim3(512), kFfnLdsBytes, st, src, table, table, H, F, hbuf);
  else
    hipLaunchKernelGGL(ffn_gemm1_kernel<false>, grid, dim3(512), kFfnLdsBytes, st, src, table, table, H, F, hbuf);
  hipLaunchKernelGGL(ffn_gemm2_kernel, grid, dim3(512), kFfnLdsBytes, st, hbuf, table, table, H, F,
                     static_cast<bf16_t*>(y_bf16));
  return check_launch(name);
}

}  // namespace probe

extern "C" int probe_grouped_ffn(const void* xp_bf16, const int32_t* slot_offsets,
                                 const void* const* w13_ptrs, const void* const* w2_ptrs, int S,
                                 int H, int F, int max_rows, void* y_bf16, void* workspace,
                                 size_t workspace_bytes, void* stream) {
  return probe::ffn_impl("probe_grouped_ffn", xp_bf16, nullptr, 1, 0, slot_offsets, w13_ptrs, w2_ptrs, S, H, F,
                         max_rows, y_bf16, workspace, workspace_bytes, stream);
}

extern "C" int probe_grouped_ffn_gather(const void* x_bf16, const int32_t* row_pair, int T, int k,
                                        const int32_t* slot_offsets, const void* const* w13_ptrs,
                                        const void* const* w2_ptrs, int S, int H, int F, int max_rows,
                                        void* y_bf16, void* workspace, size_t workspace_bytes, void* stream) {
  PROBE_REQUIRE(row_pair != nullptr || max_rows == 0 || T == 0, PROBE_EINVAL,
                "probe_grouped_ffn_gather: row_pair is NULL");
  return probe::ffn_impl("probe_grouped_ffn_gather", x_bf16, row_pair, k, T, slot_offsets, w13_ptrs, w2_ptrs, S, H,
                         F, max_rows, y_bf16, workspace, workspace_bytes, stream);
}
