// probe_route_topk / probe_predict_topk: gate logits on the matrix cores, softmax, top-k.
//
// The gate is x[T,H] (bf16) times w_gate[E,H] (fp32).  At E = 128..256 this is far above the
// fp32 vector ridge of the chip, so the product runs on the bf16 MFMA units without giving up
// fp32 weights: every weight is split (once, by probe_pack_gate, or inside the call) into three bf16 planes hi + mid + lo
// (each the round-to-nearest bf16 of what the previous planes left over), which together
// carry all 24 significand bits.  x is bf16 already, every bf16 x bf16 product is exact in
// fp32, and the MFMA accumulates in fp32.
//
//   1. split    w_gate -> planes[3][E][H] bf16 in the workspace (skipped by the *_packed entry points,
//               which are handed planes made once by probe_pack_gate)
//   2. gemm     split-K tiled GEMM (128 or 256 tokens x 128 experts x 64 k per step; small batches and gates of at most 16
//               experts go straight from global memory to the matrix cores), three MFMAs per
//               operand pair (one per plane) into one accumulator  -> partial[KS][T][ld] fp32, ld = E
//               rounded up to 4;
//               its first workgroup clears the expert counts
//               H % 64 == 0: DMA-to-LDS software pipeline shared with the grouped FFN;
//               otherwise a register-staged kernel that zero-fills the K tail
//   3. softmax  sixteen lanes per token, or a wave where tokens are few: sum the KS partials in fixed order, add the bias,
//               softmax over E, k rounds of row arg-max (ties to the lower index), weights, counts
//
// The predictor's residual MLP (Eq. 7) adds W2_hat silu(W1_hat h) to the logits before step 3:
//   a. the same GEMM with one bf16 plane of W1_hat (D rows in place of experts) -> u partials
//   b. sum of the u partials, SiLU in fp32, split of s = silu(u) into three bf16 planes laid side
//      by side along K: A' = [s_hi | s_mid | s_lo], [T][3D]
//   c. W2_hat split into planes arranged as B' = {[hi hi hi], [mid mid 0], [lo 0 0]}, [3][E][3D],
//      so that step 2's three-plane GEMM over K = 3D forms the six largest of the nine plane
//      products (what is dropped is below 2^-24 of the result)
//   d. that GEMM; its split-K slices are written behind the gate's own, and step 3 sums them all
#include <limits.h>

#include <algorithm>
#include <mutex>

#include "common.hpp"
#include "mfma_pipeline.hpp"

namespace probe {

constexpr int GBM = 128, GBN = 128, GBK = 64;

// ---- 1. split -------------------------------------------------------------------------
// planes + plane_stride * p is plane p; `planes` already points at this gate's rows inside a plane
__global__ __launch_bounds__(256) void gate_split_kernel(const float* __restrict__ w, long n,
                                                         bf16_t* __restrict__ planes, long plane_stride,
                                                         int32_t* __restrict__ counts, int E) {
  long gid = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (counts && gid < E) counts[gid] = 0;
  if (gid >= n) return;
  float v = w[gid];
  bf16_t hi = f32_to_bf16(v);
  float r1 = v - bf16_to_f32(hi);  // exact
  bf16_t mid = f32_to_bf16(r1);
  float r2 = r1 - bf16_to_f32(mid);  // exact
  bf16_t lo = f32_to_bf16(r2);
  planes[gid] = hi;
  planes[plane_stride + gid] = mid;
  planes[2 * plane_stride + gid] = lo;
}

// The expert counts that the softmax / top-k kernel adds to are cleared by the first workgroup of
// the GEMM that precedes it on the stream (n <= 256 <= threads per workgroup).
__device__ __forceinline__ void zero_counts(int32_t* __restrict__ a, int32_t* __restrict__ b, int n) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && static_cast<int>(threadIdx.x) < n) {
    if (a) a[threadIdx.x] = 0;
    if (b) b[threadIdx.x] = 0;
  }
}

// ---- 2. gemm --------------------------------------------------------------------------
template <int PL>
__global__ __launch_bounds__(256, 2) void gate_gemm_kernel(const bf16_t* __restrict__ x,
                                                           const bf16_t* __restrict__ planes,
                                                           int T, int H, int E, int k_chunk,
                                                           float* __restrict__ partial, int ld,
                                                           int32_t* __restrict__ zero0, int32_t* __restrict__ zero1,
                                                           int n_zero) {
  __shared__ u32x4 sA[GBM * 8];
  __shared__ u32x4 sB[PL][GBN * 8];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wm = wv >> 1, wn = wv & 1;
  const int m0 = blockIdx.x * GBM, n0 = blockIdx.y * GBN, ks = blockIdx.z;
  zero_counts(zero0, zero1, n_zero);
  const int kbeg = ks * k_chunk, kend = min(H, kbeg + k_chunk);
  const long plane_elems = static_cast<long>(E) * H;

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  u32x4 ra[4], rb[PL][4];
  auto gload = [&](int k0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int idx = tid + 256 * j;
      int row = idx >> 3, c = idx & 7;
      int kk = k0 + c * 8;
      bool kin = kk < kend;
      int grow = m0 + row, brow = n0 + row;
      ra[j] = u32x4{0u, 0u, 0u, 0u};
      if (kin && grow < T) ra[j] = *reinterpret_cast<const u32x4*>(x + static_cast<long>(grow) * H + kk);
#pragma unroll
      for (int p = 0; p < PL; ++p) {
        rb[p][j] = u32x4{0u, 0u, 0u, 0u};
        if (kin && brow < E)
          rb[p][j] = *reinterpret_cast<const u32x4*>(planes + p * plane_elems + static_cast<long>(brow) * H + kk);
      }
    }
  };
  auto sstore = [&]() {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int idx = tid + 256 * j;
      int row = idx >> 3, c = idx & 7;
      sA[lds_chunk_off(row, c)] = ra[j];
#pragma unroll
      for (int p = 0; p < PL; ++p) sB[p][lds_chunk_off(row, c)] = rb[p][j];
    }
  };

  if (kbeg < kend) {
    gload(kbeg);
    sstore();
  }
  __syncthreads();
  for (int k0 = kbeg; k0 < kend; k0 += GBK) {
    const bool more = k0 + GBK < kend;
    if (more) gload(k0 + GBK);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int c = 2 * kk + (lane >> 5);
      u32x4 a[2];
#pragma unroll
      for (int mi = 0; mi < 2; ++mi) a[mi] = sA[lds_chunk_off(64 * wm + 32 * mi + (lane & 31), c)];
#pragma unroll
      for (int p = PL - 1; p >= 0; --p) {
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
          u32x4 b = sB[p][lds_chunk_off(64 * wn + 32 * ni + (lane & 31), c)];
#pragma unroll
          for (int mi = 0; mi < 2; ++mi) acc[mi][ni] = mfma_32x32x16(a[mi], b, acc[mi][ni]);
        }
      }
    }
    __syncthreads();
    if (more) {
      sstore();
      __syncthreads();
    }
  }
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
      int col = n0 + 64 * wn + 32 * ni + mfma32_col(lane);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        int row = m0 + 64 * wm + 32 * mi + mfma32_row(r, lane);
        if (row < T && col < ld) partial[(static_cast<long>(ks) * T + row) * ld + col] = acc[mi][ni][r];
      }
    }
}

// ---- 2b. gemm, DMA pipeline (H % 64 == 0) --------------------------------------------
// Same split-K tiling (128 tokens x 128 experts per workgroup), on the software pipeline of the
// grouped FFN: 8 waves (2 x 4, wave tile 64 tokens x 32 experts), buffer_load-to-LDS, two LDS
// stages of 64 KB = 128 token rows + 3 planes x 128 expert rows, three MFMAs (one per plane) per
// operand pair into one accumulator.  The weight fragment is the MFMA's row operand, so a lane
// ends with four consecutive experts of one token per register quad: 16-byte stores.
// MI = 2: 128 tokens per workgroup; MI = 4: 256 tokens (two stages of 80 KB, all of the LDS), which
// moves a third less operand data per MFMA and is used for large batches.
// One plane (u = W1_hat h of the residual): a k-step is a third of the matrix work for 48 KB of operands, so the loop waits for
// loads, and the 256-token tile takes three stages (144 KB): the predictor with residual, 8192 x 7168, 256 wide, 154 -> 152.7 us.
constexpr int kGateLdsBytes = 2 * (256 + 384) * 128;
constexpr int gate_stages(int mi, int planes) { return mi == 4 && planes == 1 ? 3 : 2; }
static_assert(3 * (256 + 128) * 128 <= kGateLdsBytes, "three stages of the one-plane tile");

// STEPWISE: the products of a k-step are summed by themselves and added to the accumulators (gemm_mainloop).
template <int MI, int PL, bool STEPWISE>
__global__ __launch_bounds__(512, 2) void gate_gemm_dma_kernel(const bf16_t* __restrict__ x,
                                                               const bf16_t* __restrict__ planes,
                                                               int T, int H, int E, int k_chunk,
                                                               float* __restrict__ partial, int ld,
                                                               int32_t* __restrict__ zero0,
                                                               int32_t* __restrict__ zero1, int n_zero) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ u32x4 smem[];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wv / 4, wn = wv % 4;
  const int m0 = blockIdx.x * (64 * MI), n0 = blockIdx.y * GBN, ks = blockIdx.z;
  zero_counts(zero0, zero1, n_zero);
  const int kbeg = ks * k_chunk, klen = min(H, kbeg + k_chunk) - kbeg;
  if (klen <= 0) return;
  const int rows = T - m0;
  __amdgpu_buffer_rsrc_t rA = make_rsrc(x + static_cast<size_t>(m0) * H, static_cast<size_t>(rows) * H * 2);
  __amdgpu_buffer_rsrc_t rB = make_rsrc(planes, static_cast<size_t>(PL) * E * H * 2);
  int voff[MI + 2 * PL];
  dma_offsets<MI>(wv, lane, H * 2, [&](int r) { return min(r, rows - 1); }, voff);
  // B-tile row j: plane j / 128, expert n0 + j % 128 (clamped; columns past E are masked at the store)
  dma_offsets<2 * PL>(wv, lane, H * 2, [&](int j) { return (j >> 7) * E + min(n0 + (j & 127), E - 1); }, voff + MI);
  f32x4 acc[2 * MI][2];
#pragma unroll
  for (int i = 0; i < 2 * MI; ++i) acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  gemm_mainloop<MI, 1, PL, gate_stages(MI, PL), false, false, false, STEPWISE>(rA, rB, voff, kbeg, klen, smem, wv, lane, acc);

#pragma unroll
  for (int i = 0; i < 2 * MI; ++i) {
    const int row = 32 * MI * wm + 16 * i + (lane & 15);
    if (row < rows) {
      float* dst = partial + (static_cast<long>(ks) * T + m0 + row) * ld;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int col = n0 + 32 * wn + 16 * j + 4 * (lane >> 4);
        if (col < ld) *reinterpret_cast<f32x4*>(dst + col) = acc[i][j];
      }
    }
  }
#endif
}

// ---- 2c. gemm straight from global memory to the matrix cores --------------------------------------
// Small batches, and gates of at most 16 experts at any batch.  There the product is a stream of the gate (3 planes
// of E x H: 0.2 MB for 8 x 4096, 11 MB for 256 x 7168) or of x, and what the tiled kernels above lose is latency: at 128
// tokens they are 16..32 workgroups that each pull 64 KB per k-step, four to seven steps one after another.  Here a wave
// multiplies one fragment of 16 experts (three planes) by NT fragments of 16 tokens over a few k32 of its own, with every
// operand loaded from global memory in the layout of v_mfma_f32_16x16x32_bf16 (16 rows x 64 bytes per instruction) and all
// loads of KU k32 in flight together; the eight waves of a workgroup split its K range and add their sums in LDS in
// fixed order.  No barrier before that; K is split until there is a workgroup per CU or 16 slices.  128 tokens: 10.4 -> 6 us
// at 128 x 4096, 14.4 -> 9 us at 256 x 7168; one token: 3.5 and 4.3 us.
// A lane's eight k lie inside or outside of H as a whole (H % 8 == 0), so any such H is served.
// SPLIT_W: `w` is the fp32 gate (the second of two stacked gates in w_next) and the planes are made in registers; every weight
// is read by ceil(T / (16 NT)) waves, so below two token blocks that is less work than a launch that writes the planes
// first.  The planes are bit for bit those of gate_split_kernel.
struct GateRows {
  const bf16_t* planes;  // [PL][N][H]
  const float* w;        // SPLIT_W: fp32 [n_first][H] and, stacked below it, w_next [N - n_first][H]
  const float* w_next;
  int n_first;
};

template <int PL, bool SPLIT_W>
__device__ __forceinline__ void gate_fragment(const GateRows& g, int row, int N, int H, int k, bool in,
                                              u32x4 (&a)[PL]) {
#pragma unroll
  for (int p = 0; p < PL; ++p) a[p] = u32x4{0u, 0u, 0u, 0u};
  if (!in) return;
  if constexpr (!SPLIT_W) {
#pragma unroll
    for (int p = 0; p < PL; ++p)
      a[p] = *reinterpret_cast<const u32x4*>(g.planes + (static_cast<long>(p) * N + row) * H + k);
  } else {
    static_assert(!SPLIT_W || PL == 3, "the fp32 gate is three planes");
    const float* src = row < g.n_first ? g.w + static_cast<long>(row) * H : g.w_next + static_cast<long>(row - g.n_first) * H;
    const float4 lo4 = *reinterpret_cast<const float4*>(src + k), hi4 = *reinterpret_cast<const float4*>(src + k + 4);
    const float v[8] = {lo4.x, lo4.y, lo4.z, lo4.w, hi4.x, hi4.y, hi4.z, hi4.w};
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
      float p1[2], p2[2], p3[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        p1[i] = bf16_to_f32(f32_to_bf16(v[j + i]));
        const float r1 = v[j + i] - p1[i];  // exact
        p2[i] = bf16_to_f32(f32_to_bf16(r1));
        p3[i] = r1 - p2[i];                 // exact
      }
      a[0][j / 2] = pack_bf16x2(p1[0], p1[1]);
      a[PL > 1 ? 1 : 0][j / 2] = pack_bf16x2(p2[0], p2[1]);
      a[PL > 2 ? 2 : 0][j / 2] = pack_bf16x2(p3[0], p3[1]);
    }
  }
}

// One wave's part: acc[i] += experts row0 .. +15 times tokens t0 + 16 i .. +15 over k32 numbers s0 .. s1 - 1.
template <int NT, int KU, int PL, bool SPLIT_W>
__device__ __forceinline__ void gate_direct_wave(const bf16_t* __restrict__ x, const GateRows& g, int T, int H, int N,
                                                 int n0, int t0, int s0, int s1, int lane, f32x4 (&acc)[NT]) {
  const int row = min(n0 + (lane & 15), N - 1);
  const bf16_t* xt[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) xt[i] = x + static_cast<long>(min(t0 + 16 * i + (lane & 15), T - 1)) * H;
  for (int s = s0; s < s1; s += KU) {
    u32x4 a[KU][PL], b[KU][NT];
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      const int k = (s + u) * 32 + 8 * (lane >> 4);
      const bool in = s + u < s1 && k < H;
      gate_fragment<PL, SPLIT_W>(g, row, N, H, k, in, a[u]);
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        b[u][i] = u32x4{0u, 0u, 0u, 0u};
        if (in) b[u][i] = *reinterpret_cast<const u32x4*>(xt[i] + k);
      }
    }
#pragma unroll
    for (int u = 0; u < KU; ++u)
#pragma unroll
      for (int p = 0; p < PL; ++p)
#pragma unroll
        for (int i = 0; i < NT; ++i) acc[i] = mfma_16x16x32(a[u][p], b[u][i], acc[i]);
  }
}

// position of the four experts 4c .. 4c+3 of a token in a [token][16] LDS tile, in floats: the sixteen tokens that a
// fragment stores at once cover all 64 banks
__device__ __forceinline__ int direct_pos(int token, int c) { return token * 16 + 4 * (c ^ ((token >> 2) & 3)); }

template <int NT, int KU, int PL, bool SPLIT_W>
__global__ __launch_bounds__(512) void gate_direct_kernel(const bf16_t* __restrict__ x, GateRows g, int T, int H, int N,
                                                          int k32_per_wave, float* __restrict__ partial, int ld,
                                                          int32_t* __restrict__ zero0, int32_t* __restrict__ zero1,
                                                          int n_zero) {
  __shared__ float sums[8][16 * NT * 16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const bool one_fragment = N <= 16;  // see launch_gate_direct
  const int t0 = (one_fragment ? blockIdx.x : blockIdx.z) * 16 * NT, n0 = one_fragment ? 0 : blockIdx.x * 16;
  const int ks = one_fragment ? blockIdx.z : blockIdx.y;
  zero_counts(zero0, zero1, n_zero);
  const int steps = (H + 31) / 32, s0 = (ks * 8 + wv) * k32_per_wave;
  f32x4 acc[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  gate_direct_wave<NT, KU, PL, SPLIT_W>(x, g, T, H, N, n0, t0, s0, min(s0 + k32_per_wave, steps), lane, acc);
#pragma unroll
  for (int i = 0; i < NT; ++i)
    *reinterpret_cast<f32x4*>(&sums[wv][direct_pos(16 * i + (lane & 15), lane >> 4)]) = acc[i];
  __syncthreads();
  for (int q = tid; q < 16 * NT * 4; q += 512) {
    const int token = q >> 2, c = q & 3, t = t0 + token, col = n0 + 4 * c;
    f32x4 v = *reinterpret_cast<const f32x4*>(&sums[0][direct_pos(token, c)]);
#pragma unroll
    for (int w = 1; w < 8; ++w) v += *reinterpret_cast<const f32x4*>(&sums[w][direct_pos(token, c)]);
    if (t < T && col < ld) *reinterpret_cast<f32x4*>(partial + (static_cast<long>(ks) * T + t) * ld + col) = v;
  }
}

static int gate_prepare() {
  static std::mutex mu;
  static bool done[64] = {false};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    set_error("probe_route_topk: no current device");
    return PROBE_EHIP;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (done[dev]) return PROBE_OK;
  hipError_t err = hipSuccess;
  const void* kernels[6] = {reinterpret_cast<const void*>(gate_gemm_dma_kernel<2, 3, true>),
                            reinterpret_cast<const void*>(gate_gemm_dma_kernel<4, 3, false>),
                            reinterpret_cast<const void*>(gate_gemm_dma_kernel<4, 3, true>),
                            reinterpret_cast<const void*>(gate_gemm_dma_kernel<2, 1, true>),
                            reinterpret_cast<const void*>(gate_gemm_dma_kernel<4, 1, false>),
                            reinterpret_cast<const void*>(gate_gemm_dma_kernel<4, 1, true>)};
  for (int i = 0; i < 6 && err == hipSuccess; ++i)
    err = hipFuncSetAttribute(kernels[i], hipFuncAttributeMaxDynamicSharedMemorySize, kGateLdsBytes);
  if (err != hipSuccess) {
    set_error("probe_route_topk: cannot reserve %d bytes of LDS: %s", kGateLdsBytes, hipGetErrorString(err));
    return PROBE_EHIP;
  }
  done[dev] = true;
  return PROBE_OK;
}

// ---- 3. softmax + top-k ---------------------------------------------------------------
// Sixteen lanes (one DPP row) own one token, a wave owns four.  Lane `sub` of a row holds the
// experts 64*i + 4*sub + j (i < NV, j < 4), i.e. 16-byte pieces of the logit row, so partial
// sums are read with float4 loads and every reduction stays inside a row: four rotate-and-
// combine DPP steps give all 16 lanes the same result bit for bit.
template <int N>
__device__ __forceinline__ float dpp_ror(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 | N, 0xf, 0xf, false));
}
template <int N>
__device__ __forceinline__ int dpp_ror(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x120 | N, 0xf, 0xf, false);
}
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, dpp_ror<8>(v));
  v = fmaxf(v, dpp_ror<4>(v));
  v = fmaxf(v, dpp_ror<2>(v));
  v = fmaxf(v, dpp_ror<1>(v));
  return v;
}
__device__ __forceinline__ float row_sum(float v) {
  v += dpp_ror<8>(v);
  v += dpp_ror<4>(v);
  v += dpp_ror<2>(v);
  v += dpp_ror<1>(v);
  return v;
}
// (row 0 + row 1) + (row 2 + row 3) of a wave, lane by lane, in every row.  A swap of a register with itself leaves one
// operand of the addition in each of its two results, the same pair in the same order in all lanes.
__device__ __forceinline__ float add_rows(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

__device__ __forceinline__ int row_min_i(int v) {
  v = min(v, dpp_ror<8>(v));
  v = min(v, dpp_ror<4>(v));
  v = min(v, dpp_ror<2>(v));
  v = min(v, dpp_ror<1>(v));
  return v;
}

// Pairwise (tree) reductions over a register array: depth log2(N) instead of a chain of N - 1
// dependent operations; max and min are exact, so the result does not depend on the order.
template <int N>
__device__ __forceinline__ float tree_max(const float (&v)[N]) {
  float t[N];
#pragma unroll
  for (int i = 0; i < N; ++i) t[i] = v[i];
#pragma unroll
  for (int st = 1; st < N; st *= 2)
#pragma unroll
    for (int i = 0; i + st < N; i += 2 * st) t[i] = fmaxf(t[i], t[i + st]);
  return t[0];
}
template <int N>
__device__ __forceinline__ int tree_min(const int (&v)[N]) {
  int t[N];
#pragma unroll
  for (int i = 0; i < N; ++i) t[i] = v[i];
#pragma unroll
  for (int st = 1; st < N; st *= 2)
#pragma unroll
    for (int i = 0; i + st < N; i += 2 * st) t[i] = min(t[i], t[i + st]);
  return t[0];
}

__device__ __forceinline__ bool aligned_f4(const float* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// Logit row pieces of U tokens: the KS split-K slices are added in ascending order, then the bias row
// of the token's group.  Lane `sub` receives the experts 64*i + 4*sub + j; entries past E hold anything (a whole piece of
// four is read up to the rounded end of a row), the callers mask them.
// What bounds it is the latency of the loads, so all of a round are issued before the first is waited for: no branch stands
// between them (a slice past the last is read again and counts as zero; with its addition under a condition the compiler
// moved the load there, one wait per slice) nor in front of the bias.  256 tokens x 1024 x 8 experts 5.83 -> 5.59 us, 128 x 4096 x
// 128 11.05 -> 10.6, 8192 x 4096 x 128 37.6 -> 36.8, 16384 x 1024 x 256 group-limited 62.1 -> 59.8.  The bias is loaded beside the sums
// with one token per row, behind them with two (first / last, 16384 tokens x 7168 x 256 144.0 / 140.5).
// SG = 4: the four rows of a wave own the same token, row r adds the slices r, r + 4, ... and the four sums are added across
// the rows, (0 + 1) + (2 + 3), so that all of them hold the same bits.
template <int NV, int U, int R, int SG>
__device__ __forceinline__ void load_logit_rows(const float* __restrict__ partial, int ld, int KS,
                                                const float* __restrict__ bias, int G, int tpg, int T, int E,
                                                bool vec, int sub, int grp, const int (&tt)[U], float (&l)[U][NV * 4]) {
  constexpr int NL = NV * 4;
  const int first = SG == 1 ? 0 : grp;
  constexpr bool BIAS_FIRST = U == 1;
  if (vec) {
    float4 accv[U][NV], bv[U][NV];
    auto load_bias = [&]() {  // no branch that differs between lanes: pieces past the end read the last ones
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < NV; ++i) bv[u][i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (!bias) return;
      const float* row[U];
#pragma unroll
      for (int u = 0; u < U; ++u) row[u] = bias + static_cast<long>(G > 1 ? min(tt[u] / tpg, G - 1) : 0) * E;
      if ((E & 3) == 0) {  // whole 16-byte pieces: the bias is aligned, checked by the host
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 0; i < NV; ++i) bv[u][i] = *reinterpret_cast<const float4*>(row[u] + min(64 * i + 4 * sub, E - 4));
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 0; i < NV; ++i) {
            const int e0 = 64 * i + 4 * sub;
            bv[u][i] = make_float4(row[u][min(e0, E - 1)], row[u][min(e0 + 1, E - 1)], row[u][min(e0 + 2, E - 1)],
                                   row[u][min(e0 + 3, E - 1)]);
          }
      }
    };
    if constexpr (BIAS_FIRST) load_bias();
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < NV; ++i) accv[u][i] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int q0 = 0; q0 < KS; q0 += R * SG) {
      // all loads of a round of R split-K slices (of every token of the row) are issued before any is consumed
      float4 tmp[R][U][NV];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int q = min(q0 + r * SG + first, KS - 1);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 0; i < NV; ++i) {
            const int e0 = min(64 * i + 4 * sub, ((E + 3) & ~3) - 4);
            tmp[r][u][i] = *reinterpret_cast<const float4*>(partial + (static_cast<long>(q) * T + tt[u]) * ld + e0);
          }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const bool in = q0 + r * SG + first < KS;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 0; i < NV; ++i) {
            accv[u][i].x += in ? tmp[r][u][i].x : 0.f; accv[u][i].y += in ? tmp[r][u][i].y : 0.f;
            accv[u][i].z += in ? tmp[r][u][i].z : 0.f; accv[u][i].w += in ? tmp[r][u][i].w : 0.f;
          }
      }
    }
    if constexpr (!BIAS_FIRST) load_bias();
    if constexpr (SG == 4) {
#pragma unroll
      for (int i = 0; i < NV; ++i)
        accv[0][i] = make_float4(add_rows(accv[0][i].x), add_rows(accv[0][i].y), add_rows(accv[0][i].z), add_rows(accv[0][i].w));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        l[u][4 * i] = accv[u][i].x + bv[u][i].x;
        l[u][4 * i + 1] = accv[u][i].y + bv[u][i].y;
        l[u][4 * i + 2] = accv[u][i].z + bv[u][i].z;
        l[u][4 * i + 3] = accv[u][i].w + bv[u][i].w;
      }
    }
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int g = 0;
      if (bias) g = min(tt[u] / tpg, G - 1);
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int e = 64 * (i >> 2) + 4 * sub + (i & 3);
        float sacc = 0.f;
        if (e < E) {
          for (int q = 0; q < KS; ++q) sacc += partial[(static_cast<long>(q) * T + tt[u]) * ld + e];
          if (bias) sacc += bias[static_cast<long>(g) * E + e];
        }
        l[u][i] = sacc;
      }
    }
  }
}

// What a gate's top-k reads and writes.  `partial` points at the gate's first column; a row of a partial plane has ld entries.
struct TopkGate {
  const float* partial;
  const float* bias;
  int G, tpg;
  int32_t* topk_idx;
  float* topk_w;
  float* probs;
  int32_t* counts;
};

// gates: one, or two stacked ones (router and predictor of the fused call), number blockIdx.y
// With U = 2 two tokens per row are in flight, so that the dependent DPP chains of one overlap the other's.  A chosen logit
// is overwritten with -inf; incoming logits are clamped to >= -FLT_MAX (NaN too), so -inf only ever means "taken".  The
// weight of a winner is recomputed from its logit with the same expression as its probability, so both agree bit for bit.
template <int NV, int U, int R, int SG>
__global__ __launch_bounds__(256) void gate_softmax_topk_kernel(TopkGate gate0, TopkGate gate1, int ld, int KS, int T,
                                                                int E, int k, int renorm) {
  static_assert(SG == 1 || (SG == 4 && U == 1), "sixteen lanes or a whole wave per token");
  const TopkGate& g = blockIdx.y ? gate1 : gate0;
  const float* __restrict__ partial = g.partial;
  const float* __restrict__ bias = g.bias;
  const int G = g.G, tpg = g.tpg;
  int32_t* __restrict__ topk_idx = g.topk_idx;
  float* __restrict__ topk_w = g.topk_w;
  float* __restrict__ probs = g.probs;
  int32_t* __restrict__ counts = g.counts;
  constexpr int NL = NV * 4;
  __shared__ int32_t hist[PROBE_MAX_EXPERTS];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int sub = lane & 15, grp = lane >> 4;
  hist[tid] = 0;
  __syncthreads();
  const float ninf = -__builtin_inff(), fmin_ = -3.402823466e38f;
  const bool vec = (E & 3) == 0;
  const bool vec_in = (ld & 3) == 0 && aligned_f4(partial);
  const int tokens_per_pass = gridDim.x * (SG == 1 ? 16 * U : 4);
  for (int t0 = SG == 1 ? ((blockIdx.x * 4 + wv) * U) * 4 + grp : blockIdx.x * 4 + wv; t0 < T; t0 += tokens_per_pass) {
    // token u of this row is t0 + 4u; the rows of a wave are independent under DPP row operations
    int tt[U];
    bool live[U];
    float l[U][NL];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      live[u] = t0 + 4 * u < T;
      tt[u] = live[u] ? t0 + 4 * u : t0;
    }
    load_logit_rows<NV, U, R, SG>(partial, ld, KS, bias, G, tpg, T, E, vec_in, sub, grp, tt, l);
    float mx[U], inv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // clamp (NaN and -inf become the most negative finite value); experts past E are "taken"
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int e = 64 * (i >> 2) + 4 * sub + (i & 3);
        float v = l[u][i];
        v = (v >= fmin_) ? v : fmin_;
        l[u][i] = (e < E) ? v : ninf;
      }
      mx[u] = row_max(tree_max(l[u]));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float p[NL], sum = 0.f;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        p[i] = expf(l[u][i] - mx[u]);  // exp(-inf) = 0 for the experts past E
        sum += p[i];
      }
      sum = row_sum(sum);
      inv[u] = 1.f / sum;
      if (probs && live[u] && (SG == 1 || grp == 0)) {
        const long t = t0 + 4 * u;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          const int e0 = 64 * i + 4 * sub;
          if (vec) {
            if (e0 < E)
              *reinterpret_cast<float4*>(probs + t * E + e0) =
                  make_float4(p[4 * i] * inv[u], p[4 * i + 1] * inv[u], p[4 * i + 2] * inv[u], p[4 * i + 3] * inv[u]);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (e0 + j < E) probs[t * E + e0 + j] = p[4 * i + j] * inv[u];
          }
        }
      }
    }
    int isel[U];
    float wsel[U], wtot[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      isel[u] = 0;
      wsel[u] = 0.f;
      wtot[u] = 0.f;
    }
    for (int s = 0; s < k; ++s) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float best = row_max(tree_max(l[u]));
        // lowest expert id among the entries that hold the row maximum
        int cand[NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          const int e = 64 * (i >> 2) + 4 * sub + (i & 3);
          cand[i] = (l[u][i] == best) ? e : INT_MAX;
        }
        const int be = row_min_i(tree_min(cand));
        // its owner marks it taken
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          const int e = 64 * (i >> 2) + 4 * sub + (i & 3);
          l[u][i] = (e == be) ? ninf : l[u][i];
        }
        const float pw = expf(best - mx[u]) * inv[u];
        wtot[u] += pw;
        if (sub == s) {
          isel[u] = be;
          wsel[u] = pw;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (renorm) wsel[u] /= wtot[u];
      if (live[u] && sub < k && (SG == 1 || grp == 0)) {
        const long t = t0 + 4 * u;
        topk_idx[t * k + sub] = isel[u];
        topk_w[t * k + sub] = wsel[u];
        if (counts) atomicAdd(&hist[isel[u]], 1);
      }
    }
  }
  __syncthreads();
  if (counts && tid < E && hist[tid] != 0) atomicAdd(&counts[tid], hist[tid]);
}

// (m1, m2) = the two largest of this lane's pair and the pair N lanes away in the row
template <int N>
__device__ __forceinline__ void top2_merge(float& m1, float& m2) {
  const float o1 = dpp_ror<N>(m1), o2 = dpp_ror<N>(m2);
  m2 = fmaxf(fminf(m1, o1), fmaxf(m2, o2));
  m1 = fmaxf(m1, o1);
}

template <int CTRL>
__device__ __forceinline__ void top2_merge_dpp(float& m1, float& m2) {
  const float o1 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m1), CTRL, 0xf, 0xf, false));
  const float o2 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m2), CTRL, 0xf, 0xf, false));
  m2 = fmaxf(fminf(m1, o1), fmaxf(m2, o2));
  m1 = fmaxf(m1, o1);
}
// The same over the lanes that share a group, `lanes` = 1, 2, 4, 8 or 16 consecutive ones of a row: neighbours, pairs, then the mirror
// images of eight and sixteen lanes, each of which lies in the other half.
__device__ __forceinline__ void top2_merge_group(float& m1, float& m2, int lanes) {
  if (lanes >= 2) top2_merge_dpp<0xb1>(m1, m2);    // quad_perm 1 0 3 2
  if (lanes >= 4) top2_merge_dpp<0x4e>(m1, m2);    // quad_perm 2 3 0 1
  if (lanes >= 8) top2_merge_dpp<0x141>(m1, m2);   // row_half_mirror
  if (lanes >= 16) top2_merge_dpp<0x140>(m1, m2);  // row_mirror
}

// ---- 3b. group-limited gate -----------------------------------------------------------------
// Same lane layout and logit loading as above.  Per token: scores s (sigmoid of each logit, or the
// softmax), selection scores c = s + select_bias, a score per group of E / n_group consecutive
// experts (sum of its group_top largest c), the topk_group best groups, the k largest c among their
// experts, gating values from s.  Every decision is an arg-max over a DPP row with ties to the
// lower index, so all sixteen lanes of a token agree bit for bit.  Lane j keeps the score of group
// j (n_group <= 16); sets of groups and of consumed entries are bit masks.
template <int NV, int U, int R, int SG>
__global__ __launch_bounds__(256) void gate_grouped_topk_kernel(
    const float* __restrict__ partial, int ld, int KS, const float* __restrict__ bias, int G, int tpg,
    const float* __restrict__ select_bias, int T, int E, int k, int scoring, int n_group, int topk_group,
    int group_top, int renorm, float routed_scale, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
    float* __restrict__ scores, int32_t* __restrict__ counts) {
  constexpr int NL = NV * 4;
  __shared__ int32_t hist[PROBE_MAX_EXPERTS];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int sub = lane & 15, grp = lane >> 4;
  hist[tid] = 0;
  __syncthreads();
  const float ninf = -__builtin_inff(), fmin_ = -3.402823466e38f;
  const bool vec = (E & 3) == 0;
  const bool vec_in = (ld & 3) == 0 && aligned_f4(partial);
  const int gs = E / n_group;
  const bool aligned_groups = group_top <= 2 && gs >= 4 && gs <= 64 && (gs & (gs - 1)) == 0;
  int gid[NL];      // group of entry i, -1 past E
  float sb[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int e = 64 * (i >> 2) + 4 * sub + (i & 3);
    gid[i] = e < E ? e / gs : -1;
    sb[i] = (select_bias && e < E) ? select_bias[e] : 0.f;
  }
  const int tokens_per_pass = gridDim.x * (SG == 1 ? 16 * U : 4);
  for (int t0 = SG == 1 ? ((blockIdx.x * 4 + wv) * U) * 4 + grp : blockIdx.x * 4 + wv; t0 < T; t0 += tokens_per_pass) {
    int tt[U];
    bool live[U];
    float sc[U][NL], c[U][NL];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      live[u] = t0 + 4 * u < T;
      tt[u] = live[u] ? t0 + 4 * u : t0;
    }
    load_logit_rows<NV, U, R, SG>(partial, ld, KS, bias, G, tpg, T, E, vec_in, sub, grp, tt, sc);
    // scores (in place of the logits) and selection scores
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        float v = sc[u][i];
        v = (v >= fmin_) ? v : fmin_;  // NaN and -inf become the most negative finite value
        sc[u][i] = (gid[i] >= 0) ? v : ninf;
      }
      if (scoring == 1) {
#pragma unroll
        for (int i = 0; i < NL; ++i) sc[u][i] = 1.f / (1.f + expf(-sc[u][i]));  // 0 past E
      } else {
        const float m = row_max(tree_max(sc[u]));
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          sc[u][i] = expf(sc[u][i] - m);
          sum += sc[u][i];
        }
        const float inv = 1.f / row_sum(sum);
#pragma unroll
        for (int i = 0; i < NL; ++i) sc[u][i] *= inv;
      }
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        float v = sc[u][i] + sb[i];
        v = (v >= fmin_) ? v : fmin_;
        c[u][i] = (gid[i] >= 0) ? v : ninf;
      }
      if (scores && live[u] && (SG == 1 || grp == 0)) {
        const long t = t0 + 4 * u;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          const int e0 = 64 * i + 4 * sub;
          if (vec) {
            if (e0 < E)
              *reinterpret_cast<float4*>(scores + t * E + e0) =
                  make_float4(sc[u][4 * i], sc[u][4 * i + 1], sc[u][4 * i + 2], sc[u][4 * i + 3]);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (e0 + j < E) scores[t * E + e0 + j] = sc[u][4 * i + j];
          }
        }
      }
    }
    // group scores.  Only the VALUES of a group's largest selection scores matter, so for
    // group_top <= 2 a (largest, second) pair is merged across the row with max / min, which is
    // exact and order-free; otherwise group_top rounds of arg-max inside the group.
    float gscore[U];
    unsigned allowed[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      gscore[u] = ninf;
      allowed[u] = 0u;
    }
    if (aligned_groups) {
      // Every group is 1, 2, 4, 8 or 16 lanes of one register piece: all of a piece's groups are merged at once, with the same bits as
      // group by group, where each pass looked at every entry (call, group by group / at once, 8 groups: 75 tokens x 7168 x 256 19.5 /
      // 18.5 us, 128 x 4096 x 128 14.2 / 13.4, 16384 x 1024 x 64 27.5 / 25.9).
      float piece[U][NV];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          float m1 = c[u][4 * i], m2 = ninf;
#pragma unroll
          for (int j = 1; j < 4; ++j) {
            m2 = fmaxf(m2, fminf(m1, c[u][4 * i + j]));
            m1 = fmaxf(m1, c[u][4 * i + j]);
          }
          top2_merge_group(m1, m2, gs >> 2);
          piece[u][i] = group_top == 2 ? m1 + m2 : m1;
        }
      for (int r = 0; r < topk_group; ++r) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          float open[NV];
          int cand[NV];
#pragma unroll
          for (int i = 0; i < NV; ++i) open[i] = gid[4 * i] >= 0 && !((allowed[u] >> gid[4 * i]) & 1u) ? piece[u][i] : ninf;
          const float best = row_max(tree_max(open));
#pragma unroll
          for (int i = 0; i < NV; ++i)
            cand[i] = gid[4 * i] >= 0 && !((allowed[u] >> gid[4 * i]) & 1u) && piece[u][i] == best ? gid[4 * i] : INT_MAX;
          allowed[u] |= 1u << (row_min_i(tree_min(cand)) & 15);
        }
      }
    } else if (group_top <= 2) {
      for (int j = 0; j < n_group; ++j) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          float m1 = ninf, m2 = ninf;
#pragma unroll
          for (int i = 0; i < NL; ++i) {
            const float v = (gid[i] == j) ? c[u][i] : ninf;
            m2 = fmaxf(m2, fminf(m1, v));
            m1 = fmaxf(m1, v);
          }
          top2_merge<8>(m1, m2);
          top2_merge<4>(m1, m2);
          top2_merge<2>(m1, m2);
          top2_merge<1>(m1, m2);
          const float sum = (group_top == 2) ? m1 + m2 : m1;
          gscore[u] = (sub == j) ? sum : gscore[u];
        }
      }
    } else {
      unsigned used[U];
#pragma unroll
      for (int u = 0; u < U; ++u) used[u] = 0u;
      for (int j = 0; j < n_group; ++j) {
        float sum[U];
#pragma unroll
        for (int u = 0; u < U; ++u) sum[u] = 0.f;
        for (int r = 0; r < group_top; ++r) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            float m = ninf;
#pragma unroll
            for (int i = 0; i < NL; ++i) {
              const bool open = gid[i] == j && !((used[u] >> i) & 1u);
              m = open ? fmaxf(m, c[u][i]) : m;
            }
            const float best = row_max(m);
            int cand = INT_MAX;
#pragma unroll
            for (int i = NL - 1; i >= 0; --i) {
              const int e = 64 * (i >> 2) + 4 * sub + (i & 3);
              const bool open = gid[i] == j && !((used[u] >> i) & 1u);
              cand = (open && c[u][i] == best) ? e : cand;
            }
            const int be = row_min_i(cand);
#pragma unroll
            for (int i = 0; i < NL; ++i) {
              const int e = 64 * (i >> 2) + 4 * sub + (i & 3);
              used[u] |= (e == be) ? (1u << i) : 0u;
            }
            sum[u] += best;
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) gscore[u] = (sub == j) ? sum[u] : gscore[u];
      }
    }
    // allowed groups
    for (int r = 0; r < topk_group && !aligned_groups; ++r) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool open = sub < n_group && !((allowed[u] >> sub) & 1u);
        const float best = row_max(open ? gscore[u] : ninf);
        const int bg = row_min_i((open && gscore[u] == best) ? sub : INT_MAX);
        allowed[u] |= 1u << (bg & 15);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const bool ok = gid[i] >= 0 && ((allowed[u] >> (gid[i] & 15)) & 1u);
        c[u][i] = ok ? c[u][i] : ninf;
      }
    // k largest selection scores among the allowed experts; -inf now means "not available"
    int isel[U];
    float wsel[U], wtot[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      isel[u] = 0;
      wsel[u] = 0.f;
      wtot[u] = 0.f;
    }
    for (int s = 0; s < k; ++s) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float best = row_max(tree_max(c[u]));
        int cand[NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          const int e = 64 * (i >> 2) + 4 * sub + (i & 3);
          cand[i] = (c[u][i] == best) ? e : INT_MAX;
        }
        const int be = row_min_i(tree_min(cand));
        float mine = ninf;  // the owner's score of the winner, without the selection bias
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          const int e = 64 * (i >> 2) + 4 * sub + (i & 3);
          mine = (e == be) ? sc[u][i] : mine;
          c[u][i] = (e == be) ? ninf : c[u][i];
        }
        const float pw = row_max(mine);
        wtot[u] += pw;
        if (sub == s) {
          isel[u] = be;
          wsel[u] = pw;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (renorm) wsel[u] /= wtot[u];
      wsel[u] *= routed_scale;
      if (live[u] && sub < k && (SG == 1 || grp == 0)) {
        const long t = t0 + 4 * u;
        topk_idx[t * k + sub] = isel[u];
        topk_w[t * k + sub] = wsel[u];
        if (counts) atomicAdd(&hist[isel[u]], 1);
      }
    }
  }
  __syncthreads();
  if (counts && tid < E && hist[tid] != 0) atomicAdd(&counts[tid], hist[tid]);
}

// ---- 4. residual of the predictor (Eq. 7) ------------------------------------------------
// r[t,e] = sum_d w2_hat[e,d] * s[t,d],  s = silu(u),  u = W1_hat h summed over its split-K partials.
// Both factors are fp32; the product runs on the matrix cores at fp32 accuracy by splitting each
// factor into bf16 planes (hi + mid + lo, as for the gate) and keeping the six largest of the nine
// plane products: with the planes of s laid side by side along K,
//     A'[t]   = [ s_hi | s_mid | s_lo ]                         (bf16 [T, 3D])
//     B'_0[e] = [ w_hi | w_hi  | w_hi ],  B'_1[e] = [ w_mid | w_mid | 0 ],  B'_2[e] = [ w_lo | 0 | 0 ]
// the three-plane GEMM of the gate computes  s_hi (w_hi + w_mid + w_lo) + s_mid (w_hi + w_mid) + s_lo w_hi;
// the dropped products are below 2^-24 of the result.  Its split-K slices are written behind the
// gate's own, so the softmax / top-k kernel adds the residual like further slices of the logits.
//
// One launch makes both operands (A' by the first workgroups, B' by the last ones): they do not depend on each other, and
// either alone is as long as a launch.  A thread takes 8 consecutive hidden units of one row, 16 bytes per plane.
// 8192 tokens, 256 experts, D = 256: the whole predictor 152.7 -> 150.9 us against two launches.
struct Planes8 {
  u32x4 hi, mid, lo;
};
__device__ __forceinline__ Planes8 split_planes8(const float (&v)[8]) {
  uint32_t pk[3][4];
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    float p1[2], p2[2], p3[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      p1[i] = bf16_to_f32(f32_to_bf16(v[j + i]));
      const float r1 = v[j + i] - p1[i];      // exact
      p2[i] = bf16_to_f32(f32_to_bf16(r1));
      p3[i] = r1 - p2[i];                     // exact; rounded to bf16 by the pack below
    }
    pk[0][j / 2] = pack_bf16x2(p1[0], p1[1]);
    pk[1][j / 2] = pack_bf16x2(p2[0], p2[1]);
    pk[2][j / 2] = pack_bf16x2(p3[0], p3[1]);
  }
  return Planes8{{pk[0][0], pk[0][1], pk[0][2], pk[0][3]},
                 {pk[1][0], pk[1][1], pk[1][2], pk[1][3]},
                 {pk[2][0], pk[2][1], pk[2][2], pk[2][3]}};
}

static unsigned resid_split_blocks(int rows, int D) {
  return static_cast<unsigned>((static_cast<long>(rows) * (D / 8) + 255) / 256);
}

// a_blocks = resid_split_blocks(T, D) workgroups for A', resid_split_blocks(E, D) for B'
__global__ __launch_bounds__(256) void resid_split_kernel(const float* __restrict__ upartial, int KS2, int T,
                                                          const float* __restrict__ w2_hat, int E, int D,
                                                          unsigned a_blocks, bf16_t* __restrict__ a_planes,
                                                          bf16_t* __restrict__ b_planes) {
  const int groups = D / 8;
  const bool is_a = blockIdx.x < a_blocks;
  const long gid = static_cast<long>(is_a ? blockIdx.x : blockIdx.x - a_blocks) * blockDim.x + threadIdx.x;
  if (gid >= static_cast<long>(is_a ? T : E) * groups) return;
  const int r = static_cast<int>(gid / groups), d0 = static_cast<int>(gid % groups) * 8;
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = 0.f;
  const int slices = is_a ? KS2 : 1, rows = is_a ? T : E;
  const float* base = is_a ? upartial : w2_hat;
  for (int q = 0; q < slices; ++q) {
    const float4* src = reinterpret_cast<const float4*>(base + (static_cast<long>(q) * rows + r) * D + d0);
    const float4 lo = src[0], hi = src[1];
    v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
    v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
  }
  if (is_a) {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = v[j] / (1.f + expf(-v[j]));
  }
  const Planes8 p = split_planes8(v);
  auto put = [&](bf16_t* dst, u32x4 val) { *reinterpret_cast<u32x4*>(dst) = val; };
  if (is_a) {
    bf16_t* row = a_planes + static_cast<long>(r) * 3 * D + d0;
    put(row, p.hi);
    put(row + D, p.mid);
    put(row + 2 * D, p.lo);
  } else {
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const long plane = static_cast<long>(E) * 3 * D;
    bf16_t* row = b_planes + static_cast<long>(r) * 3 * D + d0;
    put(row, p.hi);              put(row + D, p.hi);              put(row + 2 * D, p.hi);
    put(row + plane, p.mid);     put(row + plane + D, p.mid);     put(row + plane + 2 * D, zero);
    put(row + 2 * plane, p.lo);  put(row + 2 * plane + D, zero);  put(row + 2 * plane + 2 * D, zero);
  }
}

struct RouteShape {
  bool dma;  // H % 64 == 0: the DMA-to-LDS pipeline; otherwise the register-staged kernel
  int bm;    // tokens per workgroup of the gemm (128 or 256)
  int mt, nt, ks, k_chunk;
  bool stepwise;    // DMA pipeline: sums by k-step
  int ks_room;      // slices that the workspace has room for: those of the tiled kernels, which the direct one never exceeds
  int ld;           // entries of a row of partial sums: E rounded up to whole 16-byte pieces (the last ones are read as part
                    // of a piece and not looked at)
  bool direct;      // gate_direct_kernel: `frags` fragments of 16 tokens per workgroup, `per_wave` k32 per wave
  int frags, per_wave;
  size_t planes_bytes, partial_bytes;
};

// Logits (T x E) up to which a gate takes the direct kernel, and gates that take it at any batch (16 experts are one
// fragment: a 128-expert tile would be mostly padding; figures at small_gate_frags).  Whole call, direct against tiled:
// 256 tokens x 128 experts 12.4 / 15.7 us (H = 4096; what is faster above the line is at direct_of_more).  Where H is not a multiple of 64 the
// other kernel is the register-staged one and the line lies higher: 1000 tokens x 250 experts x 7160 47.6 us, 1500 tokens staged 50.6.
// A launch holds fewer than 2^32 threads: 512 for 32 tokens here, a quarter of that in the tiled kernels, which therefore take
// the batches above kDirectTokens.
constexpr int kDirectLogits = 32768, kDirectExperts = 16, kDirectTokens = 1 << 27;

constexpr int kMaxSplitK = 16;
constexpr int kResidSplitK = 4;  // second layer of the residual: the softmax kernel reads every slice

// k-steps per slice of the tiled kernels, `want` slices wished for
static int gate_slice_steps(int ksteps, int want, int max_split) {
  if (want > max_split) want = max_split;  // the softmax kernel adds the slices one after another
  if (want > ksteps) want = ksteps;
  if (want < 1) want = 1;
  return (ksteps + want - 1) / want;
}
// Room for slices: 256-token tiles when a split of 8 or less still gives every CU a workgroup, split for one workgroup per
// CU, otherwise 128-token tiles, split for two.  The register-staged kernel runs as many; the others choose up to that.
constexpr int kBigTileItems = 32;
static bool gate_dma(int H, int E) { return H % 64 == 0 && static_cast<size_t>(3) * E * H * 2 <= 0x7fffffffull; }
static int gate_target(int bm) { return bm == 256 ? 256 : 512; }

// Fragments of 16 tokens per workgroup for a gate of at most 16 experts at any batch.  Such a product is a stream of x, and
// small batches want workgroups: one fragment, two above 8192 tokens.  But every workgroup reads the whole gate, 3 E / (16 frags)
// bytes of it for a byte of x, from the caches: with one or two fragments at every size 5000 tokens x 7168 x 16 experts took
// 56 us (tiled 33, now 26), 65536 of them 351 (258, 241).  Where that traffic is large there is a fragment for every four
// experts, and above 8192 tokens twice as many unless that fills the CUs' rounds less (40000 tokens x 7168 x 16: eight 214,
// four 194; 9000: 40 and 52); with as full rounds eight pay from H = 4096 (65536 tokens x 2048 x 12: eight 87, four 82;
// x 4096: 155 and 160).  Where it is small the workgroups count for more (9000 tokens x 256 x 16: two 11.1, eight 11.9).
static int small_gate_frags(int T, int H, int E) {
  if (T <= 2048 || static_cast<long>(T) * E * H <= 96l << 20) return T > 8192 ? 2 : 1;
  const int f = E <= 4 ? 1 : (E <= 8 ? 2 : 4);
  if (T <= 8192) return f;
  auto wgs = [&](int frags) {
    const long blocks = (static_cast<long>(T) + 16 * frags - 1) / (16 * frags);
    return blocks * std::max(256 / blocks, 1l);  // one workgroup per CU, as the split of K below aims at
  };
  const long one = wgs(f), two = wgs(2 * f);
  const long one_share = one * ((two + 255) / 256), two_share = two * ((one + 255) / 256);  // of the rounds' places in use
  return E <= 4 || two_share > one_share || (two_share == one_share && (E <= 8 || H >= 4096)) ? 2 * f : f;
}

// Tile height and slices of the DMA pipeline, from what the pieces were seen to take, in microseconds: a k-step of a round of
// workgroups (one to a CU, their LDS stages fill it) 1.2 with 128 tokens and 2.04 with 256, a slice 0.6 per MB written and
// read, every eight slices of the top-k kernel's loads 1.  Over 46 batches of 200..16384 tokens x 64, 128, 256 experts the
// choice is 0.3 % above the best of all heights and slices on average, 3.1 % at most.  Before, the slices were those that give every
// CU one (256 tokens) or two workgroups (128), rounded up, and a last round of a few workgroups followed.  Packed router with the
// same top-k, before / now: 2500 tokens x 4096 x 128 experts 28.2 / 22.6 us, 2048 x 7168 x 256 41.2 / 33.7, 5500 87.4 / 69.7, 12000
// 149.6 / 118.7; both gates of 2500 x 4096 x 128 in one call 42.6 / 30.1.
// Fewer slices are longer chains of additions: where a chain grows its sums are made by k-step, and their error against 64
// bits falls (probabilities, 5500 x 7168 x 256: 7.5e-7 before, 2.8e-7; 2500 x 4096 x 128: 2.9e-7, 2.1e-7).  The 128-token tile
// always does that; the 256-token tile loses 3 to 5 % by it and keeps to the accumulators where its chains stay as short.
// The shape that the room is made for stays unless another should be a tenth faster: below that the estimate does not decide.
static void choose_gate_tiles(RouteShape& s, int T, int ksteps) {
  const int bm_room = s.bm, steps_room = s.k_chunk / GBK;
  const double slice = 0.6e-6 * sizeof(float) * T * s.ld;
  auto cost = [&](int bm, int ks, int steps) {
    const int rounds = ((T + bm - 1) / bm * s.nt * ks + 255) / 256;
    return rounds * steps * (bm == 128 ? 1.2 : 2.04) + slice * ks + (ks + 7) / 8;
  };
  double best = 0.9 * cost(bm_room, s.ks_room, steps_room);
  for (const int bm : {128, 256}) {
    for (int ks = 1; ks <= s.ks_room; ++ks) {
      const int steps = (ksteps + ks - 1) / ks;
      if ((ksteps + steps - 1) / steps != ks || cost(bm, ks, steps) >= best) continue;  // or the same steps in fewer slices
      best = cost(bm, ks, steps);
      s.bm = bm;
      s.ks = ks;
      s.k_chunk = steps * GBK;
    }
  }
  s.mt = (T + s.bm - 1) / s.bm;
  s.stepwise = s.bm == 128 || s.k_chunk / GBK > steps_room;
}

// What the direct kernel's launch is: `frags`, `per_wave` and the slices.
static void direct_shape(RouteShape& s, int T, int H, int E, int max_split) {
  // eight fragments of tokens share a gate fragment where there are that many
  s.frags = E <= kDirectExperts ? small_gate_frags(T, H, E) : (T <= 16 ? 1 : (T <= 32 ? 2 : (T <= 64 ? 4 : 8)));
  const int k32 = (H + 31) / 32, wgs = ((E + 15) / 16) * ((T + 16 * s.frags - 1) / (16 * s.frags));
  int split = wgs > 0 ? 256 / wgs : 1;  // one workgroup per CU
  split = split < 1 ? 1 : (split > max_split ? max_split : split);
  s.per_wave = (k32 + 8 * split - 1) / (8 * split);
  s.ks = (k32 + 8 * s.per_wave - 1) / (8 * s.per_wave);
}

// Gates above kDirectLogits that the direct kernel still does faster (H % 64 == 0).  What it costs goes with the k32 per wave.  Call, tiled /
// direct.  One k32 gains from H = 1024 on: 1000 tokens x 1024 x 128 13.3 / 12.0 us, 256 x 2048 x 256 1.14 x, 384 x 2880 x 96 13.2 / 11.7; with a
// shorter H it loses where the experts fill their tiles badly (1000 x 512 x 48 8.5 / 9.4).  Two gain where the tiled kernel's columns of 128
// experts are mostly full, one at any batch, two up to two token blocks: 320 x 4096 x 128 14.6 / 13.1, 640 x 2880 x 128 15.1 / 14.0, 512 x 4096
// x 96 14.5 / 13.5, 256 x 4096 x 256 17.0 / 15.9; but 1000 x 2880 x 80 14.6 / 15.1, 192 x 2880 x 200 13.9 / 15.0.  Three lose (640 x 4096 x 128
// 16.3 / 18.2).  An fp32 gate that two token blocks share needs no launch that splits it and gains more (256 x 4096 x 256 24.1 / 15.2), also
// where packed planes lose; but packed planes and the fp32 gate give the same bits, so they go one way.  Probabilities against 64 bits over
// 546 gates from 128 to 7168 wide (164 of them go this way): 3.6e-8 of the largest (mean of the rms; 1.3e-6 at most) tiled, 3.5e-8 (1.3e-6) with those above.
// The top-k adds the slices, eight at once: two k32 in fourteen slices lose (384 x 7168 x 96 16.8 / 17.1), and so do the most logits (1000 x
// 2048 x 128 15.0 / 15.2).
constexpr int kDirectMore = 131072, kDirectTwo = 98304, kDirectBlocks = 256, kDirectWide = 1024, kDirectEmpty = 32, kDirectSlices = 8;
static bool direct_of_more(const RouteShape& direct, int T, int H, int E) {
  const long logits = static_cast<long>(T) * E;
  if (logits > kDirectMore || direct.ks > direct.ks_room) return false;
  const bool full = direct.nt * GBN - E <= kDirectEmpty;
  return (direct.per_wave == 1 && H >= kDirectWide) ||
         (direct.per_wave == 2 && full && logits <= kDirectTwo && direct.ks <= kDirectSlices &&
          (direct.nt == 1 || (direct.nt == 2 && T <= kDirectBlocks)));
}

// The residual's GEMMs keep to the line of kDirectLogits.
static RouteShape route_shape(int T, int H, int E, bool residual = false, int max_split = kMaxSplitK) {
  RouteShape s;
  s.dma = gate_dma(H, E);
  s.nt = (E + GBN - 1) / GBN;
  s.ld = (E + 3) & ~3;
  s.bm = (s.dma && static_cast<long>((T + 255) / 256) * s.nt >= kBigTileItems) ? 256 : GBM;
  s.mt = (T + s.bm - 1) / s.bm;
  int tiles = s.mt * s.nt;
  int ksteps = (H + GBK - 1) / GBK;
  const int target = gate_target(s.bm);
  const int steps_per = gate_slice_steps(ksteps, tiles > 0 ? (target + tiles - 1) / tiles : 1, max_split);
  s.k_chunk = steps_per * GBK;
  s.ks = (ksteps + steps_per - 1) / steps_per;
  s.ks_room = s.ks;
  s.stepwise = false;
  s.direct = static_cast<long>(T) * E <= (H % 64 == 0 ? 1 : 8) * kDirectLogits ||
             (E <= kDirectExperts && T <= kDirectTokens);
  s.frags = s.per_wave = 0;
  if (!s.direct && s.dma && T > 0 && !residual) {
    RouteShape d = s;
    direct_shape(d, T, H, E, max_split);
    if (direct_of_more(d, T, H, E)) {
      s = d;
      s.direct = true;
    }
  } else if (s.direct) {
    direct_shape(s, T, H, E, max_split);
  }
  if (!s.direct && s.dma && T > 0) {
    choose_gate_tiles(s, T, ksteps);
  }
  s.planes_bytes = align_up(static_cast<size_t>(3) * E * H * sizeof(bf16_t), 256);
  s.partial_bytes = align_up(static_cast<size_t>(s.ks_room) * (T > 0 ? T : 1) * s.ld * sizeof(float), 256);
  return s;
}

template <int PL, bool SPLIT_W>
static void launch_gate_direct(const RouteShape& sh, hipStream_t st, const bf16_t* x, const GateRows& g, int T, int H,
                               int N, float* partial, int32_t* zero0, int32_t* zero1, int n_zero) {
  // A gate of one fragment is served at any batch: its token blocks are on x, the one dimension that takes more than 65535 of
  // them.  With more fragments (T x N is bounded) those go first: the workgroups that share x run side by side.
  const unsigned blocks = (T + 16 * sh.frags - 1) / (16 * sh.frags);
  const dim3 grid = N <= 16 ? dim3(blocks, 1, sh.ks) : dim3((N + 15) / 16, sh.ks, blocks);
#define PROBE_DIRECT_CASE(NT, KU)                                                                                  \
  case NT:                                                                                                          \
    hipLaunchKernelGGL((gate_direct_kernel<NT, KU, PL, SPLIT_W>), grid, dim3(512), 0, st, x, g, T, H, N, sh.per_wave, \
                       partial, sh.ld, zero0, zero1, n_zero);                                                              \
    break;
  switch (sh.frags) {
    PROBE_DIRECT_CASE(1, 4)
    PROBE_DIRECT_CASE(2, 4)
    PROBE_DIRECT_CASE(4, 2)
    PROBE_DIRECT_CASE(8, 2)
  }
#undef PROBE_DIRECT_CASE
}

// x [T,H] times a stack of PL bf16 planes [PL][N][H] -> partial [ks][T][sh.ld] fp32
template <int PL>
static void launch_gate_gemm(const RouteShape& sh, hipStream_t st, const bf16_t* x, const bf16_t* planes, int T,
                             int H, int N, float* partial, int32_t* zero0 = nullptr, int32_t* zero1 = nullptr,
                             int n_zero = 0) {
  if (sh.direct) {
    launch_gate_direct<PL, false>(sh, st, x, GateRows{planes, nullptr, nullptr, 0}, T, H, N, partial, zero0, zero1, n_zero);
  } else if (sh.dma) {
    const int lds = gate_stages(sh.bm / 64, PL) * (sh.bm + 128 * PL) * 128;
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(sh.mt, sh.nt, sh.ks), dim3(512), lds, st, x, planes, T, H, N, sh.k_chunk, partial, sh.ld,
                         zero0, zero1, n_zero);
    };
    if (sh.bm == 128)
      launch(gate_gemm_dma_kernel<2, PL, true>);
    else if (sh.stepwise)
      launch(gate_gemm_dma_kernel<4, PL, true>);
    else
      launch(gate_gemm_dma_kernel<4, PL, false>);
  } else {
    hipLaunchKernelGGL(gate_gemm_kernel<PL>, dim3(sh.mt, sh.nt, sh.ks), dim3(256), 0, st, x, planes, T, H, N,
                       sh.k_chunk, partial, sh.ld, zero0, zero1, n_zero);
  }
}

// Whether the fp32 gate is split in the direct kernel's registers instead of by a launch of its own (2..7 us): at most
// two token blocks, i.e. every weight is converted at most twice, or a gate of one fragment and few blocks.
static bool split_in_registers(const RouteShape& sh, int T, int N) {
  return sh.direct && (T <= 2 * 16 * sh.frags || (N <= kDirectExperts && T <= 512));
}

// Workspace of a call: gate planes | logit partials (+ one plane for the residual) | u partials
struct RouteLayout {
  RouteShape gate, resid, resid2;  // gate GEMM; u = W1_hat h; r = W2_hat silu(u)
  size_t partial_bytes, upartial_bytes, a_bytes, b_bytes, total;
};

static RouteLayout route_layout(int T, int H, int E, int D, bool packed = false) {
  RouteLayout L;
  L.gate = route_shape(T, H, E);
  if (packed) L.gate.planes_bytes = 0;  // the caller holds the planes (probe_pack_gate)
  const size_t plane = static_cast<size_t>(T > 0 ? T : 1) * L.gate.ld * sizeof(float);
  L.upartial_bytes = L.a_bytes = L.b_bytes = 0;
  int extra = 0;
  if (D > 0) {
    L.resid = route_shape(T, H, D, true);
    L.resid2 = route_shape(T, 3 * D, E, true, kResidSplitK);
    L.upartial_bytes = L.resid.partial_bytes;
    L.a_bytes = align_up(static_cast<size_t>(T > 0 ? T : 1) * 3 * D * sizeof(bf16_t), 256);
    L.b_bytes = L.resid2.planes_bytes;
    extra = L.resid2.ks_room;
  }
  L.partial_bytes = align_up((L.gate.ks_room + extra) * plane, 256);
  L.total = L.gate.planes_bytes + L.partial_bytes + L.upartial_bytes + L.a_bytes + L.b_bytes;
  return L;
}

// The most slices x tokens (ks_room * T') over all T' <= T.  A tiled GEMM's slice count falls in steps as T grows, and a
// workspace sized for T has to serve every smaller batch: 7168 x 256 experts demands 46.7 MB for 2176 tokens, 42.2 for 2177.
// For each number of slices wished for, the largest batch that still gets it; in either range of tile heights.
static size_t most_slice_tokens(int T, int H, int E, int max_split) {
  const int nt = (E + GBN - 1) / GBN, ksteps = (H + GBK - 1) / GBK;
  const int first_big = gate_dma(H, E) ? 256 * ((kBigTileItems + nt - 1) / nt - 1) + 1 : INT_MAX;  // batch of 256-token tiles
  size_t most = 1;
  for (const int bm : {GBM, 256}) {
    const int lo = bm == 256 ? first_big : 1, hi = bm == 256 ? T : std::min(T, first_big - 1);
    for (int want = max_split; want >= 1 && lo <= hi; --want) {
      // up to (target - 1) / (want - 1) tiles wish for `want` slices or more
      const int t = want == 1 ? hi : std::min(hi, (gate_target(bm) - 1) / (want - 1) / nt * bm);
      const int steps = gate_slice_steps(ksteps, want, max_split);
      if (t >= lo) most = std::max(most, static_cast<size_t>(t) * ((ksteps + steps - 1) / steps));
      if (t == hi) break;  // fewer slices of as many tokens
    }
  }
  return most;
}

// What the workspace queries return: room for any batch of up to T tokens.
static size_t route_query_bytes(int T, int H, int E, int D, bool packed = false) {
  const RouteLayout L = route_layout(T, H, E, D, packed);
  size_t rows = most_slice_tokens(T, H, E, kMaxSplitK), u_bytes = 0;
  if (D > 0) {
    rows += most_slice_tokens(T, 3 * D, E, kResidSplitK);
    u_bytes = align_up(most_slice_tokens(T, H, D, kMaxSplitK) * L.resid.ld * sizeof(float), 256);
  }
  return L.gate.planes_bytes + align_up(rows * L.gate.ld * sizeof(float), 256) + u_bytes + L.a_bytes + L.b_bytes;
}

// workgroups of a top-k kernel that take `tokens` each; beyond 4096 they go round
static unsigned topk_blocks(int T, int tokens) { return static_cast<unsigned>(std::min((T + tokens - 1) / tokens, 4096)); }

// A whole wave per token where tokens are few and slices many: its four rows load a quarter of the slices each, all of them at
// once.  The selection is then made by all four rows, and there are four times as many workgroups to add their counts, so
// with more tokens it loses, and with up to eight slices, which sixteen lanes have in flight at once, it loses at any.  Call with sixteen
// lanes / with a wave per token: 4096 x 128 experts 64 tokens 10.1 / 9.4 us, 192 level, 256 12.0 / 12.55; 7168 x 256 64 14.9 / 12.6, 384
// 22.6 / 21.8, 512 24.0 / 23.8; 2560 x 64 32 tokens 8.2 / 7.85, 128 level; but 1088 x 128 64 tokens 8.95 / 9.2, 256 10.4 / 11.45,
// 640 x 256 256 tokens 13.7 / 14.1.  Group-limited, 75 tokens of 7168 x 256 22.1 / 19.4.
// `own` counts the gate's own slices, not those of a residual behind them: a residual of zeros leaves every bit as it was.
static bool wave_per_token(int T, int E, int own) { return own > 8 && T <= (E <= 128 ? 96 : 128) * ((E + 63) / 64); }

// Softmax and top-k of one gate, or of two stacked ones in one launch: either alone is a few microseconds of latency.  Router and
// predictor of 4096 x 128 experts, one call: 128 tokens 29.8 us in two launches of two tokens per row, 11.7 now; 1024 37.9 / 22.8,
// 2500 54.6 / 42.6, 8192 65.0 / 57.7.
static void launch_topk(hipStream_t st, const TopkGate& gate, const TopkGate* next, int ld, int KS, int own, int T, int E,
                        int k, int renorm) {
  const unsigned gates = next ? 2 : 1;
  const TopkGate& second = next ? *next : gate;
#define PROBE_TOPK_LAUNCH(NV, U, R, SG)                                                                        \
  hipLaunchKernelGGL((gate_softmax_topk_kernel<NV, U, R, SG>), dim3(topk_blocks(T, 16 * U / SG), gates), dim3(256), 0, \
                     st, gate, second, ld, KS, T, E, k, renorm)
#define PROBE_TOPK_BY_E(U, R, SG)                                                                                   \
  do {                                                                                                              \
    if (E <= 64) PROBE_TOPK_LAUNCH(1, U, R, SG);                                                                    \
    else if (E <= 128) PROBE_TOPK_LAUNCH(2, U, R, SG);                                                              \
    else PROBE_TOPK_LAUNCH(4, U, R, SG);                                                                            \
  } while (0)
  // Sixteen lanes per token: one token per row and eight slices in flight while latency bounds the kernel, two tokens and two
  // slices once instructions do.  Call, one / two: 2500 tokens x 4096 x 128 experts (11 slices) 28.8 / 31.2 us, 8192 42.0 /
  // 40.7, 16384 x 1024 x 64 38.0 / 29.4; two gates of 2500 x 4096 x 128 42.6 / 42.9, of 8192 59.1 / 57.7.  With four slices
  // or fewer there is little to keep in flight: 4096 x 4096 x 8 experts 16.2 / 15.2.
  if (wave_per_token(T, E, own))
    PROBE_TOPK_BY_E(1, 4, 4);
  else if (static_cast<long>(T) * gates > 6144 || (T > 2048 && KS <= 4))
    PROBE_TOPK_BY_E(2, 2, 1);
  else
    PROBE_TOPK_BY_E(1, 8, 1);
#undef PROBE_TOPK_BY_E
#undef PROBE_TOPK_LAUNCH
}

static void launch_grouped_topk(hipStream_t st, const TopkGate& g, int ld, int KS, const float* select_bias,
                                const probe_gating& gating, int T, int E, int k) {
#define PROBE_GROUPED_LAUNCH(NV, U, R, SG)                                                                       \
  hipLaunchKernelGGL((gate_grouped_topk_kernel<NV, U, R, SG>), dim3(topk_blocks(T, 16 * U / SG)), dim3(256), 0, st,   \
                     g.partial, ld, KS, g.bias, g.G, g.tpg, select_bias, T, E, k, gating.scoring, gating.n_group,     \
                     gating.topk_group, gating.group_top, gating.renormalize ? 1 : 0, gating.routed_scale, g.topk_idx, \
                     g.topk_w, g.probs, g.counts)
  // one token per row and up to eight slices in flight while latency bounds the kernel; two tokens and two slices once there
  // are enough rows and instructions bound it, which at more than 128 experts they did not up to 40000 tokens.  Call
  // with one / two tokens per row: 4096 x 1024 x 64 experts 24.1 / 26.2 us, 8192 30.7 / 28.4, 16384 39.6 / 32.7; 8192 x
  // 1024 x 128 33.1 / 34.1, 13421 43.1 / 36.4; 16384 x 1024 x 256 59.6 / 63.1.  There the selection holds so many registers that
  // only two slices are in flight (four: 8192 x 7168 x 256 85.6 -> 90.0, a wave per token 75 19.1 -> 19.6).
  if (wave_per_token(T, E, KS)) {
    if (E <= 64) PROBE_GROUPED_LAUNCH(1, 1, 4, 4); else if (E <= 128) PROBE_GROUPED_LAUNCH(2, 1, 4, 4); else PROBE_GROUPED_LAUNCH(4, 1, 2, 4);
  } else if (E <= 64) {
    if (T > 6144) PROBE_GROUPED_LAUNCH(1, 2, 2, 1); else PROBE_GROUPED_LAUNCH(1, 1, 8, 1);
  } else if (E <= 128) {
    if (T > 8192) PROBE_GROUPED_LAUNCH(2, 2, 2, 1); else PROBE_GROUPED_LAUNCH(2, 1, 8, 1);
  } else {
    PROBE_GROUPED_LAUNCH(4, 1, 2, 1);
  }
#undef PROBE_GROUPED_LAUNCH
}

// Router (w1_hat == nullptr) or predictor with the residual MLP of Eq. 7 (w1_hat bf16 [D,H],
// w2_hat fp32 [E,D]).
static int route_impl(const char* name, const void* x_bf16, const float* w_gate, const float* bias,
                      int bias_groups, int tokens_per_group, const void* w1_hat, const float* w2_hat, int D,
                      int T, int H, int E, int k, int renormalize, int32_t* topk_idx, float* topk_w,
                      float* probs, int32_t* expert_counts, void* workspace, size_t workspace_bytes,
                      void* stream, const probe_gating* gating = nullptr, const float* select_bias = nullptr,
                      const void* packed = nullptr) {
  // w_gate (fp32, split into planes inside the call) or packed (planes made once by probe_pack_gate)
  PROBE_REQUIRE(T >= 0 && H > 0 && E > 0 && k > 0 && k <= E, PROBE_EINVAL,
                "%s: bad dims T=%d H=%d E=%d k=%d", name, T, H, E, k);
  PROBE_REQUIRE(bias == nullptr || (bias_groups >= 1 && tokens_per_group >= 1), PROBE_EINVAL,
                "%s: bias_groups=%d tokens_per_group=%d", name, bias_groups, tokens_per_group);
  PROBE_REQUIRE(E <= PROBE_MAX_EXPERTS && k <= PROBE_MAX_TOPK && H % 8 == 0, PROBE_EUNSUPPORTED,
                "%s: needs E <= %d, k <= %d, H %% 8 == 0 (E=%d k=%d H=%d)", name, PROBE_MAX_EXPERTS,
                PROBE_MAX_TOPK, E, k, H);
  if (gating) {
    const probe_gating& g = *gating;
    PROBE_REQUIRE(g.scoring == PROBE_SCORE_SOFTMAX || g.scoring == PROBE_SCORE_SIGMOID, PROBE_EINVAL,
                  "%s: scoring=%d", name, g.scoring);
    PROBE_REQUIRE(g.n_group >= 1 && E % g.n_group == 0 && g.topk_group >= 1 && g.topk_group <= g.n_group,
                  PROBE_EINVAL, "%s: n_group=%d must divide E=%d, topk_group=%d must be in 1..n_group", name,
                  g.n_group, E, g.topk_group);
    PROBE_REQUIRE(g.group_top >= 1 && g.group_top <= E / g.n_group && k <= g.topk_group * (E / g.n_group),
                  PROBE_EINVAL, "%s: group_top=%d and k=%d must fit %d groups of %d experts", name, g.group_top, k,
                  g.topk_group, E / g.n_group);
    PROBE_REQUIRE(g.n_group <= PROBE_MAX_GROUPS, PROBE_EUNSUPPORTED, "%s: needs n_group <= %d (n_group=%d)", name,
                  PROBE_MAX_GROUPS, g.n_group);
    PROBE_REQUIRE(aligned16(select_bias), PROBE_EALIGN, "%s: select_bias must be 16-byte aligned", name);
  }
  PROBE_REQUIRE(w_gate != nullptr || packed != nullptr, PROBE_EINVAL, "%s: the gate is NULL", name);
  PROBE_REQUIRE(T == 0 || (x_bf16 && topk_idx && topk_w), PROBE_EINVAL, "%s: null pointer", name);
  PROBE_REQUIRE(aligned16(x_bf16) && aligned16(w_gate) && aligned16(packed), PROBE_EALIGN,
                "%s: x and the gate must be 16-byte aligned", name);
  PROBE_REQUIRE(aligned16(bias) && aligned16(probs), PROBE_EALIGN,
                "%s: bias and probs must be 16-byte aligned", name);
  const bool resid = D > 0;
  if (resid) {
    PROBE_REQUIRE(w1_hat && w2_hat, PROBE_EINVAL, "%s: residual weights are NULL", name);
    PROBE_REQUIRE(D % 8 == 0 && D <= PROBE_MAX_RESIDUAL_WIDTH, PROBE_EUNSUPPORTED,
                  "%s: needs D %% 8 == 0 and D <= %d (D=%d)", name, PROBE_MAX_RESIDUAL_WIDTH, D);
    PROBE_REQUIRE(aligned16(w1_hat) && aligned16(w2_hat), PROBE_EALIGN,
                  "%s: w1_hat and w2_hat must be 16-byte aligned", name);
  }
  RouteLayout L = route_layout(T, H, E, resid ? D : 0, packed != nullptr);
  const RouteShape& sh = L.gate;
  PROBE_REQUIRE(workspace && aligned16(workspace) && workspace_bytes >= L.total, PROBE_EWORKSPACE,
                "%s: workspace too small or misaligned (%zu < %zu)", name, workspace_bytes, L.total);
  if (T > 0 && (sh.dma || (resid && (L.resid.dma || L.resid2.dma)))) {
    int rc = gate_prepare();
    if (rc != PROBE_OK) return rc;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  const bf16_t* x = static_cast<const bf16_t*>(x_bf16);
  const bf16_t* planes = static_cast<const bf16_t*>(packed);
  float* partial = reinterpret_cast<float*>(static_cast<char*>(workspace) + sh.planes_bytes);
  float* upartial = reinterpret_cast<float*>(static_cast<char*>(workspace) + sh.planes_bytes + L.partial_bytes);
  const long n = static_cast<long>(E) * H;
  if (T == 0) {  // nothing to route: only the counts are cleared
    if (expert_counts)
      hipLaunchKernelGGL(gate_split_kernel, dim3((E + 255) / 256), dim3(256), 0, st, w_gate, 0l, nullptr, 0l,
                         expert_counts, E);
  } else if (packed == nullptr && !split_in_registers(sh, T, E)) {
    bf16_t* ws_planes = static_cast<bf16_t*>(workspace);
    hipLaunchKernelGGL(gate_split_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st, w_gate, n,
                       ws_planes, n, nullptr, E);
    planes = ws_planes;
  }
  if (T > 0) {
    if (planes == nullptr)
      launch_gate_direct<3, true>(sh, st, x, GateRows{nullptr, w_gate, nullptr, E}, T, H, E, partial, expert_counts,
                                  nullptr, expert_counts ? E : 0);
    else
      launch_gate_gemm<3>(sh, st, x, planes, T, H, E, partial, expert_counts, nullptr, expert_counts ? E : 0);
    int planes_to_sum = sh.ks;
    if (resid) {
      // u = W1_hat h (one bf16 plane); s = silu(u) and W2_hat split into planes; r = W2_hat s as
      // further slices of the logits
      char* base = static_cast<char*>(workspace) + sh.planes_bytes + L.partial_bytes + L.upartial_bytes;
      bf16_t* a_planes = reinterpret_cast<bf16_t*>(base);
      bf16_t* b_planes = reinterpret_cast<bf16_t*>(base + L.a_bytes);
      launch_gate_gemm<1>(L.resid, st, x, static_cast<const bf16_t*>(w1_hat), T, H, D, upartial);
      const unsigned a_blocks = resid_split_blocks(T, D);
      hipLaunchKernelGGL(resid_split_kernel, dim3(a_blocks + resid_split_blocks(E, D)), dim3(256), 0, st, upartial,
                         L.resid.ks, T, w2_hat, E, D, a_blocks, a_planes, b_planes);
      launch_gate_gemm<3>(L.resid2, st, a_planes, b_planes, T, 3 * D, E, partial + static_cast<size_t>(sh.ks) * T * sh.ld);
      planes_to_sum = sh.ks + L.resid2.ks;
    }
    const TopkGate out = {partial, bias, bias ? bias_groups : 1, bias ? tokens_per_group : 1, topk_idx, topk_w, probs,
                          expert_counts};
    if (gating)
      launch_grouped_topk(st, out, sh.ld, planes_to_sum, select_bias, *gating, T, E, k);
    else
      launch_topk(st, out, nullptr, sh.ld, planes_to_sum, sh.ks, T, E, k, renormalize ? 1 : 0);
  }
  return check_launch(name);
}

// Router of layer L-1 and zero-residual predictor of layer L on the same hidden states in one pass:
// the two gates are stacked into one operand of 2E rows per plane, one GEMM produces both sets of
// logits (x is read once, half as many split-K slices), the softmax / top-k kernel runs once per
// gate on its half of the columns.
static int route_predict_impl(const void* x_bf16, const float* w_gate, const float* bias,
                              const float* w_gate_next, const float* bias_next, int bias_groups,
                              int tokens_per_group, int T, int H, int E, int k, int renormalize,
                              int32_t* topk_idx, float* topk_w, float* probs, int32_t* expert_counts,
                              int32_t* pred_idx, float* pred_w, float* pred_probs, int32_t* pred_counts,
                              void* workspace, size_t workspace_bytes, void* stream,
                              const void* packed_stack = nullptr) {
  // (w_gate, w_gate_next) in fp32, or packed_stack: both gates packed into one stack of 2E rows
  const char* name = packed_stack ? "probe_route_predict_topk_packed" : "probe_route_predict_topk";
  PROBE_REQUIRE(T >= 0 && H > 0 && E > 0 && k > 0 && k <= E, PROBE_EINVAL,
                "%s: bad dims T=%d H=%d E=%d k=%d", name, T, H, E, k);
  PROBE_REQUIRE((bias == nullptr && bias_next == nullptr) || (bias_groups >= 1 && tokens_per_group >= 1),
                PROBE_EINVAL, "%s: bias_groups=%d tokens_per_group=%d", name, bias_groups, tokens_per_group);
  PROBE_REQUIRE(E <= PROBE_MAX_EXPERTS && k <= PROBE_MAX_TOPK && H % 8 == 0, PROBE_EUNSUPPORTED,
                "%s: needs E <= %d, k <= %d, H %% 8 == 0 (E=%d k=%d H=%d)", name, PROBE_MAX_EXPERTS,
                PROBE_MAX_TOPK, E, k, H);
  PROBE_REQUIRE(packed_stack != nullptr || (w_gate != nullptr && w_gate_next != nullptr), PROBE_EINVAL,
                "%s: a gate is NULL", name);
  PROBE_REQUIRE(T == 0 || (x_bf16 && topk_idx && topk_w && pred_idx && pred_w), PROBE_EINVAL,
                "%s: null pointer", name);
  PROBE_REQUIRE(aligned16(x_bf16) && aligned16(w_gate) && aligned16(w_gate_next) && aligned16(packed_stack),
                PROBE_EALIGN, "%s: x and the gates must be 16-byte aligned", name);
  PROBE_REQUIRE(aligned16(bias) && aligned16(bias_next) && aligned16(probs) && aligned16(pred_probs), PROBE_EALIGN,
                "%s: biases and probability outputs must be 16-byte aligned", name);
  RouteLayout L = route_layout(T, H, 2 * E, 0, packed_stack != nullptr);
  const RouteShape& sh = L.gate;
  PROBE_REQUIRE(workspace && aligned16(workspace) && workspace_bytes >= L.total, PROBE_EWORKSPACE,
                "%s: workspace too small or misaligned (%zu < %zu)", name, workspace_bytes, L.total);
  if (T > 0 && sh.dma) {
    int rc = gate_prepare();
    if (rc != PROBE_OK) return rc;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  // planes [3][2E][H]: rows 0..E-1 this layer's gate, E..2E-1 the next
  const bf16_t* planes = static_cast<const bf16_t*>(packed_stack);
  float* partial = reinterpret_cast<float*>(static_cast<char*>(workspace) + sh.planes_bytes);
  const long n = static_cast<long>(E) * H;
  if (T == 0) {  // nothing to route: only the counts are cleared
    if (expert_counts)
      hipLaunchKernelGGL(gate_split_kernel, dim3((E + 255) / 256), dim3(256), 0, st, w_gate, 0l, nullptr, 0l,
                         expert_counts, E);
    if (pred_counts)
      hipLaunchKernelGGL(gate_split_kernel, dim3((E + 255) / 256), dim3(256), 0, st, w_gate, 0l, nullptr, 0l,
                         pred_counts, E);
  } else if (packed_stack == nullptr && !split_in_registers(sh, T, 2 * E)) {
    bf16_t* ws_planes = static_cast<bf16_t*>(workspace);
    const unsigned split_grid = static_cast<unsigned>((n + 255) / 256);
    hipLaunchKernelGGL(gate_split_kernel, dim3(split_grid), dim3(256), 0, st, w_gate, n, ws_planes, 2 * n, nullptr, E);
    hipLaunchKernelGGL(gate_split_kernel, dim3(split_grid), dim3(256), 0, st, w_gate_next, n, ws_planes + n, 2 * n,
                       nullptr, E);
    planes = ws_planes;
  }
  if (T > 0) {
    if (planes == nullptr)
      launch_gate_direct<3, true>(sh, st, static_cast<const bf16_t*>(x_bf16), GateRows{nullptr, w_gate, w_gate_next, E},
                                  T, H, 2 * E, partial, expert_counts, pred_counts, E);
    else
      launch_gate_gemm<3>(sh, st, static_cast<const bf16_t*>(x_bf16), planes, T, H, 2 * E, partial, expert_counts,
                          pred_counts, E);
    const TopkGate out = {partial, bias, bias ? bias_groups : 1, bias ? tokens_per_group : 1, topk_idx, topk_w, probs,
                          expert_counts};
    const TopkGate next = {partial + E, bias_next, bias_next ? bias_groups : 1, bias_next ? tokens_per_group : 1, pred_idx,
                           pred_w, pred_probs, pred_counts};
    launch_topk(st, out, &next, sh.ld, sh.ks, sh.ks, T, E, k, renormalize ? 1 : 0);
  }
  return check_launch(name);
}

}  // namespace probe

extern "C" size_t probe_route_topk_workspace_bytes(int T, int H, int E, int k) {
  (void)k;
  if (T < 0 || H <= 0 || E <= 0) return 0;
  return probe::route_query_bytes(T, H, E, 0);
}

extern "C" size_t probe_predict_topk_workspace_bytes(int T, int H, int E, int k) {
  return probe_route_topk_workspace_bytes(T, H, E, k);
}

extern "C" size_t probe_predict_topk_residual_workspace_bytes(int T, int H, int E, int k, int D) {
  (void)k;
  if (T < 0 || H <= 0 || E <= 0 || D <= 0) return 0;
  return probe::route_query_bytes(T, H, E, D);
}

extern "C" int probe_route_topk(const void* x_bf16, const float* w_gate, const float* bias,
                                int bias_groups, int tokens_per_group, int T, int H, int E, int k,
                                int renormalize, int32_t* topk_idx, float* topk_w, float* probs,
                                int32_t* expert_counts, void* workspace, size_t workspace_bytes,
                                void* stream) {
  return probe::route_impl("probe_route_topk", x_bf16, w_gate, bias, bias_groups, tokens_per_group, nullptr,
                           nullptr, 0, T, H, E, k, renormalize, topk_idx, topk_w, probs, expert_counts,
                           workspace, workspace_bytes, stream);
}

extern "C" size_t probe_route_grouped_workspace_bytes(int T, int H, int E, int k) {
  return probe_route_topk_workspace_bytes(T, H, E, k);
}

// The router with a model's own gate: same GEMM, group-limited selection in place of the plain top-k.
extern "C" int probe_route_grouped(const void* x_bf16, const float* w_gate, const float* bias, int bias_groups,
                                   int tokens_per_group, const float* select_bias, const probe_gating* gating,
                                   int T, int H, int E, int k, int32_t* topk_idx, float* topk_w, float* scores,
                                   int32_t* expert_counts, void* workspace, size_t workspace_bytes,
                                   void* stream) {
  PROBE_REQUIRE(gating != nullptr, PROBE_EINVAL, "probe_route_grouped: gating is NULL");
  return probe::route_impl("probe_route_grouped", x_bf16, w_gate, bias, bias_groups, tokens_per_group, nullptr,
                           nullptr, 0, T, H, E, k, gating->renormalize, topk_idx, topk_w, scores, expert_counts,
                           workspace, workspace_bytes, stream, gating, select_bias);
}

// Eq. 7 with the residual at its zero initialisation is the cloned router applied to the
// previous layer's hidden states: the same kernels, fed with (h_{L-1}, W_L, b_L).
extern "C" int probe_predict_topk(const void* h_prev_bf16, const float* w_gate_next,
                                  const float* bias_next, int bias_groups, int tokens_per_group,
                                  int T, int H, int E, int k, int renormalize, int32_t* pred_idx,
                                  float* pred_w, float* probs, int32_t* pred_counts, void* workspace,
                                  size_t workspace_bytes, void* stream) {
  return probe::route_impl("probe_predict_topk", h_prev_bf16, w_gate_next, bias_next, bias_groups,
                           tokens_per_group, nullptr, nullptr, 0, T, H, E, k, renormalize, pred_idx, pred_w,
                           probs, pred_counts, workspace, workspace_bytes, stream);
}

// Eq. 7 in full: the frozen prior plus W2_hat silu(W1_hat h).
extern "C" int probe_predict_topk_residual(const void* h_prev_bf16, const float* w_gate_next,
                                           const float* bias_next, int bias_groups, int tokens_per_group,
                                           const void* w1_hat_bf16, const float* w2_hat, int D, int T, int H,
                                           int E, int k, int renormalize, int32_t* pred_idx, float* pred_w,
                                           float* probs, int32_t* pred_counts, void* workspace,
                                           size_t workspace_bytes, void* stream) {
  PROBE_REQUIRE(D > 0, PROBE_EINVAL, "probe_predict_topk_residual: D=%d", D);
  return probe::route_impl("probe_predict_topk_residual", h_prev_bf16, w_gate_next, bias_next, bias_groups,
                           tokens_per_group, w1_hat_bf16, w2_hat, D, T, H, E, k, renormalize, pred_idx, pred_w,
                           probs, pred_counts, workspace, workspace_bytes, stream);
}

extern "C" size_t probe_route_predict_topk_workspace_bytes(int T, int H, int E, int k) {
  (void)k;
  if (T < 0 || H <= 0 || E <= 0) return 0;
  return probe::route_query_bytes(T, H, 2 * E, 0);
}

extern "C" int probe_route_predict_topk(const void* x_bf16, const float* w_gate, const float* bias,
                                        const float* w_gate_next, const float* bias_next, int bias_groups,
                                        int tokens_per_group, int T, int H, int E, int k, int renormalize,
                                        int32_t* topk_idx, float* topk_w, float* probs, int32_t* expert_counts,
                                        int32_t* pred_idx, float* pred_w, float* pred_probs,
                                        int32_t* pred_counts, void* workspace, size_t workspace_bytes,
                                        void* stream) {
  return probe::route_predict_impl(x_bf16, w_gate, bias, w_gate_next, bias_next, bias_groups, tokens_per_group, T,
                                   H, E, k, renormalize, topk_idx, topk_w, probs, expert_counts, pred_idx, pred_w,
                                   pred_probs, pred_counts, workspace, workspace_bytes, stream);
}

// ---- the gate packed once -------------------------------------------------------------------
// The router's (W_L, b_L) are frozen (Sec. 4.2), so the split of the fp32 gate into three bf16 planes
// need not be repeated on every call: probe_pack_gate writes the planes once, the *_packed entry points
// take them in place of the fp32 matrix.
extern "C" size_t probe_pack_gate_bytes(int H, int E_stack) {
  if (H <= 0 || E_stack <= 0) return 0;
  return probe::align_up(static_cast<size_t>(3) * E_stack * H * sizeof(probe::bf16_t), 256);
}

extern "C" int probe_pack_gate(const float* w_gate, int H, int E, int stack_rows, int row_offset,
                               void* packed, void* stream) {
  using namespace probe;
  PROBE_REQUIRE(H > 0 && E > 0 && stack_rows >= E && row_offset >= 0 && row_offset + E <= stack_rows, PROBE_EINVAL,
                "probe_pack_gate: bad dims H=%d E=%d stack_rows=%d row_offset=%d", H, E, stack_rows, row_offset);
  PROBE_REQUIRE(H % 8 == 0, PROBE_EUNSUPPORTED, "probe_pack_gate: needs H %% 8 == 0 (H=%d)", H);
  PROBE_REQUIRE(w_gate && packed, PROBE_EINVAL, "probe_pack_gate: null pointer");
  PROBE_REQUIRE(aligned16(w_gate) && aligned16(packed), PROBE_EALIGN,
                "probe_pack_gate: w_gate and packed must be 16-byte aligned");
  const long n = static_cast<long>(E) * H;
  hipLaunchKernelGGL(gate_split_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), w_gate, n,
                     static_cast<bf16_t*>(packed) + static_cast<long>(row_offset) * H,
                     static_cast<long>(stack_rows) * H, nullptr, E);
  return check_launch("probe_pack_gate");
}

extern "C" size_t probe_route_topk_packed_workspace_bytes(int T, int H, int E, int k) {
  (void)k;
  if (T < 0 || H <= 0 || E <= 0) return 0;
  return probe::route_query_bytes(T, H, E, 0, true);
}

extern "C" int probe_route_topk_packed(const void* x_bf16, const void* packed_gate, const float* bias,
                                       int bias_groups, int tokens_per_group, int T, int H, int E, int k,
                                       int renormalize, int32_t* topk_idx, float* topk_w, float* probs,
                                       int32_t* expert_counts, void* workspace, size_t workspace_bytes,
                                       void* stream) {
  PROBE_REQUIRE(packed_gate != nullptr, PROBE_EINVAL, "probe_route_topk_packed: packed_gate is NULL");
  return probe::route_impl("probe_route_topk_packed", x_bf16, nullptr, bias, bias_groups, tokens_per_group, nullptr,
                           nullptr, 0, T, H, E, k, renormalize, topk_idx, topk_w, probs, expert_counts, workspace,
                           workspace_bytes, stream, nullptr, nullptr, packed_gate);
}

extern "C" int probe_predict_topk_packed(const void* h_prev_bf16, const void* packed_gate_next,
                                         const float* bias_next, int bias_groups, int tokens_per_group, int T,
                                         int H, int E, int k, int renormalize, int32_t* pred_idx, float* pred_w,
                                         float* probs, int32_t* pred_counts, void* workspace,
                                         size_t workspace_bytes, void* stream) {
  PROBE_REQUIRE(packed_gate_next != nullptr, PROBE_EINVAL, "probe_predict_topk_packed: packed_gate_next is NULL");
  return probe::route_impl("probe_predict_topk_packed", h_prev_bf16, nullptr, bias_next, bias_groups,
                           tokens_per_group, nullptr, nullptr, 0, T, H, E, k, renormalize, pred_idx, pred_w, probs,
                           pred_counts, workspace, workspace_bytes, stream, nullptr, nullptr, packed_gate_next);
}

extern "C" int probe_route_grouped_packed(const void* x_bf16, const void* packed_gate, const float* bias,
                                          int bias_groups, int tokens_per_group, const float* select_bias,
                                          const probe_gating* gating, int T, int H, int E, int k,
                                          int32_t* topk_idx, float* topk_w, float* scores,
                                          int32_t* expert_counts, void* workspace, size_t workspace_bytes,
                                          void* stream) {
  PROBE_REQUIRE(gating != nullptr, PROBE_EINVAL, "probe_route_grouped_packed: gating is NULL");
  PROBE_REQUIRE(packed_gate != nullptr, PROBE_EINVAL, "probe_route_grouped_packed: packed_gate is NULL");
  return probe::route_impl("probe_route_grouped_packed", x_bf16, nullptr, bias, bias_groups, tokens_per_group,
                           nullptr, nullptr, 0, T, H, E, k, gating->renormalize, topk_idx, topk_w, scores,
                           expert_counts, workspace, workspace_bytes, stream, gating, select_bias, packed_gate);
}

extern "C" size_t probe_route_predict_topk_packed_workspace_bytes(int T, int H, int E, int k) {
  (void)k;
  if (T < 0 || H <= 0 || E <= 0) return 0;
  return probe::route_query_bytes(T, H, 2 * E, 0, true);
}

extern "C" int probe_route_predict_topk_packed(const void* x_bf16, const void* packed_stack, const float* bias,
                                               const float* bias_next, int bias_groups, int tokens_per_group,
                                               int T, int H, int E, int k, int renormalize, int32_t* topk_idx,
                                               float* topk_w, float* probs, int32_t* expert_counts,
                                               int32_t* pred_idx, float* pred_w, float* pred_probs,
                                               int32_t* pred_counts, void* workspace, size_t workspace_bytes,
                                               void* stream) {
  PROBE_REQUIRE(packed_stack != nullptr, PROBE_EINVAL, "probe_route_predict_topk_packed: packed_stack is NULL");
  return probe::route_predict_impl(x_bf16, nullptr, bias, nullptr, bias_next, bias_groups, tokens_per_group, T, H, E,
                                   k, renormalize, topk_idx, topk_w, probs, expert_counts, pred_idx, pred_w,
                                   pred_probs, pred_counts, workspace, workspace_bytes, stream, packed_stack);
}
