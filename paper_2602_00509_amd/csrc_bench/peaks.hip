// Measurement aid of bench.py, built into its own library (libprobe_peaks.so) and not part of libprobe:
// an MFMA-only loop (16x16x32 bf16, the instruction of the GEMM main loops) with its operands in registers.  bench.py times it to report what the matrix cores of
// the box sustain with no memory instruction in flight, for zero operands and for random bf16 operands
// (the chip is power-limited under matrix work and the operand bits decide how far).
//
//   double peaks_mfma_flops_per_launch(int workgroups, int iters)      flops of one launch (host arithmetic)
//   int    peaks_mfma(float* out, int workgroups, int iters, int random_operands, void* stream)
//          out: device, fp32 [workgroups * 512] (one checksum per thread; keeps the loop alive);
//          returns 0, -1 for bad arguments, -5 if the launch was rejected
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace peaks {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

__device__ __forceinline__ f32x4 mfma_16x16x32(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

__device__ __forceinline__ uint32_t xorshift(uint32_t& s) {
  s ^= s << 13;
  s ^= s >> 17;
  s ^= s << 5;
  return s;
}

// two bf16 values with random sign and mantissa and one of four exponents (|v| in [1/8, 2))
__device__ __forceinline__ uint32_t random_bf16x2(uint32_t& s) {
  const uint32_t r = xorshift(s);
  const uint32_t e1 = 0x3c + ((r >> 8) & 3), e2 = 0x3c + ((r >> 24) & 3);
  return (r & 0x807f807fu) | (e1 << 7) | (e2 << 23);
}

// 8 waves per workgroup, each with an 8 x 4 grid of 16x16 accumulators, columns back and forth as in the GEMM main loop.
__global__ __launch_bounds__(512, 2) void mfma_peak_kernel(float* __restrict__ out, int iters, int random) {
  uint32_t s = threadIdx.x * 2654435761u + blockIdx.x * 40503u + 12345u;
  u32x4 a[8], b[4];
  for (int i = 0; i < 8; ++i)
    for (int j = 0; j < 4; ++j) a[i][j] = random ? random_bf16x2(s) : 0u;
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) b[i][j] = random ? random_bf16x2(s) : 0u;
  f32x4 acc[8][4];
  for (int i = 0; i < 8; ++i)
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int j = (i & 1) ? 3 - c : c;
        acc[i][j] = mfma_16x16x32(b[j], a[i], acc[i][j]);
      }
    if (random) a[0][0] ^= 0x00150015u;  // keep the operand bits moving
  }
  float sum = 0.f;
  for (int i = 0; i < 8; ++i)
    for (int j = 0; j < 4; ++j)
      for (int r = 0; r < 4; ++r) sum += acc[i][j][r];
  out[blockIdx.x * blockDim.x + threadIdx.x] = sum;
}

}  // namespace peaks

extern "C" double peaks_mfma_flops_per_launch(int workgroups, int iters) {
  // 8 waves x 32 MFMAs per iteration x 2 * 16 * 16 * 32 flops
  return static_cast<double>(workgroups) * 8.0 * iters * 32.0 * 16384.0;
}

extern "C" int peaks_mfma(float* out, int workgroups, int iters, int random_operands, void* stream) {
  if (out == nullptr || workgroups <= 0 || workgroups > 65536 || iters <= 0) return -1;
  hipLaunchKernelGGL(peaks::mfma_peak_kernel, dim3(workgroups), dim3(512), 0, static_cast<hipStream_t>(stream), out,
                     iters, random_operands);
  return hipGetLastError() == hipSuccess ? 0 : -5;
}
