// Matrix-core throughput probe for the benchmark's measured-peak figure. It is
// built into its own library (libmte_probe.so), not into libmte: it measures
// the chip, it is no part of the encoder.
//
// Every wave runs `iters` rounds of sixteen independent v_mfma_f32_16x16x32_f16,
// the form of the projection GEMMs, on the products of four A and four B
// fragments of random values (no memory traffic inside the loop), so the
// kernel's duration gives the dense fp16 rate the chip sustains at the clock it
// runs under that load. Operands matter: the card's power limit sets that clock,
// and zero operands, which toggle no bits, run at 2.37 PFLOP/s where random ones
// run at 1.86 ... 1.96.
//
//   int mte_probe_mfma(int32_t blocks, int32_t iters, float *sink, hipStream_t stream);
//
// Enqueues `blocks` workgroups of four waves on `stream`; every wave does
// iters * 16 MFMAs of 16384 flops. sink: device float[blocks * 256], one value
// per thread, overwritten. Returns 0, -1 for a null sink or non-positive
// blocks / iters (checked before any HIP call), -3 if the launch fails.
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kFrags = 4;   // fragments per operand; kFrags^2 independent accumulators

// A value in [-1, 1) from a hash of n.
__device__ __forceinline__ _Float16 draw(uint32_t n) {
  n ^= n >> 16;
  n *= 0x7feb352dU;
  n ^= n >> 15;
  n *= 0x846ca68bU;
  n ^= n >> 16;
  return (_Float16)((float)(int32_t)n * (1.f / 2147483648.f));
}

// (the bound on waves per SIMD keeps the accumulators in place; without it the
// compiler rotates them through register copies between the MFMAs)
__global__ __launch_bounds__(256, 2) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mfma_probe(int iters, float *sink) {
  const uint32_t seed = (blockIdx.x * 256u + threadIdx.x) * (2u * kFrags * 8u);
  f16x8 a[kFrags], b[kFrags];
#pragma unroll
  for (int f = 0; f < kFrags; ++f)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      a[f][e] = draw(seed + 8 * f + e);
      b[f][e] = draw(seed + 8 * (kFrags + f) + e);
    }
  f32x4 acc[kFrags][kFrags];
#pragma unroll
  for (int i = 0; i < kFrags; ++i)
#pragma unroll
    for (int j = 0; j < kFrags; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < kFrags; ++i)
#pragma unroll
      for (int j = 0; j < kFrags; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[i], b[j], acc[i][j], 0, 0, 0);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < kFrags; ++i)
#pragma unroll
    for (int j = 0; j < kFrags; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) s += acc[i][j][r];
  sink[blockIdx.x * 256 + threadIdx.x] = s;
}

}  // namespace

extern "C" int mte_probe_mfma(int32_t blocks, int32_t iters, float *sink, hipStream_t stream) {
  if (!sink || blocks <= 0 || iters <= 0) return -1;
  hipLaunchKernelGGL(k_mfma_probe, dim3(blocks), dim3(256), 0, stream, iters, sink);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}
