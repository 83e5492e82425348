// Row-wise kernels of the vision tower: patch extraction in merge-group
// order with the rotary table of the patches' places, and LayerNorm.
#include "common.h"
#include "launch.h"

namespace mte {

// Patch p of image n (merge-group order: groups of merge x merge patches
// row-major over the image, patches row-major inside a group) sits at patch
// row ph = merge*gr + dr, column pw = merge*gc + dc. Its vector is the
// image's pixels under it in (channel, row, column) order, the flattening
// of a Conv2d weight [hidden, C, patch, patch].
struct PatchGeom {
  int C, H, W, patch, merge;
  int gw;            // merge groups per row: W / (patch * merge)
  int per_image;     // patches per image
};

__device__ __forceinline__ void patch_rc(const PatchGeom &g, int p, int &ph, int &pw) {
  const int mm = g.merge * g.merge;
  const int grp = p / mm, in = p % mm;
  ph = g.merge * (grp / g.gw) + in / g.merge;
  pw = g.merge * (grp % g.gw) + in % g.merge;
}

// The rotary entries of a patch depend on its place only: pair j turns by the
// patch row (axis 1) or column (axis 2) times inv_freq[j], angle and sincos in
// float64, rounded.
__device__ __forceinline__ void patch_rope(const PatchGeom &g, const RopeParams &rp, int T, int half, size_t i,
                                           float *rcos, float *rsin) {
  if (i >= (size_t)T * half) return;
  const int tok = (int)(i / half), j = (int)(i % half);
  int ph, pw;
  patch_rc(g, tok % g.per_image, ph, pw);
  const double ang = (double)(rp.axis[j] == 1 ? ph : rp.axis[j] == 2 ? pw : 0) * rp.inv_freq[j];
  double sv, cv;
  sincos(ang, &sv, &cv);
  rcos[i] = (float)cv;
  rsin[i] = (float)sv;
}

// One launch opens the tower: the first rope_blocks blocks build the rotary
// table (256 entries each), the others extract patches, V consecutive values
// of a patch row per thread. V = 8 (16-byte accesses of bf16 pixels) where a
// patch row is a multiple of 8 pixels, else 1. Bound by memory; one value per
// thread, with its divisions, took 20 us for 16 images of 256x256 (6.3 MB in, 6.3
// MB out), and the positions and the table 5 us each in launches of their own.
template <typename TI, typename TO, int V>
__global__ __launch_bounds__(256) void k_vision_open(const TI *__restrict__ px, TO *__restrict__ out, PatchGeom g,
                                                     size_t total, RopeParams rp, int T, int half, int rope_blocks,
                                                     float *__restrict__ rcos, float *__restrict__ rsin) {
  if ((int)blockIdx.x < rope_blocks) {
    patch_rope(g, rp, T, half, (size_t)blockIdx.x * 256 + threadIdx.x, rcos, rsin);
    return;
  }
  typedef TI vi __attribute__((ext_vector_type(V), aligned(sizeof(TI))));   // pixels: a caller's buffer
  typedef TO vo __attribute__((ext_vector_type(V)));
  const size_t i = ((size_t)(blockIdx.x - rope_blocks) * 256 + threadIdx.x) * V;
  if (i >= total) return;
  const int K = g.C * g.patch * g.patch;
  const int row = (int)(i / K), k = (int)(i % K);
  const int n = row / g.per_image, p = row % g.per_image;
  int ph, pw;
  patch_rc(g, p, ph, pw);
  const int pp = g.patch * g.patch;
  const int c = k / pp, ky = (k % pp) / g.patch, kx = k % g.patch;
  const size_t src = (((size_t)n * g.C + c) * g.H + (size_t)ph * g.patch + ky) * g.W + (size_t)pw * g.patch + kx;
  const vi x = *(const vi *)(px + src);
  vo y;
#pragma unroll
  for (int e = 0; e < V; ++e) y[e] = from_f32<TO>(to_f32(x[e]));
  *(vo *)(out + i) = y;
}

hipError_t launch_vision_open(int in_fmt, const void *pixels, int n, int C, int H, int W, int patch, int merge,
                              int out_fmt, void *out, int half, const RopeParams &rp, float *rcos, float *rsin,
                              hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (H % (patch * merge) || W % (patch * merge)) return hipErrorInvalidValue;
  const PatchGeom g{C, H, W, patch, merge, W / (patch * merge), (H / patch) * (W / patch)};
  const int T = n * g.per_image;
  const size_t total = (size_t)T * C * patch * patch;
  const int v = patch % 8 == 0 ? 8 : 1;          // then every vector lies in one patch row
  const int rope_blocks = (int)(((size_t)T * half + 255) / 256);
  const dim3 grid((unsigned)(rope_blocks + (total / v + 255) / 256));
#define MTE_OPEN(TI, TO, V)                                                                                     \
  hipLaunchKernelGGL((k_vision_open<TI, TO, V>), grid, dim3(256), 0, s, (const TI *)pixels, (TO *)out, g, total, \
                     rp, T, half, rope_blocks, rcos, rsin)
  if (in_fmt == FMT_BF16 && out_fmt == FMT_F16) { if (v == 8) MTE_OPEN(bf16, f16, 8); else MTE_OPEN(bf16, f16, 1); }
  else if (in_fmt == FMT_F32 && out_fmt == FMT_F32) { if (v == 8) MTE_OPEN(float, float, 8); else MTE_OPEN(float, float, 1); }
  else return hipErrorInvalidValue;
#undef MTE_OPEN
  return hipGetLastError();
}

// LayerNorm of one row per 256-thread block: y = (x - mean) / sqrt(var + eps)
// * g + b, mean and (biased) variance over the D values, two passes over
// values held in registers (D <= 256 * kLnPer).
constexpr int kLnPer = 16;

template <typename TO>
__global__ __launch_bounds__(256) void k_layernorm(const float *__restrict__ x, const float *__restrict__ g,
                                                   const float *__restrict__ b, TO *__restrict__ y, int D,
                                                   float eps) {
  __shared__ float red[4];
  const float *xr = x + (size_t)blockIdx.x * D;
  float v[kLnPer];
  float s = 0.f;
#pragma unroll
  for (int k = 0; k < kLnPer; ++k) {
    const int c = threadIdx.x + 256 * k;
    v[k] = c < D ? xr[c] : 0.f;
    s += v[k];
  }
  auto block_sum = [&](float t) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) t = warp_sum_xor(t, m);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
  };
  const float mean = block_sum(s) / (float)D;
  float q = 0.f;
#pragma unroll
  for (int k = 0; k < kLnPer; ++k) {
    const int c = threadIdx.x + 256 * k;
    const float d = c < D ? v[k] - mean : 0.f;
    q += d * d;
  }
  const float rs = rsqrtf(block_sum(q) / (float)D + eps);
  TO *yr = y + (size_t)blockIdx.x * D;
#pragma unroll
  for (int k = 0; k < kLnPer; ++k) {
    const int c = threadIdx.x + 256 * k;
    if (c < D) yr[c] = from_f32<TO>((v[k] - mean) * rs * g[c] + b[c]);
  }
}

// The same with one wave per row (four rows per block) for D a multiple of
// 256: each lane holds NV 16-byte groups of the row (coalesced loads), and
// both reductions stay inside the wave.
template <typename TO, int NV>
__global__ __launch_bounds__(256) void k_layernorm_wave(const float *__restrict__ x, const float *__restrict__ g,
                                                        const float *__restrict__ b, TO *__restrict__ y, int rows,
                                                        int D, float eps) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const float *xr = x + (size_t)row * D;
  f32x4 v[NV];
  float s = 0.f;
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = *(const f32x4 *)(xr + 4 * (lane + 64 * k));
  // up to 1024 values the gains and biases are loaded with the row (one memory
  // latency for all); wider rows have no registers to spare for them
  f32x4 gg[NV], bb[NV];
  if constexpr (NV <= 4) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      gg[k] = *(const f32x4 *)(g + 4 * (lane + 64 * k));
      bb[k] = *(const f32x4 *)(b + 4 * (lane + 64 * k));
    }
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) s += (v[k][0] + v[k][1]) + (v[k][2] + v[k][3]);
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) s = warp_sum_xor(s, m);
  const float mean = s / (float)D;
  float q = 0.f;
#pragma unroll
  for (int k = 0; k < NV; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float d = v[k][e] - mean;
      q += d * d;
    }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) q = warp_sum_xor(q, m);
  const float rs = rsqrtf(q / (float)D + eps);
  TO *yr = y + (size_t)row * D;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int c = 4 * (lane + 64 * k);
    if constexpr (NV > 4) {
      gg[k] = *(const f32x4 *)(g + c);
      bb[k] = *(const f32x4 *)(b + c);
    }
    typedef TO vo __attribute__((ext_vector_type(4)));
    vo y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = from_f32<TO>((v[k][e] - mean) * rs * gg[k][e] + bb[k][e]);
    *(vo *)(yr + c) = y;
  }
}

template <typename TO>
static bool layernorm_wave(const float *x, const float *g, const float *b, TO *y, int rows, int D, float eps,
                           hipStream_t s) {
  const dim3 grid((rows + 3) / 4);
  switch (D / 256) {
#define MTE_LN(nv) case nv: hipLaunchKernelGGL((k_layernorm_wave<TO, nv>), grid, dim3(256), 0, s, x, g, b, y, rows, D, eps); return true;
    MTE_LN(1) MTE_LN(2) MTE_LN(3) MTE_LN(4) MTE_LN(6) MTE_LN(8) MTE_LN(12) MTE_LN(16)
#undef MTE_LN
  }
  return false;
}

hipError_t launch_layernorm(const float *x, const float *g, const float *b, int out_fmt, void *y, int rows, int D,
                            float eps, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (D > 256 * kLnPer) return hipErrorInvalidValue;
  if (D % 256 == 0 && ((uintptr_t)x | (uintptr_t)g | (uintptr_t)b) % 16 == 0) {
    const bool ok = out_fmt == FMT_F16 ? layernorm_wave(x, g, b, (f16 *)y, rows, D, eps, s)
                    : out_fmt == FMT_F32 ? layernorm_wave(x, g, b, (float *)y, rows, D, eps, s)
                                         : false;
    if (ok) return hipGetLastError();
  }
  if (out_fmt == FMT_F16)
    hipLaunchKernelGGL(k_layernorm<f16>, dim3(rows), dim3(256), 0, s, x, g, b, (f16 *)y, D, eps);
  else if (out_fmt == FMT_F32)
    hipLaunchKernelGGL(k_layernorm<float>, dim3(rows), dim3(256), 0, s, x, g, b, (float *)y, D, eps);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// dst row (r / group) * group_stride + r % group = src row r (float src,
// dst FMT_F32 or FMT_BF16 rounded to nearest even); other dst rows untouched.
template <typename TD>
__global__ __launch_bounds__(256) void k_scatter_rows(const float *__restrict__ src, TD *__restrict__ dst, int cols,
                                                      int group, int group_stride) {
  const int r = blockIdx.x;
  const size_t dr = (size_t)(r / group) * group_stride + r % group;
  const float *sr = src + (size_t)r * cols;
  TD *d = dst + dr * cols;
  for (int c = threadIdx.x; c < cols; c += 256) d[c] = from_f32<TD>(sr[c]);
}

hipError_t launch_scatter_rows(const float *src, int dst_fmt, void *dst, int rows, int cols, int group,
                               int group_stride, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (group <= 0 || group_stride < group) return hipErrorInvalidValue;
  if (dst_fmt == FMT_F32)
    hipLaunchKernelGGL(k_scatter_rows<float>, dim3(rows), dim3(256), 0, s, src, (float *)dst, cols, group,
                       group_stride);
  else if (dst_fmt == FMT_BF16)
    hipLaunchKernelGGL(k_scatter_rows<bf16>, dim3(rows), dim3(256), 0, s, src, (bf16 *)dst, cols, group,
                       group_stride);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mte
