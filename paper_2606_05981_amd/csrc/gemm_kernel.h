// Projection GEMMs of the decoder layer on gfx950 matrix cores.
//
// C = A[M, K] * W[N, K]^T, A = activations (row-major, K contiguous),
// W = weights in blocks of 16 rows x one K stage (see packed_at where they are
// written), so that a workgroup streams whole blocks.
//
// Precision modes:
//  MODE_F32: A and W fp32, v_mfma_f32_16x16x4_f32.
//  MODE_F16: A and W fp16, v_mfma_f32_16x16x32_f16, fp32 accumulation. The
//   weights are bf16 values held as fp16 times a power of two chosen per
//   matrix so that its largest magnitude lands in [2^14, 2^15): every bf16
//   value down to 2^-31 of that maximum converts exactly. Activations are
//   rounded once to fp16 (an 11-bit significand, against bf16's 8) after a
//   power-of-two pre-scale that a static bound keeps in fp16 range; the
//   epilogue multiplies the product by the inverse of both scales (`scale`,
//   exact). One MFMA per fragment at the same dense rate as bf16.
//  MODE_F8W: A fp16 as in MODE_F16; W OCP e4m3 codes (one byte per weight)
//   with one power-of-two scale per output row (`cs`). The codes are staged
//   through LDS at half the bytes of fp16 and widened to fp16 after the LDS
//   read (exact: every e4m3 value is an fp16 value), in the k-step that uses
//   them; the accumulators are multiplied by their column's scale before the
//   epilogue.
//
// Why 16x16x32 and not 32x32x16 (the same dense rate on paper): under random
// operands these GEMMs run at the card's power limit, and per flop the 16x16
// form moves a quarter of the accumulator and twice the operand values
// through the register file. Measured with no memory traffic (eight waves a
// CU, random fp16 operands): 1.86 PFLOP/s with 16x16x32 against 1.69 with
// 32x32x16 (2.37 and 2.42 on zeros, where power does not limit).
//
// Each workgroup (4, 6 or 8 waves, WM x WN) owns a BM x BN output tile; each
// wave a (BM/WM) x (BN/WN) block of 16x16 MFMA tiles. Eight waves, or two
// four-wave workgroups per CU, put two waves on every SIMD, so one wave's
// LDS reads and waits overlap the other's MFMAs. K is walked in stages of
// 128 bytes per row, staged through a ring of 2-8 LDS slots (one barrier
// per stage): the loads of the next P stages are in flight while the current
// one feeds the MFMAs. The deep rings serve small M (one frame), where a
// workgroup's whole K range is a handful of stages: all of them are then in
// flight at once and the kernel waits for memory once, not once per stage.
//
// LDS rows are 128 bytes = 8 chunks of 16 bytes; chunk c of row r is stored
// at slot c ^ (r >> 1 & 7): fragment reads are free of bank conflicts (see swz),
// and since the slot depends on r % 16 only, every fragment of a wave is one lane
// address plus a constant.
//
// Epilogues are fused: fp32 store with the per-head QK-norm and rotary
// embedding of the q and k heads (QKV projection; a wave's columns cover
// whole heads, so a head's sum of squares is a reduction over the wave's
// lanes and both members of each rotary pair sit in one lane), SwiGLU over
// gate/up rows interleaved in blocks of 16 (MLP up-projection: two adjacent
// 16-column tiles hold 16 gate and the 16 matching up columns of the same
// lanes; written in the activation format) and accumulation into
// the fp32 residual stream (attention output projection and MLP
// down-projection). With K split over workgroups (small M), each
// split stores its partial sum instead, and the kernel that consumes the
// product adds the partials up in split order, so results do not depend on
// the order in which workgroups finish.
#pragma once

#include <cmath>
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace mte {

constexpr int kStageBytes = 128;   // bytes of K per row and stage

struct GemmArgs {
  const char *A;
  const char *W;
  void *C;            // EPI_STORE / EPI_RESID / EPI_PARTIAL: float; EPI_SWIGLU / EPI_GELU: activation format
  size_t c_plane;     // EPI_PARTIAL: elements between the partial sums of two K splits
  int M, N, K, ldc;
  int k_chunk;        // K range of one split (gridDim.z splits)
  float scale;        // product multiplier (inverse operand pre-scales)
  float out_scale;    // EPI_SWIGLU / EPI_GELU output multiplier
  QkvEpi qe;          // EPI_QKV
  const float *cs;    // MODE_F8W: per-column (weight row) scales [N]
  const float *bias;  // [N] added to the product before the epilogue (unsplit launches), or null
  const float *resid; // EPI_RESID: the residual stream that is read, C's shape and pitch (C itself, or rows that C takes over)
  // Order of the tiles: gm x gn tiles (M x N) per K split, in groups of gh M
  // tiles, a group column by column. Workgroup i of a launch runs on XCD i % 8;
  // XCD x takes the x-th contiguous eighth of that sequence, so the tiles it has
  // in flight are a block of the product and share rows of A and of W in its L2.
  int gm, gn, gh;
};

// Chunk swizzles for rows of 128 bytes (8 chunks) and 64 bytes (4 chunks),
// functions of r % 16. A fragment read takes 16 rows at two logical chunks c and
// c + 1 per half-wave, and the LDS serves a 16-byte read in groups of 16 lanes
// that are not consecutive: lanes 0-3, 12-15 and 20-27 of a half together, then
// the rest, i.e. rows 0-3 and 12-15 of one chunk with rows 4-11 of the other. With
// r >> 1 those 16 pieces lie in 16 distinct bank groups (SQ_LDS_BANK_CONFLICT 0);
// r ^ (r >> 3 & 1) keeps 16 consecutive rows of one chunk apart and is 2-way
// conflicted on this pattern (8 cycles a read instead of 4).
template <int CH>
__device__ __forceinline__ int swz(int r, int c) {
  if constexpr (CH == 8) return c ^ ((r >> 1) & 7);
  else return c ^ ((r >> 2) & 3);
}

// Eight OCP e4m3 codes (k order, byte 0 first) -> eight fp16 values, exact
// (v_cvt_scalef32_pk_f16_fp8 with scale 1: e4m3's range [2^-9, 448] and its
// 3-bit significand fit fp16).
__device__ __forceinline__ f16x8 widen_e4m3(u32x2 w) {
  typedef _Float16 h2 __attribute__((ext_vector_type(2)));
  const h2 a = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8((int)w[0], 1.f, false);
  const h2 b = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8((int)w[0], 1.f, true);
  const h2 c = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8((int)w[1], 1.f, false);
  const h2 d = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8((int)w[1], 1.f, true);
  return f16x8{a[0], a[1], b[0], b[1], c[0], c[1], d[0], d[1]};
}

// x + the same value of lane (l + n) mod 16 in its 16-lane row (DPP row_ror:n).
template <int n>
__device__ __forceinline__ float add_row_ror(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + n, 0xf, 0xf, false));
}
// Sum of x over the lane's 16-lane row, in every lane of it.
__device__ __forceinline__ float sum_row16(float x) {
  x = add_row_ror<8>(x);
  x = add_row_ror<4>(x);
  x = add_row_ror<2>(x);
  return add_row_ror<1>(x);
}

// Column of block j of a wave's QKV tile, from the wave's first: 16 j, or with
// HALF (a wave owns half of a 128-wide head) 16 j and 32 more from the third
// block on, so that the two waves of a head hold its columns 0..31, 64..95 and
// 32..63, 96..127 and both members of every rotary pair (c, c + 64) sit in one
// lane of one wave.
template <bool HALF>
__device__ __forceinline__ constexpr int qkv_col(int j) { return 16 * j + (HALF && j >= 2 ? 32 : 0); }

// EPI_QKV epilogue of one wave: rows mw.. (TM blocks of 16), columns cw +
// qkv_col(j) (TN blocks of 16 = whole heads of HD columns, or HALF of one), mw
// and cw wave-uniform. Lane
// l holds column l % 16 of every block and rows 4 (l / 16) + 0..3. For each
// row and q or k head: RMS-normalise (sum of squares over the wave's blocks of
// the head and the 16 lanes that hold the row; with HALF the two waves of a
// head add their sums through `xs`, LDS that no copy or read uses any more, one
// slot of 16 TM rows per wave) and rotate pair
// (c, c + HD/2), i.e. column blocks (jb, jb + HJB/2) of one lane. Gains are
// read once; the rotary table values of a block of 16 rows are read before
// they are used. bs[j]: bias / scale of the lane's column. With q.qk the result goes out in the fp16 attention operand
// layout.
template <int HD, bool HALF, int TM, int TN>
__device__ __forceinline__ void qkv_epilogue(const f32x4 (&acc)[TM][TN], const f32x4 (&bs)[TN],
                                             const GemmArgs &g, int cw, int mw, int lane, float *xs, int wave) {
  constexpr int HJB = HALF ? TN : HD / 16;        // column blocks per head in the wave
  constexpr int NH = TN / HJB;                    // heads of the wave
  static_assert(TN % HJB == 0 && (!HALF || (HD == 128 && TN == 4)), "whole heads or one half per wave");
  const QkvEpi &q = g.qe;
  const int lc = lane & 15, rg = lane >> 4;
  const int M = g.M;
  float *C = (float *)g.C;
  bool rot[NH], anyrot = false;
  float gsc[TN];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int cb = cw + h * HD;
    rot[h] = cb < q.rot_cols;                     // wave-uniform
    anyrot |= rot[h];
    const float *gn = cb < q.nq_cols ? q.qn : q.kn;
#pragma unroll
    for (int jj = 0; jj < HJB; ++jj) gsc[h * HJB + jj] = (rot[h] && gn) ? gn[(cb + qkv_col<HALF>(jj)) % HD + lc] : 1.f;
  }
  const int pc = HALF ? cw % HD : 0;              // the wave's first rotary pair
  if constexpr (HALF) {
    if (q.qn) {                                   // workgroup-uniform
      __syncthreads();                            // every wave's copies have landed
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        f32x4 ss = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const float v = (acc[i][j][r] + bs[j][0]) * g.scale;
            ss[r] += v * v;
          }
          ss[r] = sum_row16(ss[r]);
        }
        if (lc == 0) *(f32x4 *)(xs + (wave * TM + i) * 16 + 4 * rg) = ss;
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int mb = mw + i * 16;
    // the rotary entries of a row depend on the pair index only: one set of
    // HJB / 2 blocks serves every head of the wave
    float tc[4][HJB / 2], ts[4][HJB / 2];
    if (anyrot) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const size_t rb = (size_t)min(mb + 4 * rg + r, M - 1) * (HD / 2) + pc + lc;
#pragma unroll
        for (int jj = 0; jj < HJB / 2; ++jj) {
          tc[r][jj] = q.rcos[rb + jj * 16];
          ts[r][jj] = q.rsin[rb + jj * 16];
        }
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int jj = 0; jj < HJB / 2; ++jj) {
          tc[r][jj] = 1.f;
          ts[r][jj] = 0.f;
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = mb + 4 * rg + r;
      float v[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) v[j] = (acc[i][j][r] + bs[j][0]) * g.scale;
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        if (!rot[h]) continue;
        if (q.qn) {
          float ss = 0.f;
          if constexpr (HALF) {
            ss = xs[(wave * TM + i) * 16 + 4 * rg + r] + xs[((wave ^ 1) * TM + i) * 16 + 4 * rg + r];
          } else {
#pragma unroll
            for (int jj = 0; jj < HJB; ++jj) ss += v[h * HJB + jj] * v[h * HJB + jj];
            ss = sum_row16(ss);
          }
          const float rs = rsqrtf(ss / (float)HD + q.eps);
#pragma unroll
          for (int jj = 0; jj < HJB; ++jj) v[h * HJB + jj] = v[h * HJB + jj] * rs * gsc[h * HJB + jj];
        }
#pragma unroll
        for (int jj = 0; jj < HJB / 2; ++jj) {
          const int j = h * HJB + jj, jp = j + HJB / 2;
          const float u = v[j], w = v[jp];
          v[j] = u * tc[r][jj] - w * ts[r][jj];
          v[jp] = w * tc[r][jj] + u * ts[r][jj];
        }
      }
      if (q.qk) {
        // attention operand layout: q and k heads as fp16 rows (v below)
        if (m < M) {
          f16 *qr = q.qk + (size_t)m * q.rot_cols + cw + lc;
#pragma unroll
          for (int h = 0; h < NH; ++h) {
            if (!rot[h]) continue;
            const float pre = cw + h * HD < q.nq_cols ? q.q_pre : q.k_pre;
#pragma unroll
            for (int jj = 0; jj < HJB; ++jj) qr[qkv_col<HALF>(h * HJB + jj)] = (f16)(v[h * HJB + jj] * pre);
          }
        }
      } else if (m < M) {
        float *p = C + (size_t)m * g.ldc + cw + lc;
#pragma unroll
        for (int j = 0; j < TN; ++j) p[qkv_col<HALF>(j)] = v[j];
      }
    }
    if (q.qk && (mb & ~31) < M) {
      // v heads as V^T tiles: a lane's four rows of its column are four
      // consecutive values of the tile's fragment order (row 16 b + 4 g + r at
      // position 16 b + 8 (g % 2) + 4 (g / 2) + r). Rows past M are written as
      // zeros, also a whole block of them where its 32-token tile has live rows;
      // tiles wholly past M are not part of the batch.
      const float sv = g.scale * q.v_pre;
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        if (rot[h]) continue;
#pragma unroll
        for (int jj = 0; jj < HJB; ++jj) {
          const int j = h * HJB + jj;
          const int dv = cw + qkv_col<HALF>(j) + lc - q.rot_cols;
          f16 *dst = q.vt + (((size_t)(mb >> 5) * q.hkv + dv / HD) * HD + dv % HD) * 32 + (mb & 16) +
                     8 * (rg & 1) + 4 * (rg >> 1);
          f16x4 y;
#pragma unroll
          for (int r = 0; r < 4; ++r) y[r] = (f16)(mb + 4 * rg + r < M ? (acc[i][j][r] + bs[j][0]) * sv : 0.f);
          *(f16x4 *)dst = y;
        }
      }
    }
  }
}

// The main loop keeps P stages in an LDS ring filled by direct global->LDS
// loads. Per k-step (64 bytes of K per row) a wave runs X rows of Y MFMAs: the
// fragments of the longer side of its tile (X of them) are each used by one
// row and then replaced by the next k-step's, those of the shorter side (Y)
// are used by every row and double-buffered; that costs X + 2 Y fragments of
// registers instead of 2 (X + Y). One
// barrier per stage, placed after the first row of the stage's last k-step:
// before it each wave waits for its own loads of the next stage and for its
// own LDS reads (the last k-step's fragments are already in registers).
// After it, all waves' loads of stage kt+1 are in LDS and no wave reads slot
// kt % P again, so the loads of stage kt+P go into that slot, and the first
// fragments of stage kt+1 are read while the last MFMAs of stage kt run.
// Raw s_barrier (no fence) keeps the compiler from forcing vmcnt(0) at the
// barrier; the waits are explicit.
template <int MODE, int BM, int BN, int WM, int WN, int P, int EPI, int OCC>
__global__ __launch_bounds__(64 * WM * WN, OCC) __attribute__((amdgpu_waves_per_eu((OCC * WM * WN + 3) / 4, (OCC * WM * WN + 3) / 4))) void k_gemm(GemmArgs g) {
  typedef typename std::conditional<MODE == MODE_F32, float, f16>::type T;
  constexpr bool W8 = MODE == MODE_F8W;           // one-byte weights
  constexpr int ROWB = kStageBytes;
  constexpr int KS = ROWB / (int)sizeof(T);       // k elements per stage
  constexpr int CH = ROWB / 16;                   // 16-byte chunks per A row per stage
  constexpr int CHW = W8 ? CH / 2 : CH;           // 16-byte chunks per W row per stage
  constexpr int WTM = BM / WM, WTN = BN / WN;     // wave tile
  constexpr int TM = WTM / 16, TN = WTN / 16;     // 16x16 MFMA tiles per wave
  constexpr int ACH = BM * CH, BCH = BN * CHW;    // chunks per stage (A / W)
  constexpr int NW = WM * WN;                     // waves per workgroup
  constexpr int NT = 64 * NW;                     // threads per workgroup
  // DMA rounds: each wave instruction fills one group of 64 chunks. A last,
  // partial round repeats the matrix's final group in the waves past it
  // (the same bytes to the same LDS slots), so every wave issues the same
  // number of loads and the vmcnt waits stay exact.
  static_assert(ACH % 64 == 0 && BCH % 64 == 0, "whole 64-chunk groups");
  constexpr int AG = ACH / 64, BG = BCH / 64;     // chunk groups per stage
  constexpr int AR = (AG + NW - 1) / NW, BR = (BG + NW - 1) / NW;   // DMA instructions per thread
  constexpr int LOADS = AR + BR;                  // per thread per stage
  constexpr int STAGE = ACH + BCH;                // u32x4 slots per stage
  static_assert(NW == 4 || NW == 6 || NW == 8, "4, 6 or 8 waves");
  static_assert(BM % 32 == 0 && WTM % 16 == 0 && WTN % 16 == 0, "wave tile");
  static_assert(EPI != EPI_SWIGLU || WTN % 32 == 0, "gate/up pairs within a wave");
  static_assert(LOADS * (P - 1) < 64 && P >= 2 && P <= 16, "vmcnt range, ring depth");
  typedef typename Frag<T>::type frag_t;

  extern __shared__ u32x4 lds[];                  // [P][STAGE]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  int tn, tm, tz;
  {
    // XCD of this workgroup and its index among that XCD's workgroups -> its
    // place t in the tile sequence (XCDs below the remainder take one more)
    const int total = gridDim.x, xcd = blockIdx.x & 7, plane = g.gm * g.gn;
    const int t = xcd * (total >> 3) + min(xcd, total & 7) + ((int)blockIdx.x >> 3);
    tz = t / plane;
    const int u = t - tz * plane, grp = u / (g.gh * g.gn), m1 = grp * g.gh;
    const int h = min(g.gh, g.gm - m1), v = u - m1 * g.gn;
    tn = v / h;
    tm = m1 + v - tn * h;
  }
  const int n0 = tn * BN, m0 = tm * BM;
  const int M = g.M;
  const size_t rowb = (size_t)g.K * sizeof(T);    // row pitch in bytes (A; W unless W8)
  const size_t kb0 = (size_t)tz * g.k_chunk * sizeof(T);
  const size_t rowbw = W8 ? (size_t)g.K : rowb;
  constexpr int SBW = W8 ? ROWB / 2 : ROWB;       // bytes of a W row per stage
  const size_t kb0w = (W8 ? (size_t)tz * g.k_chunk : kb0) * 16;
  const int nk = g.k_chunk / KS;

  // DMA sources: instruction c of this thread fills LDS slot q = (c*NW + wave)*64 + lane
  // of its matrix (row q / CH, swizzled slot q % CH, logical chunk slot ^ f(row)).
  // As 32-bit byte offsets from g.A and g.W (the host keeps both matrices
  // under 4 GiB). The W rows of DMA instruction c are instruction 0's plus
  // c * BROWS when every round is whole and the step keeps the chunk swizzle
  // (a multiple of 16 rows): one offset and a uniform stride then replace BR
  // of them (registers the larger tiles need for their fragments).
  constexpr int BROWS = NW * 64 / CHW;
  constexpr bool BSTRIDE = BG % NW == 0 && BROWS % 16 == 0;
  uint32_t pa[AR], pb[BSTRIDE ? 1 : BR];
  const size_t bstep = (size_t)BROWS * rowbw;
#pragma unroll
  for (int c = 0; c < AR; ++c) {
    const int q = min(c * NW + wave, AG - 1) * 64 + lane, r = q / CH, ch = swz<CH>(r, q % CH);
    pa[c] = (uint32_t)((size_t)min(m0 + r, M - 1) * rowb + ch * 16);
  }
#pragma unroll
  for (int c = 0; c < (BSTRIDE ? 1 : BR); ++c) {
    const int q = min(c * NW + wave, BG - 1) * 64 + lane, r = q / CHW, ch = swz<CHW>(r, q % CHW);
    pb[c] = (uint32_t)((size_t)((n0 + r) & ~15) * rowbw + (r & 15) * SBW + ch * 16);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  const int uwave = __builtin_amdgcn_readfirstlane(wave);   // wave-uniform in an SGPR
  // DMA load x (0 <= x < LOADS) of K-stage `ks` into ring slot `slot`.
  auto dma_one = [&](int ks, int slot, int x) {
    const uint32_t st = lds0 + (uint32_t)(slot * STAGE) * 16u;
    const size_t ko = (size_t)ks * ROWB;
    if (x < AR) {
      dma16(g.A + kb0 + ko, pa[x], st + (uint32_t)(min(x * NW + uwave, AG - 1) * 64) * 16u);
    } else {
      const int c = x - AR;
      const char *wb = g.W + kb0w + (size_t)ks * (16 * SBW);
      if constexpr (BSTRIDE) dma16(wb + c * bstep, pb[0], st + (uint32_t)(ACH + min(c * NW + uwave, BG - 1) * 64) * 16u);
      else dma16(wb, pb[c], st + (uint32_t)(ACH + min(c * NW + uwave, BG - 1) * 64) * 16u);
    }
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // fp32 operands: the products of one stage (32 of K) are summed by themselves in
  // `part` and then added to acc, so that a sum over K rounds K / 32 times at its
  // full size, not K / 4 times (two 256-wide layers against float64, mean over 12
  // inputs, same tiles and splits: 32 tokens 3.6e-7 against 4.7e-7 with one chain, 2 x
  // 128 tokens 4.1e-7 against 5.7e-7, 8 x 320 tokens 4.4e-7 against 8.8e-7). Adding a
  // tile's sum while later tiles' MFMAs run was slower (128x128 tile of four waves, 64
  // stages: 142 us against 135).
  constexpr bool STAGED = MODE == MODE_F32;
  f32x4 part[STAGED ? TM : 1][STAGED ? TN : 1];
  if constexpr (STAGED) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) part[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  constexpr int KK = CH / 4;                      // k-steps per stage
  static_assert(KK == 2, "fragment buffer parity");
  constexpr bool RA = TM >= TN;                   // rows of MFMAs run over the A fragments
  constexpr int X = RA ? TM : TN, Y = RA ? TN : TM;
  constexpr int NM = TM * TN;                     // MFMAs per k-step
  constexpr int NR = TM + TN;                     // fragment reads per k-step
  // the side with X fragments uses buffer 0 only
  frag_t fa[2][TM], fb[2][TN];
  // W8: the raw codes of a W fragment (8 bytes per lane) are read into fw; the
  // first MFMA of a k-step that uses them widens them into fb[0].
  typedef typename std::conditional<W8, u32x2, char>::type wraw_t;
  wraw_t fw[2][TN];
  const int lc = lane & 15, rg = lane >> 4;
  // Byte offsets of the lane's fragment of tile 0 within a stage, per k-step;
  // tile t is 16 rows further (the swizzle repeats every 16 rows). A lane takes
  // 16 bytes of K: chunk 4 kk + l / 16 of its row (W8: 8 of them, half a chunk).
  // QKV tiles with 64 columns a wave: half a head of 128 (see qkv_col), or one of 64
  constexpr bool MAYHALF = EPI == EPI_QKV && WTN == 64 && WN % 2 == 0;
  const bool half = MAYHALF && g.qe.hd == 128;    // launch-uniform
  auto wave_col = [&](int n) { return half ? (n >> 1) * 128 + (n & 1) * 32 : n * WTN; };   // first column of wave column n
  uint32_t oa[KK], ow[KK], ow2[KK];               // ow2: tiles from TN / 2 on
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    oa[kk] = (uint32_t)((wm * WTM + lc) * CH + swz<CH>(lc, 4 * kk + rg)) * 16u;
    const int wr = wave_col(wn) + lc;
    if constexpr (W8) ow[kk] = (uint32_t)ACH * 16u + (uint32_t)(wr * CHW + swz<CHW>(lc, 2 * kk + (rg >> 1))) * 16u + (rg & 1) * 8u;
    else ow[kk] = (uint32_t)ACH * 16u + (uint32_t)(wr * CH + swz<CH>(lc, 4 * kk + rg)) * 16u;
    ow2[kk] = ow[kk] + (half ? 32u * CHW * 16u : 0u);
  }
  const char *ldsb = (const char *)lds;
  // Fragment t of A / W of k-step kk of the ring slot at byte offset `st`
  auto read_a = [&](uint32_t st, int kk, int b, int t) {
    fa[b][t] = *(const frag_t *)(ldsb + (st + oa[kk]) + t * 16 * CH * 16);
  };
  auto read_w = [&](uint32_t st, int kk, int b, int t) {
    const uint32_t o = st + (MAYHALF && t >= TN / 2 ? ow2[kk] : ow[kk]);
    if constexpr (W8) fw[b][t] = *(const u32x2 *)(ldsb + o + t * 16 * CHW * 16);
    else fb[b][t] = *(const frag_t *)(ldsb + o + t * 16 * CH * 16);
  };
  // Fragment o of the X side (buffer 0) / y of the Y side (buffer b)
  auto read_x = [&](uint32_t st, int kk, int o) { if constexpr (RA) read_a(st, kk, 0, o); else read_w(st, kk, 0, o); };
  auto read_y = [&](uint32_t st, int kk, int b, int y) { if constexpr (RA) read_w(st, kk, b, y); else read_a(st, kk, b, y); };
  // EPI_QKV wants a lane to hold one column (V^T rows, QK-norm over 16 lanes);
  // the others form the transposed tile, so that a lane holds four consecutive
  // columns of one row and stores them at once.
  constexpr bool TRANS = EPI != EPI_QKV;
  auto mfma_one = [&](int cur, int m) {
    const int o = m / Y, y = m % Y;
    const int i = RA ? o : y, j = RA ? y : o;
    const int ba = RA ? 0 : cur, bw = (RA && !W8) ? cur : 0;
    if constexpr (W8) {
      if (RA ? o == 0 : y == 0) fb[0][j] = widen_e4m3(fw[RA ? cur : 0][j]);
    }
    f32x4 *c = &acc[i][j];
    if constexpr (STAGED) c = &part[i][j];
    if constexpr (TRANS) mfma16(*c, fb[bw][j], fa[ba][i]);
    else mfma16(*c, fa[ba][i], fb[bw][j]);
  };
  // The loads of stage kt+P are issued in NPART parts: part 0 right after the
  // barrier of stage kt, parts 1.. in the k-steps of stage kt+1 before its
  // barrier. With P >= 3 every stage still has P-2 whole stages of loads in
  // flight behind it at the barrier that waits for it; P = 2 issues each
  // stage whole, after the barrier.
  constexpr int NPART = (P >= 3) ? KK : 1;
  constexpr int PART = (LOADS + NPART - 1) / NPART;

  // One k-step: the NM MFMAs on Y-side buffer `cur`, with the side work spread
  // between them in issue order -- the next k-step's fragments (k-step rkk of
  // the slot at rst; an X fragment as soon as its row is done, the Y fragments,
  // which the next k-step needs first, over the first half) and DMA loads
  // [d0, d1) of stage ks into slot `slot`. With `bar`, the barrier of the stage
  // (after this wave's loads of the next stage have landed) goes after the
  // first row, ahead of all side work.
  // Each unit of side work is pinned behind its MFMA by a scheduling
  // barrier, so the matrix core keeps busy while it issues.
  auto kstep = [&](int cur, uint32_t rst, int rkk, int ks, int slot, int d0, int d1, bool bar) {
    const int b0 = bar ? Y - 1 : 0;              // first MFMA with side work behind it
    const int nd = d1 - d0;
    // units of side work before MFMA m, of n spread over MFMAs [b0, b0 + w)
    auto upto = [&](int m, int n, int w) { return m <= b0 ? 0 : m >= b0 + w ? n : ((m - b0) * n + w - 1) / w; };
    const int wy = (NM - b0 + 1) / 2, wd = NM - b0;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      mfma_one(cur, m);
      if (bar && m == b0) {
        wait_vm_lds0<(P - 2) * LOADS>();   // this wave's loads of the next stage landed, its reads done
        __builtin_amdgcn_s_barrier();      // ... everyone's: slot kt % P is free
        asm volatile("" ::: "memory");     // keep LDS reads of the next stage below it
      }
#pragma unroll
      for (int y = upto(m, Y, wy); y < upto(m + 1, Y, wy); ++y) read_y(rst, rkk, cur ^ 1, y);
      if (m % Y == Y - 1) read_x(rst, rkk, m / Y);
#pragma unroll
      for (int d = upto(m, nd, wd); d < upto(m + 1, nd, wd); ++d) dma_one(ks, slot, d0 + d);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // The loop body is branch-free (a branch between LDS reads and their
  // use makes the waitcnt pass drain all outstanding reads): every iteration
  // issues its loads -- past the end, repeats of the last stage into slots
  // that are never read again -- so every wait is a fixed vmcnt.
  // Prologue: stages 0..P-2 whole and part 0 of stage P-1 (P = 2: stages
  // 0..P-1 whole), then stage 0 must have landed.
  constexpr int PRE_FULL = (NPART > 1) ? P - 1 : P;
  constexpr int PRE_PART = (NPART > 1) ? (PART < LOADS ? PART : LOADS) : 0;
#pragma unroll
  for (int s = 0; s < PRE_FULL; ++s)
#pragma unroll
    for (int x = 0; x < LOADS; ++x) dma_one(min(s, nk - 1), s, x);
#pragma unroll
  for (int x = 0; x < PRE_PART; ++x) dma_one(min(P - 1, nk - 1), P - 1, x);
  wait_vm<(PRE_FULL - 1) * LOADS + PRE_PART>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int y = 0; y < Y; ++y) read_y(0, 0, 0, y);
#pragma unroll
  for (int o = 0; o < X; ++o) read_x(0, 0, o);
  for (int kt = 0; kt < nk; ++kt) {
    const uint32_t st = (uint32_t)((kt % P) * STAGE) * 16u;
    const uint32_t nx = (uint32_t)(((kt + 1) % P) * STAGE) * 16u;
    const int ksa = min(kt + P - 1, nk - 1), sla = (kt + P - 1) % P;   // parts 1.. issued here
    const int ksb = min(kt + P, nk - 1), slb = kt % P;                  // part 0 issued here
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const int cur = kk & 1;
      if (kk + 1 < KK) {
        const int q = kk + 1;                       // DMA part of this k-step
        const int d0 = (NPART > 1) ? min(q * PART, LOADS) : 0;
        const int d1 = (NPART > 1) ? min((q + 1) * PART, LOADS) : 0;
        kstep(cur, st, kk + 1, ksa, sla, d0, d1, false);
      } else {
        const int d1 = (NPART > 1) ? min(PART, LOADS) : LOADS;
        kstep(cur, nx, 0, ksb, slb, 0, d1, true);
      }
    }
    if constexpr (STAGED) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          acc[i][j] += part[i][j];
          part[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
  }
  wait_vm<0>();                          // no load may land after the workgroup ends
  const int uwm = uwave / WN, uwn = uwave % WN;
  const int mw = m0 + uwm * WTM, cw = n0 + wave_col(uwn);   // wave-uniform
  // The lane's column(s) of column block j: cw + 16 j + lc (QKV halves: see
  // qkv_col), or (TRANS) the four from cw + 16 j + 4 rg.
  const int cl = cw + (TRANS ? 4 * rg : lc);
  auto col = [&](int j) { return cl + (MAYHALF && half ? qkv_col<true>(j) : 16 * j); };
  if constexpr (W8) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      f32x4 c;
      if constexpr (TRANS) c = *(const f32x4 *)(g.cs + col(j));
      else { const float c1 = g.cs[col(j)]; c = f32x4{c1, c1, c1, c1}; }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] *= c[r];
    }
  }
  // bias / scale added to the accumulators (zero without a bias): `scale` is a
  // power of two, so (acc + bias / scale) * scale rounds exactly like
  // acc * scale + bias. Selected values and not a branch around the adds: a
  // branch here makes the compiler hold a second copy of the accumulators.
  f32x4 bs[TN];
  if constexpr (EPI != EPI_SWIGLU && EPI != EPI_PARTIAL) {
#pragma unroll
    for (int j = 0; j < TN; ++j) bs[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (g.bias) {
      const float ib = 1.f / g.scale;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        if constexpr (TRANS) bs[j] = *(const f32x4 *)(g.bias + col(j)) * ib;
        else { const float b1 = g.bias[col(j)] * ib; bs[j] = f32x4{b1, b1, b1, b1}; }
      }
    }
  }

  if constexpr (EPI == EPI_QKV) {
    // (the host only launches tiles whose waves cover whole heads or halves)
    if (g.qe.hd == 128) {
      if constexpr (TN % 8 == 0) qkv_epilogue<128, false, TM, TN>(acc, bs, g, cw, mw, lane, (float *)lds, uwave);
      else if constexpr (MAYHALF) qkv_epilogue<128, true, TM, TN>(acc, bs, g, cw, mw, lane, (float *)lds, uwave);
    } else {
      if constexpr (TN % 4 == 0) qkv_epilogue<64, false, TM, TN>(acc, bs, g, cw, mw, lane, (float *)lds, uwave);
    }
    return;
  }
  // The other epilogues: lane l holds row mw + 16 i + l % 16 and, per column
  // block j, columns cw + 16 j + 4 (l / 16) + 0..3.
  typedef typename std::conditional<MODE == MODE_F32, f32x4, f16x4>::type out4;   // activation outputs
  typedef typename std::conditional<MODE == MODE_F32, float, f16>::type TO;
  if constexpr (EPI == EPI_SWIGLU) {
    // Column blocks 2b and 2b+1 of the interleaved product hold the gate and
    // up values of outputs f = 16 b + 0..15. With z = scale*g and u = scale*up,
    //   silu(z) * u * out_scale = (g * up) / (1 + 2^(g * (-scale*log2 e))) * (scale^2 * out_scale).
    const float c1 = -g.scale * 1.4426950408889634f;
    const float s2 = g.scale * g.scale * g.out_scale;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = mw + i * 16 + lc;
      if (m >= M) continue;
      TO *p = (TO *)g.C + (size_t)m * g.ldc + (cw >> 1) + 4 * rg;
#pragma unroll
      for (int j = 0; j < TN; j += 2) {
        out4 y;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float ga = acc[i][j][r], up = acc[i][j + 1][r];
          const float e = __builtin_amdgcn_exp2f(ga * c1);
          y[r] = (TO)((ga * up) * __builtin_amdgcn_rcpf(1.f + e) * s2);
        }
        *(out4 *)(p + j * 8) = y;
      }
    }
    return;
  }
  if constexpr (EPI == EPI_GELU) {
    // tanh-approximated GELU: 0.5 z (1 + tanh(u)) with u = sqrt(2/pi) (z + 0.044715 z^3) is
    // z / (1 + exp(-2u)), one exp and one hardware reciprocal instead of a library tanh
    // (large negative z: exp overflows to inf and the result is 0). With z = scale * a,
    //   gelu(z) * out_scale = a / (1 + 2^(c0 a (1 + k2 a^2))) * (scale * out_scale),
    // c0 = -2 sqrt(2/pi) log2(e) scale, k2 = 0.044715 scale^2.
    const float k2 = 0.044715f * g.scale * g.scale;
    const float c0 = -1.5957691216057308f * 1.4426950408889634f * g.scale;
    const float so = g.scale * g.out_scale;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = mw + i * 16 + lc;
      if (m >= M) continue;
      TO *p = (TO *)g.C + (size_t)m * g.ldc + cl;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        out4 y;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float a = acc[i][j][r] + bs[j][r];
          const float e = __builtin_amdgcn_exp2f(a * fmaf(a * a, k2, 1.f) * c0);
          y[r] = (TO)(a * __builtin_amdgcn_rcpf(1.f + e) * so);
        }
        *(out4 *)(p + j * 16) = y;
      }
    }
    return;
  }
  // EPI_STORE / EPI_PARTIAL: C = scale * acc; EPI_RESID: C = resid + scale * acc (one
  // rounding: scale is a power of two), the old values of two 16-row blocks all
  // read before the first store so that their latencies overlap.
  float *C = (float *)g.C + (EPI == EPI_PARTIAL ? (size_t)tz * g.c_plane : 0) + cl;
  constexpr int IB = TM % 2 == 0 ? 2 : 1;
#pragma unroll
  for (int i0 = 0; i0 < TM; i0 += IB) {
    f32x4 old[IB][TN];
    if constexpr (EPI == EPI_RESID) {
#pragma unroll
      for (int i = 0; i < IB; ++i) {
        const float *p = g.resid + cl + (size_t)min(mw + (i0 + i) * 16 + lc, M - 1) * g.ldc;
#pragma unroll
        for (int j = 0; j < TN; ++j) old[i][j] = *(const f32x4u *)(p + j * 16);
      }
    }
#pragma unroll
    for (int i = 0; i < IB; ++i) {
      const int m = mw + (i0 + i) * 16 + lc;
      if (m >= M) continue;
      float *p = C + (size_t)m * g.ldc;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        f32x4 y;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float a = EPI == EPI_PARTIAL ? acc[i0 + i][j][r] : acc[i0 + i][j][r] + bs[j][r];
          y[r] = EPI == EPI_RESID ? fmaf(a, g.scale, old[i][j][r]) : a * g.scale;
        }
        *(f32x4u *)(p + j * 16) = y;
      }
    }
  }
}

// A tile configuration is a compile-time instantiation of k_gemm. stage_us,
// tile_us: its measured costs for the planner, by Mode (fp32, fp16, e4m3 weights).
struct TileCfg {
  int bm, bn, wm, wn, p, occ, f32, w8;
  double stage_us[3], tile_us[3];
};

template <int MODE, int BM, int BN, int WM, int WN, int P, int EPI, int OCC, int F32, int W8>
static hipError_t run(const GemmArgs &a, int splits, hipStream_t s) {
  if constexpr (EPI == EPI_QKV && (BN / WN) % 64 != 0) {
    return hipErrorInvalidValue;  // the QK-norm epilogue needs whole heads per wave
  } else if constexpr (EPI == EPI_SWIGLU && (BN / WN) % 32 != 0) {
    return hipErrorInvalidValue;  // gate/up pairs within a wave
  } else if constexpr (MODE == MODE_F32 && !F32) {
    return hipErrorInvalidValue;  // fp32 operands are built for a few tiles only
  } else if constexpr (MODE == MODE_F8W && (!W8 || EPI == EPI_GELU || EPI == EPI_STORE)) {
    return hipErrorInvalidValue;  // e4m3 weights: not every tile, decoder epilogues
  } else {
    constexpr int lds_bytes = P * (BM + (MODE == MODE_F8W ? BN / 2 : BN)) * kStageBytes;
    auto kern = k_gemm<MODE, BM, BN, WM, WN, P, EPI, OCC>;
    static const hipError_t attr = hipFuncSetAttribute(
        (const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (attr != hipSuccess) return attr;
    const dim3 grid(a.gm * a.gn * splits);
    hipLaunchKernelGGL(kern, grid, dim3(64 * WM * WN), lds_bytes, s, a);
    return hipGetLastError();
  }
}


// Tile table: id -> instantiation (bm, bn, wave layout wm x wn, LDS ring
// stages, workgroups per CU, built for fp32 operands too, built for e4m3
// weights too), then the planner's costs in us of one tile alone on its CU, per
// 128-byte K stage and per tile (prologue, epilogue): fp16 weights, e4m3 weights,
// fp32. The LDS ring (p * (bm + bn) * 128 bytes, bn / 2 for
// e4m3 weights) must fit 160 KB / occ. bm a multiple of 32 (V^T tiles).
// The costs are least-squares fits (relative error) of the planner's model to
// sweeps of every tile on MI355X at 16 ... 10240 rows (fp32: ... 4096); they rank
// tiles and do not predict times. Over the decoder's projections at width 2048,
// at width 1024 and the vision tower's the pick is 0.8%, 1.6% and 0.2% slower than
// the fastest tile on average (e4m3 1.1%, fp32 1.1%), single ones up to 23% (e4m3 29%).
// The model's time of an unsplit launch is 9-17% rms off (e4m3 7-15%, its 32x64
// tile 33%; fp32 4-6%), and low where the epilogue's bytes count, which it has no
// term for: the 10240-row output projection, 101 us, is put at 72. The
// 256x256 tile spills in its loop with e4m3 weights (nine times slower).
// fp32 products are bound by the fp32 MFMAs, a sixteenth of the fp16 rate: a stage
// costs 2-5 times what it does in fp16, and how evenly the rows divide over the chip
// decides. Planned with the fp16 costs, on four-wave tiles of 128x128, 128x64, 64x64
// and 32x64 only, one layer at width 2048 took 522 us at 337 rows and 3333 at 4096;
// on these tiles 358 and 3146.
#define MTE_TILE_TABLE(X) \
  X(0, 256, 256, 4, 2, 2, 1, 0, 0, 1.335, 10.86, 0.000, 0.00, 0.000, 0.00)             \
  X(1, 192, 384, 2, 4, 2, 1, 0, 1, 1.309, 15.45, 1.250, 14.30, 0.000, 0.00)            \
  X(2, 224, 256, 2, 4, 2, 1, 0, 1, 1.216, 10.07, 1.594, 9.60, 0.000, 0.00)             \
  X(3, 160, 256, 2, 4, 3, 1, 0, 1, 0.835, 8.18, 0.891, 7.67, 0.000, 0.00)              \
  X(4, 128, 256, 4, 2, 3, 1, 0, 1, 0.754, 7.23, 0.857, 6.89, 0.000, 0.00)              \
  X(5, 192, 256, 4, 2, 2, 1, 0, 1, 1.119, 8.73, 1.015, 8.91, 0.000, 0.00)              \
  X(6, 192, 128, 4, 2, 4, 1, 1, 1, 0.593, 5.47, 0.635, 5.27, 3.120, 5.47)              \
  X(7, 192, 128, 6, 1, 3, 1, 0, 1, 0.664, 5.86, 0.785, 5.36, 0.000, 0.00)              \
  X(8, 128, 128, 4, 2, 4, 1, 1, 1, 0.461, 4.42, 0.459, 4.25, 2.091, 4.19)              \
  X(9, 128, 128, 4, 1, 4, 1, 0, 1, 0.486, 4.62, 0.577, 4.13, 0.000, 0.00)              \
  X(10, 96, 128, 2, 4, 4, 1, 1, 1, 0.385, 3.82, 0.313, 3.22, 1.588, 2.66)              \
  X(11, 96, 128, 6, 1, 5, 1, 0, 1, 0.452, 4.32, 0.617, 3.91, 0.000, 0.00)              \
  X(12, 96, 64, 2, 2, 8, 1, 1, 1, 0.271, 3.10, 0.276, 2.87, 0.870, 2.49)               \
  X(13, 64, 128, 4, 1, 6, 1, 0, 1, 0.374, 3.63, 0.483, 3.16, 0.000, 0.00)              \
  X(14, 128, 64, 4, 1, 6, 1, 1, 1, 0.326, 3.36, 0.393, 3.13, 1.167, 3.59)              \
  X(15, 32, 128, 2, 2, 8, 1, 1, 1, 0.267, 2.62, 0.296, 2.30, 0.624, 2.74)              \
  X(16, 64, 64, 2, 2, 8, 1, 0, 1, 0.211, 2.29, 0.209, 2.20, 0.000, 0.00)               \
  X(17, 64, 32, 4, 1, 6, 2, 0, 1, 0.191, 1.40, 0.196, 1.40, 0.000, 0.00)               \
  X(18, 32, 64, 2, 2, 6, 2, 1, 1, 0.196, 1.45, 0.190, 1.35, 0.374, 1.15)

template <int MODE, int EPI>
static hipError_t run_id(int id, const GemmArgs &a, int splits, hipStream_t s) {
  switch (id) {
#define MTE_TILE_CASE(idv, bm, bn, wm, wn, p, occ, f32, w8, su, tu, su8, tu8, su32, tu32) \
  case idv: return run<MODE, bm, bn, wm, wn, p, EPI, occ, f32, w8>(a, splits, s);
    MTE_TILE_TABLE(MTE_TILE_CASE)
#undef MTE_TILE_CASE
  }
  return hipErrorInvalidValue;
}

template <int MODE>
static hipError_t launch_mode(int epi, int tile, int splits, const GemmArgs &a, hipStream_t s) {
  switch (epi) {
    case EPI_STORE: return run_id<MODE, EPI_STORE>(tile, a, splits, s);
    case EPI_SWIGLU: return run_id<MODE, EPI_SWIGLU>(tile, a, splits, s);
    case EPI_RESID: return run_id<MODE, EPI_RESID>(tile, a, splits, s);
    case EPI_QKV: return run_id<MODE, EPI_QKV>(tile, a, splits, s);
    case EPI_GELU: return run_id<MODE, EPI_GELU>(tile, a, splits, s);
    default: return run_id<MODE, EPI_PARTIAL>(tile, a, splits, s);
  }
}

}  // namespace mte
