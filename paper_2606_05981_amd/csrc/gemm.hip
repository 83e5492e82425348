// Planning and launch of the projection GEMMs (k_gemm, gemm_kernel.h): a
// tile configuration and K split per (M, N, K, epilogue), from a model of the
// launch's time: rounds of workgroups over the chip times each tile's measured
// costs.
#include "gemm_kernel.h"

namespace mte {

static const TileCfg kTiles[] = {
#define MTE_TILE_INFO(id, bm, bn, wm, wn, p, occ, f32, w8, su, tu, su8, tu8, su32, tu32) \
  {bm, bn, wm, wn, p, occ, f32, w8, {su32, su, su8}, {tu32, tu, tu8}},
    MTE_TILE_TABLE(MTE_TILE_INFO)
#undef MTE_TILE_INFO
};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

// QKV on tile `id` with two waves of 64 columns per 128-wide head.
static bool half_heads(int id, int epi, int col_align) {
  const TileCfg &t = kTiles[id];
  return epi == EPI_QKV && col_align == 128 && t.bn / t.wn == 64 && t.wn % 2 == 0;
}

// Whether tile `id` can run an (N, K, epilogue, splits) product: N a multiple of
// its width, each K split a whole number of stages, fp32 operands only on the
// tiles built for them. col_align: columns a wave must cover in whole units
// (heads for the QKV epilogue, which also takes two waves of 64 columns per
// 128-wide head; 32-column gate/up pairs for SwiGLU).
static bool tile_fits(int id, int N, int K, int esz, int epi, int splits, int col_align, bool w8) {
  const TileCfg &t = kTiles[id];
  if (N % t.bn || (esz == 4 && !t.f32) || (w8 && !t.w8)) return false;
  if (t.p * (t.bm + (w8 ? t.bn / 2 : t.bn)) * kStageBytes * t.occ > 160 * 1024) return false;   // LDS ring
  const int ks = kStageBytes / esz;
  if (K % splits || (K / splits) % ks) return false;
  if ((epi == EPI_QKV || epi == EPI_SWIGLU) && (t.bn / t.wn) % col_align && !half_heads(id, epi, col_align)) return false;
  return true;
}

// How many tile times a launch of `wgs` workgroups takes on 256 CUs. One
// workgroup per CU (occ 1): the whole rounds, and for a last round that fills
// only a fraction f of the chip 0.85 + 0.15 f of one (a part-filled round is
// hardly shorter, but the clock under the power limit is a little higher). Two
// per CU: a CU with both takes 1.5 times as long as with one.
static double tile_rounds(int64_t wgs, int occ) {
  const double f = (double)wgs / 256.0;
  const double full = std::floor(f / occ), rem = f - occ * full;
  double r = full * (occ == 2 ? 1.5 : 1.0);
  if (rem > 0) r += rem <= 1.0 ? 0.85 + 0.15 * rem : 1.0 + 0.5 * (0.5 + 0.5 * (rem - 1.0));
  return r;
}

// Tile and K split of a product: the pair with the least modelled time,
//   launch + rounds * (stages * stage_us + tile_us) + what a split adds.
// A split adds one fp32 plane per split to what the consumer reads (at about
// 4 TB/s) and, for QKV and SwiGLU, a kernel of its own to finish the product
// (3 us). Splits are considered up to 2048 rows (2 above 512), where the
// unsplit tiles cannot fill the chip, and only where the partial sums fit
// `ws_elems`. In place of a table of measured choices per projection: rounds
// decide at every row count between the measured ones too (10240 rows of a
// 2048-wide product: 223 us on 160x256 tiles, two whole rounds, against 291 on
// 256x256, 1.25 rounds).
// Splitting an fp32 product into single K stages has to be modelled 4% faster (the
// model is 4-6% off there) than the shallower split: the stages are then only added
// up one after the other by the consumer, which rounds more often at full size. Two
// 256-wide layers against float64, 55 ... 176 tokens: 1.5% larger error on average where the
// QKV product was split by 8 and not by 4 for a gain of less than that.
constexpr double kSingleStageGain = 0.04;

struct Plan {
  int tile, splits;
};
static Plan plan_model(int M, int N, int K, int esz, int epi, int col_align, size_t ws_elems, bool w8) {
  Plan best{-1, 1};
  double cost_min = 1e30;
  for (int sp = 1; sp <= 8; sp *= 2) {
    if (sp > 1 && (M > 2048 || (M > 512 && sp > 2) || (size_t)sp * M * N > ws_elems)) break;
    double add = 0.0;
    if (sp > 1) add = (double)sp * M * N * 4.0 / 4e6 + (epi == EPI_RESID ? 0.3 : 3.0);
    for (int id = 0; id < kNumTiles; ++id) {
      if (!tile_fits(id, N, K, esz, sp > 1 ? EPI_PARTIAL : epi, sp, col_align, w8)) continue;
      const TileCfg &t = kTiles[id];
      const int64_t wgs = (int64_t)(N / t.bn) * ((M + t.bm - 1) / t.bm) * sp;
      const double stages = (double)K / sp * esz / kStageBytes;
      // (heads halved over two waves: 4% more, their exchange and second pass)
      const int mode = w8 ? MODE_F8W : esz == 4 ? MODE_F32 : MODE_F16;
      const double tile = stages * t.stage_us[mode] + t.tile_us[mode];
      const double cost = 2.0 + tile_rounds(wgs, t.occ) * tile * (half_heads(id, sp > 1 ? EPI_PARTIAL : epi, col_align) ? 1.04 : 1.0) + add;
      const bool single = esz == 4 && sp > best.splits && K / sp * esz == kStageBytes;
      if (cost < cost_min * (single ? 1.0 - kSingleStageGain : 1.0)) {
        cost_min = cost;
        best = Plan{id, sp};
      }
    }
  }
  return best;
}

// plan_model, remembered per thread for the shapes of the last few products
// (a forward plans the same four per layer; the model takes about a
// microsecond of host time).
static Plan plan(int M, int N, int K, int esz, int epi, int col_align, size_t ws_elems, bool w8) {
  struct Entry {
    int M, N, K, esz, epi, col_align, w8;
    size_t ws_elems;
    Plan p;
  };
  constexpr int kEntries = 16;
  static thread_local Entry memo[kEntries] = {};   // M = 0: empty
  static thread_local int next = 0;
  for (const Entry &e : memo)
    if (e.M == M && e.N == N && e.K == K && e.esz == esz && e.epi == epi && e.col_align == col_align &&
        e.w8 == (int)w8 && e.ws_elems == ws_elems)
      return e.p;
  const Plan p = plan_model(M, N, K, esz, epi, col_align, ws_elems, w8);
  memo[next] = Entry{M, N, K, esz, epi, col_align, (int)w8, ws_elems, p};
  next = (next + 1) % kEntries;
  return p;
}

// M tiles per group of the tile order (GemmArgs.gh). Measured 1, 2, 4, 8 and 16
// at 1536 ... 10240 rows: 4 is the fastest or within 1.5% of it everywhere (the
// 10240-row gate/up product 400 us with 8 and 404 with 4; 6759 x 2048 x 6144
// 150 us with 4, 153 with 16).
constexpr int kGroupM = 4;

static int col_unit(int epi, const QkvEpi *qe) { return epi == EPI_QKV ? qe->hd : 32; }

hipError_t launch_mode_f8w(int epi, int tile, int splits, const GemmArgs &a, hipStream_t s);

hipError_t launch_gemm_tile(int mode, int epi, int tile, int splits, const void *A, const void *W,
                            void *C, size_t c_plane, int M, int N, int K, int ldc, float scale,
                            float out_scale, const QkvEpi *qe, hipStream_t s, const float *col_scale,
                            const float *bias, const float *resid) {
  if (M <= 0) return hipSuccess;
  const bool w8 = mode == MODE_F8W;
  if (bias && (splits > 1 || epi == EPI_SWIGLU)) return hipErrorInvalidValue;
  const int esz = mode == MODE_F32 ? 4 : 2;
  if (epi == EPI_QKV && (!qe || (qe->hd != 64 && qe->hd != 128))) return hipErrorInvalidValue;
  if (w8 && !col_scale) return hipErrorInvalidValue;
  // the kernel addresses both operands with 32-bit byte offsets
  if ((size_t)M * K * esz > 0xFFFFFFFFull || (size_t)N * K * (w8 ? 1 : esz) > 0xFFFFFFFFull)
    return hipErrorInvalidValue;
  if (tile < 0 || tile >= kNumTiles || splits < 1 ||
      !tile_fits(tile, N, K, esz, epi, splits, col_unit(epi, qe), w8) || (splits > 1 && epi != EPI_PARTIAL))
    return hipErrorInvalidValue;
  const int gm = (M + kTiles[tile].bm - 1) / kTiles[tile].bm, gn = N / kTiles[tile].bn;
  GemmArgs a{(const char *)A, (const char *)W, C, c_plane, M, N, K, ldc, K / splits, scale, out_scale,
             epi == EPI_QKV ? *qe : QkvEpi{}, w8 ? col_scale : nullptr, bias,
             resid ? resid : (const float *)C, gm, gn, gm < kGroupM ? gm : kGroupM};
  if (w8) return launch_mode_f8w(epi, tile, splits, a, s);
  return mode == MODE_F16 ? launch_mode<MODE_F16>(epi, tile, splits, a, s)
                          : launch_mode<MODE_F32>(epi, tile, splits, a, s);
}

hipError_t launch_gemm(int mode, int epi, const void *A, const void *W, void *C, int M, int N, int K,
                       int ldc, float scale, float out_scale, float *ws, size_t ws_elems,
                       int *splits_out, const QkvEpi *qe, hipStream_t s, const float *col_scale,
                       const float *bias, const float *resid) {
  *splits_out = 0;
  if (M <= 0) return hipSuccess;
  if (epi == EPI_QKV && !qe) return hipErrorInvalidValue;
  const Plan p = plan(M, N, K, mode == MODE_F32 ? 4 : 2, epi, col_unit(epi, qe), (ws && !bias) ? ws_elems : 0,
                      mode == MODE_F8W);
  if (p.tile < 0) return hipErrorInvalidValue;
  if (p.splits > 1) {
    *splits_out = p.splits;
    return launch_gemm_tile(mode, EPI_PARTIAL, p.tile, p.splits, A, W, ws, (size_t)M * N, M, N, K, N, scale,
                            1.f, nullptr, s, col_scale);
  }
  return launch_gemm_tile(mode, epi, p.tile, 1, A, W, C, 0, M, N, K, ldc, scale, out_scale, qe, s, col_scale,
                          bias, resid);
}

}  // namespace mte
