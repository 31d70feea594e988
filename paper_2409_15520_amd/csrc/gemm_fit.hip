// The tiles of gemm_fit.h: which products take them, and which shape.
#include "gemm_fit.h"

namespace mpz {
namespace {

template <int WGN, int WGM, int NI, int NJ, int ST, int EPI>
hipError_t launch_fit_lr(hipStream_t st, const MfmaGemmArgs& a) {
  return a.n_seg ? launch_fit<WGN, WGM, NI, NJ, ST, EPI, true>(st, a) : launch_fit<WGN, WGM, NI, NJ, ST, EPI, false>(st, a);
}

}  // namespace

// shapes: 0 = 192 features x 256 tokens, 1 = 256 x 192, 2 = 192 x 128, 3 = 128 x 192, 4 = 256 x 128, 5 = 128 x 128; int8 weights: 1, 3, 4, 5 and
// 6 = 256 x 256
bool gemm_fit_supported(const MfmaGemmArgs& a, int shape) {
  if (a.w_absmax != nullptr || a.k_splits > 1 || a.ce_max != nullptr || a.K % 64 || !fetch_aligned(a)) return false;
  if (a.act >= 0 && a.act != MPZ_ACT_RELU) return false;
  const int es = a.out_f32 ? 4 : 2;
  if (((uintptr_t)a.out | (uintptr_t)a.residual) & 15 || a.N * es % 16 || a.ldo * es % 16 || a.ldo > (1 << 21) || (uintptr_t)a.bias & 3) return false;
  if (!a.out_f32 && a.residual != nullptr) return false;
  if ((uintptr_t)a.w_scale & 3) return false;
  const bool wide192 = shape == 0 || shape == 2, rope = a.rope_cos != nullptr;
  if (a.dual) { if (a.out_f32 || a.n_seg || a.act >= 0 || rope || wide192 || a.dual_offset % 4) return false; }
  if (rope) {
    if (a.out_f32 || a.act >= 0 || wide192 || (a.rope_dh != 64 && a.rope_dh != 128) || a.rope_cols % a.rope_dh) return false;
  }
  if ((a.out_f32 && a.act >= 0) || (a.w_scale != nullptr ? wide192 : shape == 6)) return false;
  if (a.n_seg) {
    if (a.act >= 0 || a.rows_per_copy % 32 || a.M % 32) return false;
    const int cols = rope ? a.rope_dh : wide192 ? 96 : 64;    // a wave's
    for (int s = 0; s < a.n_seg; ++s)
      if ((a.seg[s].rp != 16 && a.seg[s].rp != 32) || a.seg[s].col_begin % cols || a.seg[s].col_end % cols) return false;
  }
  return true;
}

// What a product takes in tiles of one shape, ns: every round of 256 tiles costs its edges (first fetch, epilogue; an fp32 output and its
// residual by the share of the CUs that are at it) and its K-tiles; a K-tile takes a fifth less where few CUs are busy (the clock and the
// caches are theirs).  The constants are a least-squares fit to 989 products of 23 weights of the shapes in use (K 768 to 11008; 272 to
// 16384 tokens), each timed in every shape: rms 6 % (256 x 256 in gemm_pipe.hip: 4 %).
struct FitCost { int bn, bm, edge, edge_f32, k_tile; };
constexpr FitCost kFitCost[] = {{192, 256, 7000, 7700, 1034}, {256, 192, 5700, 7250, 1060}, {192, 128, 4400, 4050, 580},
                                {128, 192, 3900, 4570, 580}, {256, 128, 5000, 5560, 725}, {128, 128, 2900, 3140, 434}};
constexpr FitCost kPipeCost = {256, 256, 8900, 5300, 1253};
// int8 weights, 460 products of 20 weights (rms 5 - 9 %): the widening is a tenth of a K-tile's time, the more where a code serves fewer tokens
constexpr FitCost kFitCost8[] = {{}, {256, 192, 6700, 8600, 1084}, {}, {128, 192, 4030, 5240, 629}, {256, 128, 5520, 6470, 871},
                                 {128, 128, 3150, 3760, 496}, {256, 256, 8200, 16000, 1313}};
double cost_of(const MfmaGemmArgs& a, const FitCost& c, bool filled = false) {    // filled: of its tiles, as if every round were whole
  const int cn = a.dual ? c.bn / 2 : c.bn;
  const long tiles = (long)((a.N + cn - 1) / cn) * ((a.M + c.bm - 1) / c.bm), rounds = (tiles + 255) / 256;
  const double fill = (tiles - (rounds - 1) * 256) / 256.0;
  if (filled) return tiles / 256.0 * (c.edge + (a.out_f32 ? c.edge_f32 : 0) + a.K / 64 * (double)c.k_tile);
  return (double)rounds * c.edge + (a.out_f32 ? (rounds - 1 + fill) * c.edge_f32 : 0.0) + a.K / 64 * (double)c.k_tile * (rounds - 0.2 + 0.2 * fill);
}

// The shape that takes a product for which the rules of gemm_mfma.hip choose `tile`, or -1: that tile.  Of the shapes that take it the one
// that costs least by the sums above (on average 0.5 % more than the fastest of them).  Against the tile chosen so far (ratio of its time
// to the shape's; bf16: 989 products, int8: 460):
//   * up to 128 tiles of 128 x 128 the smaller tiles stay ahead: more blocks, and what bounds such a product is what a CU can fetch (0.4 - 0.97;
//     int8, whose staged tile is the same size, 0.87 - 1.05); likewise where 128 x 64 ones fit the CUs (0.93 - 0.97), and outputs that are mostly
//     residual traffic (fp32, K <= 1024: one round of small tiles 0.95 - 0.98, int8 two 0.90 - 0.99).  Not gate and up, whose staged
//     tile has two weight operands to an activation: 66 to 132 small tiles 1.2 - 1.7, int8 1.6 - 1.9;
//   * 128 x 128, 192 x 128 and 128 x 64 tiles beyond that: 0.99 - 1.5, 1.14 on average; gate and up in 128 x 128: 1.31 (int8 1.15, 1.43);
//   * the 256 x 256 tile of gemm_pipe.hip: where its rounds are part-filled 1.0 - 1.45, else down to 0.77, so the sums decide, with 4 % in
//     its favour (K = 11008, whose many K-tiles the smaller shapes fetch more slowly than the sums say, 0.90 - 0.97 at that margin: 13 %;
//     weights that outgrow the last-level cache, whatever K: 0.83 - 1.1 at 0.82 to 0.88 by the sums, 1.0 - 1.26 below: 18 %);
//     from four of its rounds on it stays (0.9 - 1.03 beyond), and for gate and up of up to 384 tokens, which are a stream of weights
//     (0.87 - 0.94).  The staged 256 x 256 tile of int8 weights: 1.0 - 1.35, 1.13 on average, two rounds and more included.
int gemm_fit_shape(const MfmaGemmArgs& a, int tile) {
  if (a.tile_cfg >= 20 && a.tile_cfg < 27) return gemm_fit_supported(a, a.tile_cfg - 20) ? a.tile_cfg - 20 : -1;
  if (a.tile_cfg != 0) return -1;
  const bool int8 = a.w_scale != nullptr;
  const long n128 = (a.N + 127) / 128, t1 = n128 * ((a.M + 127) / 128);
  if (t1 <= (a.dual ? 64 : 128) || (tile == 9 && n128 * ((a.M + 63) / 64) <= 256)) return -1;
  if (a.out_f32 && a.K <= 1024 && t1 <= (int8 ? 512 : 256)) return -1;
  double least = 0.0;
  if (tile == 6 && !int8) {
    const int cn = a.dual ? 128 : 256;
    if ((long)((a.N + cn - 1) / cn) * ((a.M + 255) / 256) > 1024 || (a.dual && a.M <= 384)) return -1;
    const size_t weights = (size_t)(a.dual ? 2 : 1) * a.N * a.K * 2;
    least = (weights >= (size_t)240 << 20 ? 0.82 : a.K > 8192 ? 0.87 : 0.96) * cost_of(a, kPipeCost);
  }
  int shape = -1;
  for (int s = 0; s < 7; ++s) {
    if (!gemm_fit_supported(a, s)) continue;
    const double c = cost_of(a, int8 ? kFitCost8[s] : kFitCost[s]);
    if (least == 0.0 || c < least) { least = c; shape = s; }
  }
  return shape;
}

// A block's four products of T tokens in one pass, over the mean of two sums between which two halves at the same time lie: the halves
// one behind the other, each in rounds of its own, and the halves as if no CU were ever idle.  (All by the costs above.  At 54 sizes of six other models, 4 layers, the faster way or one within 3 % of it but at five, up to 5 %; int8 at all 54.)
double gemm_fit_halves_gain(int d, int nqkv, int d_ffn, bool gate_up, bool int8, long T) {
  const int shapes[4][4] = {{nqkv, d, 0, 0}, {d, d, 1, 0}, {d_ffn, d, 0, gate_up}, {d, d_ffn, 1, 0}};   // columns, K, fp32 output, gate and up
  double whole = 0.0, apart = 0.0, filled = 0.0;
  for (const auto& g : shapes) {
    MfmaGemmArgs a{};
    a.N = g[0]; a.K = g[1]; a.out_f32 = g[2]; a.dual = g[3];
    double w = 0.0, p = 0.0, f = 0.0;
    auto least = [](double& m, double c) { m = m == 0.0 || c < m ? c : m; };
    for (int s = 0; s <= 6; ++s) {
      const FitCost& c = int8 ? kFitCost8[s] : s < 6 ? kFitCost[s] : kPipeCost;
      if (c.bn == 0 || (c.bn == 192 && (a.dual || d >= 1024))) continue;
      a.M = (int)T;
      least(w, cost_of(a, c));
      a.M = (int)(T / 2);
      least(p, 2.0 * cost_of(a, c));
      least(f, 2.0 * cost_of(a, c, true));
    }
    whole += w; apart += p; filled += f;
  }
  return 2.0 * whole / (apart + filled);
}

hipError_t launch_gemm_fit(hipStream_t st, const MfmaGemmArgs& a, int shape) {
  if (a.w_scale != nullptr) return launch_gemm_fit_int8(st, a, shape);
#define SHAPES(EPI)                                              \
  switch (shape) {                                               \
    case 1: return launch_fit_lr<4, 2, 4, 6, 2, EPI>(st, a);     \
    case 3: return launch_fit_lr<2, 4, 4, 3, 3, EPI>(st, a);     \
    case 4: return launch_fit_lr<4, 2, 4, 4, 3, EPI>(st, a);     \
    default: return launch_fit_lr<2, 4, 4, 2, 4, EPI>(st, a);    \
  }
  if (a.dual) {
    switch (shape) {
      case 1: return launch_fit<4, 2, 4, 6, 2, FIT_DUAL, false>(st, a);
      case 3: return launch_fit<2, 4, 4, 3, 3, FIT_DUAL, false>(st, a);
      case 4: return launch_fit<4, 2, 4, 4, 3, FIT_DUAL, false>(st, a);
      default: return launch_fit<2, 4, 4, 2, 4, FIT_DUAL, false>(st, a);
    }
  }
  if (a.rope_cos != nullptr) {
    if (a.rope_dh == 128) { SHAPES(FIT_ROPE128) }
    SHAPES(FIT_ROPE64)
  }
  if (a.out_f32) {
    if (shape == 0) return launch_fit_lr<2, 4, 6, 4, 2, FIT_F32>(st, a);
    if (shape == 2) return launch_fit_lr<2, 4, 6, 2, 3, FIT_F32>(st, a);
    SHAPES(FIT_F32)
  }
  if (shape == 0) return launch_fit_lr<2, 4, 6, 4, 2, FIT_BF16>(st, a);
  if (shape == 2) return launch_fit_lr<2, 4, 6, 2, 3, FIT_BF16>(st, a);
  SHAPES(FIT_BF16)
#undef SHAPES
}

}  // namespace mpz
