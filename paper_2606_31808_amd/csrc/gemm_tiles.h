// The weight GEMM's tile shapes and the rules that pick one, and the LM head's
// kernel; plain C++, so that the host can check which launch takes which.
#pragma once
#include <cmath>

namespace lmop {

// A tile of 16*mi tokens x 16*fj*nw columns: nw waves side by side along N,
// each with all tokens and fj strips of 16 columns, kp panels of 64 features
// per ring stage, kk steps of 32 features per phase, occ workgroups per CU.
// kk = 0: gemm_split_kernel (loaders, converters and a multiplier).
// t1[format], t2[format]: measured time per 64-feature panel in ns with one
// workgroup on a CU and, where two fit, with two (format 0 = int4, 1 = FP8);
// 0 = not offered in this format, because another shape is never slower.
struct GemmTile {
  int mi, fj, nw, kp, kk, occ;
  float t1[2], t2[2];
  // the split shapes fit one kind of epilogue: the residual add takes single
  // strips, the others need pairs of strips in one wave
  bool add = true, pairs = true;
  constexpr int bm() const { return 16 * mi; }
  constexpr int bn() const { return 16 * fj * nw; }
  constexpr bool offered(bool fp8, bool add_epilogue) const {
    return t1[fp8] > 0.f && (add_epilogue ? add : pairs);
  }
};

// large token tiles convert each weight for more tokens; small ones reach
// more CUs, and walk K in stages of several panels
constexpr GemmTile kGemmTiles[] = {
    {8, 4, 4, 1, 1, 2, {900.f, 1040.f}, {1620.f, 1590.f}},
    {8, 2, 4, 1, 1, 2, {560.f, 500.f}, {943.f, 855.f}},
    {4, 2, 4, 2, 2, 2, {330.f, 430.f}, {560.f, 540.f}},
    {4, 1, 4, 2, 2, 2, {215.f, 215.f}, {350.f, 350.f}},
    {2, 2, 4, 4, 4, 1, {0.f, 195.f}, {0.f, 0.f}},
    {2, 2, 4, 1, 1, 2, {300.f, 250.f}, {415.f, 380.f}},
    {2, 1, 4, 4, 4, 2, {140.f, 0.f}, {220.f, 0.f}},
    {1, 1, 4, 4, 4, 2, {127.f, 112.f}, {200.f, 180.f}},
    {1, 1, 4, 8, 8, 1, {105.f, 97.f}, {0.f, 0.f}},
    {1, 1, 1, 8, 0, 1, {55.f, 55.f}, {0.f, 0.f}, true, false},
    {1, 2, 1, 4, 0, 1, {85.f, 85.f}, {0.f, 0.f}, false, true},
};
constexpr int kNumGemmTiles = sizeof(kGemmTiles) / sizeof(kGemmTiles[0]);

// Estimated time of the GEMM's M x N tiles per 64-feature panel: rounds over
// the 256 CUs, the last one with one workgroup a CU if they suffice.  The
// pipeline's fill and the epilogue (3-4 us of a launch) are left out, and one
// table serves the three epilogues.  Over 23 token counts from 1 to 16384 and
// the projections of the 8B and 1B widths the shape picked is the fastest or
// within 5% of it in 158 of 184 launches in int4 and 176 in FP8, at worst 12%
// slower (1B QKV of 400-1,000 tokens, O of 700 and of 4,096).
inline float gemm_tile_cost(const GemmTile& t, bool fp8, int M, int N, int K) {
  if ((K / 64) % t.kp != 0) return INFINITY;
  const long tiles = (long)((M + t.bm() - 1) / t.bm()) * (N / t.bn());
  const long round = 256 * t.occ, full = tiles / round, rem = tiles % round;
  const float tf = t.occ == 2 ? t.t2[fp8] : t.t1[fp8];
  return full * tf + (rem == 0 ? 0.f : rem <= 256 ? t.t1[fp8] : t.t2[fp8]);
}

// The shape (index into kGemmTiles) with the least estimated time for M
// tokens, N columns (a multiple of 256) and K features (of 64).  Every shape
// sums each output in the same order, so the choice never changes a bit.
inline int pick_gemm_tile(bool fp8, bool add_epilogue, int M, int N, int K) {
  int best = 0;
  float cost = INFINITY;
  for (int i = 0; i < kNumGemmTiles; ++i) {
    if (!kGemmTiles[i].offered(fp8, add_epilogue)) continue;
    const float c = gemm_tile_cost(kGemmTiles[i], fp8, M, N, K);
    if (c < cost) {
      cost = c;
      best = i;
    }
  }
  return best;
}

// Whether the LM head streams its weight through registers (head_few_kernel)
// or takes the LDS ring (head2_kernel).  The ring has a workgroup per pair of
// 128-entry vocabulary tiles, so up to 512 tiles (V = 65,536) it runs one round
// of the 256 CUs, in a time that neither V nor the rows change much, and twice
// that from there on.  The stream has a wave per tile, which slows down with
// every group of 16 rows.  Measured, us, stream against ring at d = 4096:
//   V = 128256: 9 rows 155 / 213, 32: 160 / 219, 64: 212 / 232
//   V = 66048: 16 rows 109 / 204, 32: 124 / 210, 64: 195 / 221
//   V = 50304: 1 row 101 / 106, 16: 105 / 105, 20: 111 / 108, 64: 192 / 114
//   V = 32000: 17 rows 103 / 105, 32: 117 / 107, 64: 190 / 113
//   V = 16384: 20 rows 104 / 106, 24: 107 / 106, 28: 110 / 106
//   V = 2048: 17 rows 92 / 103, 32: 105 / 105, 64: 173 / 110
// so below 65,536 the line is at 16 to 32 rows; at d = 2048 it lies a few rows
// higher.  65 rows do not fit a wave's registers.
constexpr bool head_streams(int rows, int vocab) {
  const int tiles = (vocab + 127) / 128;
  return rows <= (tiles > 512 ? 64 : tiles > 256 ? 16 : tiles > 128 ? 20 : tiles > 16 ? 24 : 32);
}

}  // namespace lmop
