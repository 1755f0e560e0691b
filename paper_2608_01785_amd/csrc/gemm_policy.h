// Which kernel runs a prefill-sized GEMM: the persistent 256 x 256 kernel or
// one of the small-tile shapes.  Pure C++; no HIP types.
#pragma once

#include <cstdint>

namespace hs {

// Small-tile shapes: bn weight rows x bm activation rows per block.  `base`,
// `stage` and `round` are microseconds of a launch, of one 64-wide K stage of
// one block's tile, and of a tile's prologue and epilogue.
struct GemmTileShape {
  int bn, bm;
  float base, stage, round;
};

constexpr int kGemmTiles = 7;
constexpr GemmTileShape kGemmTileShapes[kGemmTiles] = {
    {64, 64, 3.8f, 0.206f, 0.09f},   {128, 64, 4.3f, 0.326f, 0.27f},  {128, 96, 4.3f, 0.395f, 0.68f},
    {128, 128, 4.7f, 0.457f, 0.84f}, {128, 160, 5.7f, 0.559f, 0.53f}, {128, 192, 5.2f, 0.594f, 1.3f},
    {256, 192, 2.9f, 0.995f, 5.4f},
};
// The same for the persistent kernel: a full 256 x 256 unit's stage, a
// 128-row half unit's, and either's epilogue.
constexpr float kGemmBigBase = 6.2f, kGemmBigStage = 1.353f, kGemmBigHalf = 1.286f, kGemmBigRound = 4.8f;
// A small tile has to be this much cheaper on paper.
constexpr float kGemmTileMargin = 0.93f;

// Index into kGemmTileShapes, or -1 for the persistent kernel, for an
// [M, K] x [N, K]^T product on `cus` compute units.
//
// Every output element is summed in the same order whichever kernel runs, so
// the choice may follow the budget.  It is a matter of rounds: a CU's time is
// the tiles it gets times the time of a tile, and a 256 x 256 tile (cheapest
// per product, 1.35 us a stage against 4 x 0.46) only pays when there are
// several per CU.  The constants were fitted to launches with fp16 weights;
// epilogue and weight format do not enter.  tests/gemm_rule_sweep.py times
// all eight kernels over eleven products with their own epilogues, 130 to 9151
// rows and six budgets: the choice takes 0.8 % more than the fastest kernel on
// average with fp16 weights and 3.2 % with bf16 ones (20 and 29 % at most, one
// row count before the next shape pays), at most 2.6 % more than the
// persistent kernel (9151 x 3584 x 18944 on 96 CUs), and half its time in the
// geometric mean.  At 389 x 3584 x 18944 on 160 CUs: 337 us persistent, 112 in
// 128 x 96 tiles; at 9151 x 3584 x 18944 on 256 CUs 1036 against 1124
// (256 x 192), so large batches keep the persistent kernel.
inline int gemm_tile_choice(int M, int N, int K, int cus) {
  const float stages = float(K) / 64.0f;
  auto up = [](int64_t a, int64_t b) { return int64_t((a + b - 1) / b); };
  // The persistent kernel's schedule (see gemm.hip): full rounds, then the
  // last round as halves when it would leave half the blocks idle, and a last
  // row tile of at most 128 rows as halves of its own.
  const int64_t tm = up(M, 256), tn = N / 256;
  const bool short_last = M - (tm - 1) * 256 <= 128;
  const int64_t n_full = (short_last ? tm - 1 : tm) * tn, n_short = short_last ? tn : 0;
  const int64_t grid = tm * tn < cus ? tm * tn : cus;
  int64_t full = n_full / grid, half = 0;
  const int64_t tail = n_full - full * grid;
  if (tail > 0 && 2 * tail + n_short <= grid) {
    half = 1;
  } else {
    full += tail > 0;
    const int64_t rest = n_short - (tail > 0 ? grid - tail : 0);
    half = rest > 0 ? up(rest, grid) : 0;
  }
  float best = kGemmTileMargin *
               (kGemmBigBase + stages * (kGemmBigStage * float(full) + kGemmBigHalf * float(half)) +
                kGemmBigRound * float(full + half));
  int pick = -1;
  for (int i = 0; i < kGemmTiles; ++i) {
    const GemmTileShape& t = kGemmTileShapes[i];
    const float rounds = float(up(up(M, t.bm) * (N / t.bn), cus));
    const float cost = t.base + rounds * (stages * t.stage + t.round);
    if (cost < best) {
      best = cost;
      pick = i;
    }
  }
  return pick;
}

}  // namespace hs
