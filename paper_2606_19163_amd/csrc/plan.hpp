// Tile and K split of the conv-mode GEMMs whose grid does not fill the GPU
// (small images, batches and token counts).  Host only.
#pragma once

#include <algorithm>

#include "kernels.hpp"

namespace pulse {

struct ConvPlan {
  int tile, ks, ksteps;  // K splits over blocks, K-steps per split
};

inline long conv_tile_count(int tile, long P, int N) {
  const TileInfo ti = tile2_info(tile);
  return ((P + ti.bm - 1) / ti.bm) * ((N + ti.bn - 1) / ti.bn);
}

// ks splits of K, without an empty one
inline ConvPlan conv_plan_of(int tile, long ks, int K) {
  ConvPlan p;
  p.tile = tile;
  const long kt = K / tile2_info(tile).bk;
  p.ksteps = (int)((kt + ks - 1) / ks);
  p.ks = (int)((kt + p.ksteps - 1) / p.ksteps);
  return p;
}

// Time model of one launch, its constants fitted to 33 shapes of 64 to 8192
// rows (every tile with up to 16 splits; the model's choice is 2 % above the
// fastest in the mean): `t0` us of launch, set-up and epilogue, `step` us per
// K-step (of one of the tile's `kg` K groups) with one block per CU, and
// (1 + share) times that with two; `again` us for each further round of blocks
// past the resident ones, which set up and write out once more (measured at
// 128 to 2048 blocks over K = 64 to 2048: 64 x 64 in two K groups, one block
// per CU, 6.7 us with 256 blocks of K = 128, 11.5 with 512, 20.9 with 1024).
// Without it small tiles and K splits were taken in several rounds: 24 x 32 x 32
// pixels, 128 -> 64 3x3, 22.7 us (32 x 64 in four groups, 768 blocks) against
// 15.1 (64 x 128); 13056 tokens, 128 -> 128, 7.9 (32 x 64) against 6.5; 1472 x
// 1024 over 9216 50.1 (five splits) against 48.1.  Of 265 random plans that it
// changes, images and tokens, the mean is 12 % faster, none but one slower by
// more than 1 %; in a stage 0 to 3 %.
struct ConvCost {
  int tile, kg;
  double t0, step, share, again;
};

// What a K split costs besides its partials' traffic (the finalize launch),
// and what a caller pays for a reduction of the output that the launch does
// not do itself.
constexpr double CONV_T_FINALIZE = 2.6, CONV_BYTES_PER_US = 5.0e6;

// The reduction a launch is asked to do in its epilogue: the output's
// GroupNorm statistics (a K split's finalize does them too) or the
// GroupNorm-backward sums (only whole tiles inside an image, no K split).
enum ConvWant { CONV_PLAIN = 0, CONV_STATS = 1, CONV_GNB = 2 };

// The cheapest of the 64-channel bf16 tiles and K splits of at most ks_max
// for P pixels x N columns over K; wide: the 128-row tile of this N.
// part_max (floats, < 0: no limit): the partials a split may take.  A tile
// of 32 or 64 rows puts four to ten times the blocks of a 128-row one on the
// GPU, K groups inside a block shorten its chain of K-steps without partials
// in HBM.  Measured against the 128-row tiles with a K split (us, finalize
// included): 2 x 8 x 8 pixels, 1280 -> 1280 3x3: 17.1 (64 x 64 in two
// groups, 6 splits) against 24.9; 2560 -> 1280 23.5 against 33.7;
// 4 x 16 x 16, 512 -> 512: 17.3 (32 x 64 in two groups) against 27.2;
// 32 x 32, 320 -> 320: 12.6 against 20.4; 2 x 64 x 64, 320 -> 320: 27.7
// (64 x 128) against 33.8; 512 tokens, 3072 -> 768: 13.6 (32 x 64 in four
// groups) against 25.5 for 64 x 128 in one, 768 -> 768 7.4 against 10.5.
inline ConvPlan conv_plan_small(long P, int N, int K, int hw, int wide, long ks_max,
                                long part_max, ConvWant want) {
  static const ConvCost costs[] = {
      {TILE2_C128x160, 1, 10.0, 0.62, 0.09, 9.0}, {TILE2_C128x128, 1, 9.9, 0.52, 0.45, 6.6},
      {TILE2_C64x128S3, 1, 5.1, 0.45, 0.21, 4.4}, {TILE2_C32x64, 1, 4.3, 0.24, 0.38, 2.0},
      {TILE2_C32x64G2, 2, 5.0, 0.33, 0.74, 3.6},  {TILE2_C32x64G4, 4, 5.6, 0.59, 0.0, 4.3},
      {TILE2_C64x64G2, 2, 5.3, 0.52, 0.0, 4.2},
  };
  ConvPlan best = conv_plan_of(wide, 1, K);
  double least = 1e30;
  for (const ConvCost& c : costs) {
    const TileInfo ti = tile2_info(c.tile);
    if (ti.bm == 128 && c.tile != wide) continue;
    const long tiles = conv_tile_count(c.tile, P, N), kt = K / ti.bk;
    for (long ks = 1; ks <= std::min(ks_max, std::max(1L, kt / 4)); ++ks) {
      const ConvPlan p = conv_plan_of(c.tile, ks, K);
      if (p.ks != ks) continue;  // the same split as a smaller count
      if (ks > 1 && part_max >= 0 && ks * P * N > part_max) break;
      const long steps = (p.ksteps + c.kg - 1) / c.kg;
      const long per_cu = (tiles * ks + 255) / 256;
      const long conc = std::min(per_cu, (long)std::min(ti.per_cu, 2));
      const long rounds = (per_cu + conc - 1) / conc;
      double t = c.t0 + rounds * steps * c.step * (conc > 1 ? 1.0 + c.share : 1.0) +
                 (per_cu - 1) / ti.per_cu * c.again;
      if (ks > 1) t += CONV_T_FINALIZE + ks * P * (double)N * 8.0 / CONV_BYTES_PER_US;
      const bool whole = ks == 1 && hw % ti.bm == 0;
      if (want == CONV_STATS && ks == 1 && !whole) t += 5.0;
      if (want == CONV_GNB && !whole) t += 8.0;
      if (t < least) {
        least = t;
        best = p;
      }
    }
  }
  return best;
}

}  // namespace pulse
