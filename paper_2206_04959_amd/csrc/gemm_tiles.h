// Tile shapes of the bf16 GEMM and the choice among them (host side; gemm.hip has
// the kernels).
#pragma once

#include "kernels.h"

namespace merak {

constexpr int kBK = 64;  // K per stage

struct GemmBatch {
  GemmProblem p[kMaxGroup];
  int tile_start[kMaxGroup + 1];
  int n_probs;
};

// Tile shapes of the bf16 kernel: BM x BN with WM x WN waves and NS LDS stages.
enum TileCfg {
  TILE_AUTO = 0,
  TILE_256x256_W4_S2 = 1,  // 2x2 waves of 128x128
  TILE_256x128_W4_S3 = 2,  // 2x2 waves of 128x64
  TILE_128x256_W4_S3 = 3,  // 2x2 waves of 64x128
  TILE_128x128_W4_S2 = 4,  // 2x2 waves of 64x64
  TILE_128x128_W4_S3 = 5,
  TILE_128x128_W4_S4 = 6,
  TILE_256x256_W8_S2 = 7,  // 2x4 waves of 128x64
  TILE_256x128_W8_S3 = 8,  // 4x2 waves of 64x64
  TILE_128x192_W4_S2 = 9,   // 2x2 waves of 64x96
  TILE_256x192_W8_S2 = 10,  // 4x2 waves of 64x96
  TILE_COUNT = 11,          // end of the shapes merak_gemm_tile_override offers
  TILE_128x128_W8_S4,       // 4x2 waves of 32x64
  TILE_256x128_W8_S2,       // 4x2 waves of 64x64
  TILE_128x192_W8_S4,       // 4x2 waves of 32x96
  TILE_192x128_W8_S4,       // 2x4 waves of 96x32
  TILE_64x128_W8_S4         // 2x4 waves of 32x32 (A with K contiguous)
};

inline long long tile_count(const GemmBatch& b, int bm, int bn) {
  long long t = 0;
  for (int i = 0; i < b.n_probs; ++i) t += (long long)((b.p[i].M + bm - 1) / bm) * ((b.p[i].N + bn - 1) / bn);
  return t;
}

// Tile choice of a launch that shares the chip with other launches (the stage's
// streams), measured inside the stage step.  Large tiles on 8 waves (two per
// SIMD) move the fewest operand bytes per FLOP through L2 and LDS, and CUs that
// a launch leaves idle run the other streams' work: the input- and
// weight-gradient GEMMs (B read with M/N contiguous) run as 256 x 256 tiles,
// every other GEMM with at least 128 such tiles as 256 x 192 tiles, narrower
// problems (most GEMMs of stages with 2048-row sub-micro-batches) as 256 x 128
// tiles with a 3-stage ring while that still gives at least 100 tiles, and the
// narrowest (the projection's input gradient at N = h/t = 768) as 128 x 128
// tiles of eight waves.  Against 128 x 192 tiles everywhere the stage step
// measured +6.3% (819 -> 870 TFLOP/s); 256 x 256 for the weight gradients added
// 0.6%, the 256 x 128 rule 2.9% on the 1.5B-shaped stage and 1.8% on the
// 2.5B-shaped shard, the last rule 0.7% on the 8.3B-shaped shard (10.15 ->
// 10.07 ms).  The choice for a launch alone (below) is 2-6% slower here
// (8.3B-shaped 10.32, 1.5B-shaped 11.97 against 11.69, 2.5B-shaped 6.08 against
// 5.75, 20B-shaped 15.35 against 14.85 ms).
inline int choose_tile_shared(const GemmBatch& b, bool b_t) {
  if (b_t && tile_count(b, 256, 256) >= 128) return TILE_256x256_W8_S2;
  if (tile_count(b, 256, 192) >= 128) return TILE_256x192_W8_S2;
  if (tile_count(b, 256, 128) >= 100) return TILE_256x128_W8_S3;
  return TILE_128x128_W8_S4;
}

// Tile choice of a launch that has the chip to itself: the least estimated
// time.  One workgroup runs per CU, so a launch takes whole rounds of 256
// tiles; a round costs `fix` us plus `stage` us per K stage of 64, both
// measured with 256 tiles (3072 to 4096 rows and columns, K = 1024 and 4096), and
// a partly filled round 0.45 + 0.55 x its fill of that (less contention for the
// operands).  Larger tiles come first and give way only to an estimate 6%
// lower: past one round they also keep the higher clock.  Measured (us, before
// -> after): 2048 x 1600 x 1600 26.4 -> 17.3, 4096 x 768 x 3072 37.4 -> 24.7,
// 1024 x 1024 x 1280 18.3 -> 10.4, 1920 x 3840 x 4096 (weight gradient) 73 ->
// 65.6, 4096 x 4096 x 4096 144 -> 110; 4096 x 3072 x 3072 stays 68.4.
// Two calls at once, one per stream, take between 0.6 and 1.1 times what they took
// with the rule above and 128 x 192 tiles of four waves as its last shape (us a
// pair): 1024 x 1024 x 1024 18.2 -> 10.3, 2048 x 6400 x 1600 87 -> 83, 2048 x 1920 x
// 3840 with 2048 x 1600 x 1600 54 -> 47; but 8192 x 3072 x 3072 237 -> 248, 2048 x 1920
// x 3840 60 -> 63 and 1920 x 3840 x 4096 (weight gradient) 112 -> 124.
inline int choose_tile_alone(const GemmBatch& b, bool a_t) {
  static const struct {
    int bm, bn, cfg;
    float fix, stage;
  } kTiles[] = {
      {256, 256, TILE_256x256_W8_S2, 3.6f, 1.585f}, {256, 192, TILE_256x192_W8_S2, 2.7f, 1.2f},
      {256, 128, TILE_256x128_W8_S2, 1.8f, 0.89f},  {192, 128, TILE_192x128_W8_S4, 1.35f, 0.67f},
      {128, 192, TILE_128x192_W8_S4, 1.35f, 0.67f}, {128, 128, TILE_128x128_W8_S4, 0.9f, 0.48f},
      {64, 128, TILE_64x128_W8_S4, 0.45f, 0.33f},
  };
  constexpr float kLaunch = 5.0f;  // us, whatever the tile
  int k_max = 0;
  for (int i = 0; i < b.n_probs; ++i) k_max = b.p[i].K > k_max ? b.p[i].K : k_max;
  int best = TILE_256x256_W8_S2;
  float best_us = 0.0f;
  for (const auto& t : kTiles) {
    if (a_t && t.cfg == TILE_64x128_W8_S4) continue;  // needs A with K contiguous
    const long long n = tile_count(b, t.bm, t.bn), rest = n % 256;
    const float rounds = (float)(n / 256) + (rest ? 0.45f + 0.55f * (float)rest / 256.0f : 0.0f);
    const float us = kLaunch + rounds * (t.fix + t.stage * (float)(k_max / kBK));
    if (best_us == 0.0f || us < 0.94f * best_us) {
      best = t.cfg;
      best_us = us;
    }
  }
  return best;
}

}  // namespace merak
