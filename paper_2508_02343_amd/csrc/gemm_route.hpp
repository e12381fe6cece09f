// Which kernel multiplies operands of given sizes.  Host arithmetic only, no
// HIP: tests compile it by itself.
#pragma once

#include <stdint.h>

namespace mm {

// The decode kernel, the K-splitting kernel with one of its tile shapes, the
// LDS-tiled kernel with 256 x 128 or 256 x 256 tiles.
enum class GemmKernel { kDirect, kSplit, kTiled128, kTiled256 };

struct GemmRoute {
  GemmKernel kernel;
  int shape;  // index into kSplitShapes (kSplit)
};

struct GemmSizes {
  int64_t m, n;  // activation rows, weight rows
  int steps[3];  // layout steps per group
  int cus;       // CUs of the device
};

// Tile shapes of the K-splitting kernel (32-row units of weight and activation
// rows) and their measured cost, in 10 ns, on 256 CUs: a call takes about once +
// rounds * (round + step * S), S the layout steps weighted by their bytes (an
// E2M1 step 1), one round the tiles the CUs hold at once, one each (the two
// small shapes share a CU between workgroups, which the figures include).  From
// 64 .. 512 rows x K = 1024, 4096, 14336, 27648 x N = 4096 .. 14336; e.g. 2 x 2
// at K = 4096: 6.9 us for up to 256 tiles, 12.6 for 512; the LDS-tiled 256 x 128
// tile 17.7-22.8 us up to 256 tiles, 38.6-42 for 512.
struct SplitShape {
  int tn, tm, once, round;
  double step;
};
constexpr SplitShape kSplitShapes[] = {
    {1, 1, 330, 20, 4.5}, {2, 1, 340, 20, 6.7}, {2, 2, 120, 180, 10.5}, {2, 3, 200, 220, 14.5}, {2, 4, 200, 330, 16.8},
};
constexpr int kNumSplitShapes = sizeof(kSplitShapes) / sizeof(kSplitShapes[0]);
constexpr SplitShape kTiledCost = {8, 4, 0, 520, 36.5};  // the LDS-tiled kernel's 256 x 128 tile

// Workgroups of 512 threads in one launch: a grid has less than 2^32 threads.
constexpr int64_t kMaxSplitTiles = ((int64_t)1 << 23) - 1;

// Up to this many activation rows (two 16-row tiles) the decode kernel may
// run: it has a strip of weight rows for every CU where the K-splitting
// kernel's 32-row tiles have one for every second.  Weights from HBM, 75 / 18.75
// / 6.25 % split, decode kernel against the K-splitting one (us, N x K): 20 rows
// 4096 x 4096 5.2 / 6.7, 6144 x 4096 6.3 / 7.9; 32 rows 4096 x 14336 10.9 / 14.5,
// 14336 x 4096 9.3 / 8.9; 64 rows 4096 x 4096 6.9 / 5.7, 1024 x 4096 6.3 / 4.9.
constexpr int64_t kDirectMaxM = 32;
// ... unless the weight is larger than this and not mostly 8-bit codes: the
// K-splitting kernel streams long weights faster (us, 8 rows, decode kernel
// against it: 28672 x 4096 mixed, 71 MB, 15.7 / 12.7, E2M1 62 MB 12.9 / 11.4;
// 5120 x 27648 mixed, 86 MB, 23.0 / 18.4), the decode kernel the short ones
// (14336 x 4096 mixed, 36 MB, 8.2 / 8.1; 4096 x 4096, 10 MB, 4.4 / 4.7) and
// E4M3 (28672 x 4096, 21.3 / 23.5; 5120 x 27648, 34 / 38).
constexpr int64_t kDirectMaxWeight = 40ll << 20;

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t tile_count(int64_t n, int64_t m, int tn, int tm) { return ceil_div(n, 32 * tn) * ceil_div(m, 32 * tm); }

inline GemmRoute gemm_route(const GemmSizes& a) {
  const int64_t rn = ceil_div(a.n, 32) * 32, rm = ceil_div(a.m, 32) * 32;  // the padded rows
  const int64_t b8 = rn * 128 * a.steps[2], bytes = rn * (64 * (int64_t)a.steps[0] + 96 * (int64_t)a.steps[1]) + b8;
  if (a.m <= kDirectMaxM && (bytes <= kDirectMaxWeight || 2 * b8 > bytes)) return {GemmKernel::kDirect, 0};
  const double steps = a.steps[0] + a.steps[1] * (25.0 / 17) + a.steps[2] * (33.0 / 17);
  auto cost = [&](const SplitShape& s) {
    const int64_t rounds = ceil_div(tile_count(a.n, a.m, s.tn, s.tm), a.cus);
    return s.once + (double)rounds * (s.round + s.step * steps);
  };
  // 256 x 256 tiles when they give every CU at least one, else 256 x 128
  // (twice the tiles)
  GemmRoute best = {tile_count(a.n, a.m, 8, 8) >= a.cus ? GemmKernel::kTiled256 : GemmKernel::kTiled128, 0};
  double least = cost(kTiledCost);
  for (int i = 0; i < kNumSplitShapes; ++i) {
    const SplitShape& s = kSplitShapes[i];
    if (32 * s.tn > rn || 32 * s.tm > rm || tile_count(a.n, a.m, s.tn, s.tm) > kMaxSplitTiles) continue;
    const double c = cost(s);
    if (c < least) {
      least = c;
      best = {GemmKernel::kSplit, i};
    }
  }
  return best;
}

}  // namespace mm
