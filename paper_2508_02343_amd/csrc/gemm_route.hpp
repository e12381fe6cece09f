// Which kernel multiplies operands of given sizes, and how it shares out the
// work.  Host arithmetic only, no HIP: tests compile it by itself.
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

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t tile_count(int64_t n, int64_t m, int tn, int tm) { return ceil_div(n, 32 * tn) * ceil_div(m, 32 * tm); }

// Wavefronts per group where a workgroup's W wavefronts each work on one group:
// one for each group that has steps, then one at a time to the group whose
// wavefronts have the most to do each, a step of group G counting cost[G]
// (ties: the wider format).
inline void share_waves(const int* steps, const int* cost, int W, int* w) {
  for (int G = 0; G < 3; ++G) w[G] = steps[G] > 0 ? 1 : 0;
  for (int k = w[0] + w[1] + w[2]; k < W && k > 0; ++k) {
    int best = -1;
    int most = -1;
    for (int G = 2; G >= 0; --G) {
      if (w[G] == 0) continue;
      const int c = (steps[G] + w[G] - 1) / w[G] * cost[G];  // (at most 2^23 steps)
      if (c > most) {
        most = c;
        best = G;
      }
    }
    ++w[best];
  }
}
constexpr int kEvenCost[3] = {1, 1, 1};     // (decode kernel)
constexpr int kByteCost[3] = {17, 25, 33};  // a row's step with its scales, in 4 bytes (K-splitting kernel)

// ---- the decode kernel ----

// Up to this many activation rows (four 16-row tiles) the decode kernel may run.
constexpr int64_t kDirectMaxM = 64;

// Weight rows and wavefronts per workgroup of the decode kernel.
struct DirectPlan {
  int rows, waves;
};

// One activation tile (m <= 16): a whole 32-row group per workgroup (each
// step's loads are one contiguous 2 KB record) with four wavefronts when that
// still gives every CU a strip, else 16-row strips with eight wavefronts.
// Measured against the even spread below on this tile: 7.7 against 8.3 us
// (N = 14336, E2M1), equal for E4M3.
// More: the fewest multiple of 8 rows (at least 16, at most 64) that spreads the
// weight rows evenly over k workgroups per CU, k as small as that allows, so
// that every CU streams about the same number of bytes and each activation
// fragment feeds up to four weight tiles.
inline DirectPlan direct_plan(int64_t m, int64_t n, int cus) {
  if (m <= 16) return ceil_div(n, 32) >= cus ? DirectPlan{32, 4} : DirectPlan{16, 8};
  int64_t k = n / (64 * (int64_t)cus);
  for (k = k < 1 ? 1 : k;; ++k) {
    const int64_t r = ceil_div(ceil_div(n, k * cus), 8) * 8;
    if (r <= 64) return DirectPlan{r < 16 ? 16 : (int)r, 8};
  }
}

// ---- the K-splitting kernel ----

// Tile shapes in 32-row units of weight and activation rows.
struct SplitShape {
  int tn, tm;
};
constexpr SplitShape kSplitShapes[] = {{1, 1}, {2, 1}, {2, 2}, {2, 3}, {2, 4}};
constexpr int kNumSplitShapes = sizeof(kSplitShapes) / sizeof(kSplitShapes[0]);

// ---- the choice: the kernel with the least estimated time ----
//
// Estimates in us, fitted to 8000 sizes (1 .. 8192 x 128 .. 27648 x 512 .. 28672,
// E2M1, E3M2, E4M3 and mixed splits) on 256 CUs with the weights in rotation
// beyond the caches, as replays of a captured graph: within 4-9 % (K-splitting and
// tiled kernels) and 8-10 % (decode kernel) in the mean square.  With weights that
// stay in the cache, as the rule before this one was fitted, the K-splitting
// kernel looks up to 1.6 times faster than it is in a model.  Against every
// kernel measured at these and 3100 more sizes the choice is 0.6 % slower than the
// best in the mean; the former rule was 7 % slower, worst (us, the former choice /
// now, M x K x N): 8192 x 128 x 14336 E2M1 212 / 66, 24 x 27648 x 4096 E2M1 21.8 /
// 15.1, 8 x 27648 x 4096 mixed 26.6 / 16.1.
//
// A kernel's time is a sum over the parts that bound it at some sizes: its
// launch, the rounds of tiles over the CUs, in each round the longest chain of
// steps of a wavefront (latency) and the steps of the tile (its loads and
// MFMAs), and the bytes of the operands and of the result.
struct GemmCost {
  double once;     // per call
  double round;    // per round of tiles
  double chain;    // per round and step of the longest chain
  double step;     // per round and step of the K loop
  double w, x, y;  // per 2^20 bytes of weight, activation and result
};
constexpr GemmCost kSplitCost[kNumSplitShapes] = {
    {2.68, 0.0429, 0.0528, 0.0549, 0.084, 0.143, 0.549}, {2.83, 0.0739, 0.0388, 0.0684, 0.102, 0, 0.594},
    {1.79, 1.73, 0, 0.112, 0.0859, 0.0276, 0.195}, {1.32, 2.81, 0, 0.125, 0.11, 0.238, 0.247},
    {1.51, 3.58, 0.0783, 0.132, 0.12, 0.424, 0.0965}};
constexpr GemmCost kTiled128Cost = {4.74, 0, 0, 0.42, 0.0564, 0, 0.256};
constexpr GemmCost kTiled256Cost = {0, 9.2, 0, 0.583, 0.0828, 0.158, 0.00553};

// The decode kernel's rounds are strips per CU, at least one, without rounding
// up (several run on a CU at a time); with one activation tile and 16 or 32 weight
// rows per workgroup, with two and with four activation tiles.
struct DirectCost {
  double once, round;
  double chain, chain_m, chain_n;  // per round and step of the longest chain: fixed, per 16 activation rows, per 16 weight rows
  double w, y;
};
constexpr DirectCost kDirectCost[4] = {
    {2.32, 0, 0, 0.0509, 0.17, 0.111, 0.0414}, {2.76, 0.153, 0, 0.00368, 0.00246, 0.188, 0.306},
    {0.631, 1.82, 0.23, 0, 0, 0.134, 2.08}, {0, 2.88, 0.0375, 0.0936, 0.0649, 0.0853, 1.44}};

// A step's time in the estimates: E2M1 1.  E3M2 codes are 24 bytes per lane and
// block: two loads (K-splitting kernel), three (decode kernel).
constexpr double kStepTime[3] = {1, 27.0 / 17, 33.0 / 17}, kDirectStepTime[3] = {1, 2, 33.0 / 17};

// The estimates scatter by a few percent: between near equals the decode kernel
// (up to kDirectMaxM rows) and the tiled one (above) are taken.  Without the
// handicap five times as many of the 11100 sizes lose more than 3 % to them.
constexpr double kHandicap = 1.06;

inline double longest_chain(const int* steps, const int* cost, int W, const double* time) {
  int w[3];
  share_waves(steps, cost, W, w);
  double most = 0;
  for (int G = 0; G < 3; ++G) {
    if (!steps[G]) continue;
    const double c = (steps[G] + w[G] - 1) / w[G] * time[G];
    most = c > most ? c : most;
  }
  return most;
}

inline GemmRoute gemm_route(const GemmSizes& a) {
  constexpr double kMB = 1 << 20;
  constexpr int64_t kMaxThreads = (int64_t)1 << 32;  // a launch has fewer
  const int64_t rn = ceil_div(a.n, 32) * 32, rm = ceil_div(a.m, 32) * 32;  // the padded rows
  const int* S = a.steps;
  const double row_bytes = 68.0 * S[0] + 100.0 * S[1] + 132.0 * S[2];  // with scales
  const double w = (double)rn * row_bytes / kMB, x = (double)rm * row_bytes / kMB, y = 2.0 * (double)a.m * (double)a.n / kMB;
  const double steps = S[0] * kStepTime[0] + S[1] * kStepTime[1] + S[2] * kStepTime[2];
  const double chain = longest_chain(S, kByteCost, 8, kStepTime);
  auto cost = [&](const GemmCost& c, int tn, int tm) {
    const double rounds = (double)ceil_div(tile_count(a.n, a.m, tn, tm), a.cus);
    return c.once + rounds * (c.round + c.chain * chain + c.step * steps) + c.w * w + c.x * x + c.y * y;
  };
  const double tiled = a.m <= kDirectMaxM ? kHandicap : 1.0;
  GemmRoute best = {GemmKernel::kTiled256, 0};
  double least = tiled * cost(kTiled256Cost, 8, 8);
  auto offer = [&](double c, GemmRoute r, int64_t threads) {
    if (threads < kMaxThreads && c < least) {
      least = c;
      best = r;
    }
  };
  offer(tiled * cost(kTiled128Cost, 8, 4), {GemmKernel::kTiled128, 0}, tile_count(a.n, a.m, 8, 4) * 512);
  if (a.m <= kDirectMaxM) {
    const DirectPlan p = direct_plan(a.m, a.n, a.cus);
    const DirectCost& c = kDirectCost[a.m <= 16 ? (p.waves == 8 ? 0 : 1) : (a.m <= 32 ? 2 : 3)];
    const int64_t strips = ceil_div(a.n, p.rows);
    const double rounds = strips > a.cus ? (double)strips / a.cus : 1.0;
    const double per_step = c.chain + c.chain_m * (double)a.m / 16 + c.chain_n * p.rows / 16;
    offer(c.once + rounds * (c.round + per_step * longest_chain(S, kEvenCost, p.waves, kDirectStepTime)) + c.w * w + c.y * y,
          {GemmKernel::kDirect, 0}, strips * 64 * p.waves);
  }
  for (int i = 0; i < kNumSplitShapes; ++i) {
    const SplitShape& s = kSplitShapes[i];
    if (32 * s.tn > rn || 32 * s.tm > rm) continue;  // the operands have not so many rows
    offer(kHandicap * cost(kSplitCost[i], s.tn, s.tm), {GemmKernel::kSplit, i}, tile_count(a.n, a.m, s.tn, s.tm) * 512);
  }
  return best;
}

}  // namespace mm
