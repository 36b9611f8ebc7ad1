// Which tile variant of the matrix kernel a launch takes, and whether its long reductions are spread over blocks.
// Plain host code.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <vector>

namespace sna {

struct TileWork { int M, K, kt, taps; };              // one problem: output rows and columns, K steps of the whole reduction, R * S
struct TileShape { int bm, bn, max_steps; };          // one variant: its tile, and the most K steps one block may walk
struct TileChoice { int variant; bool split; };

// K chunking, a function of the reduction length only: the same layer of the same subnet is
// summed in the same order whatever it is batched with and however its blocks are laid out.
inline int chunk_steps(int kt_all) {
  const int n = kt_all <= 24 ? 1 : (kt_all <= 64 ? 2 : 4);
  return (kt_all + n - 1) / n;
}

// The expected time of a launch with a tile variant, in microseconds on MI355X, is
//   launch + per_cu * (block + steps * (step or step_taps [+ walk]))
// and, when reductions are spread over blocks, 1.9 us + 1.6 us per MB of partial sums.  per_cu is the launch's blocks per
// CU (whole below four: a second block on some CUs lasts as long as on all), `steps` the K steps one block walks, averaged
// over the blocks; step_taps is the step of a convolution with more than one tap, `walk` what folding chunk sums in
// registers adds to it where it costs occupancy.  The constants were fitted, for the order of the variants where they lie
// close, to 612 launch shapes of the three bf16 families (batches 1 to 64, every variant with and without split
// reductions, in place inside a forward), before the 32x32 deep ring was given two waves, lone pointwise launches their
// preloaded arguments and blocks their XCDs of tile_map.h.  With the kernels as they are, 830 launch shapes of the same
// families (medians of 7), the variant it picks is on average 1.3 % slower than the fastest of all, and by time: 0.3 %
// where it picks 28 to 30, 1 to 5 % for the others.  128-row tiles with 64-row ones for launches below 256 tiles were 35 %
// slower.
struct TileCost { int variant; float launch, block, step, step_taps, walk; };
constexpr TileCost kTileCosts[] = {
    {28, 2.76f, 0.36f, 0.111f, 0.134f, 0.f},            // 32x32, deep ring
    {29, 2.64f, 1.30f, 0.247f, 0.317f, 0.f},            // 64x64, deep ring
    {30, 1.82f, 4.83f, 0.426f, 0.456f, 0.f},            // 128x96, deep ring
    {4, 2.77f, 0.37f, 0.354f, 0.571f, 0.f},             // 64x64
    {27, 5.80f, 0.31f, 0.368f, 0.323f, 0.055f},         // 64x64, one stage
    {25, 4.31f, 0.25f, 0.364f, 0.536f, 0.061f},         // 64x128, one stage
    {1, 5.06f, 0.34f, 0.414f, 0.410f, 0.f},             // 128x64
    {2, 6.81f, 0.56f, 0.945f, 0.478f, 0.f},             // 128x96
    {8, 2.26f, 1.62f, 0.340f, 0.412f, 0.f},             // 64x128, fetching waves
    {9, 2.77f, 2.48f, 0.338f, 0.357f, 0.f},             // 128x64, fetching waves
    {11, 1.73f, 4.21f, 0.488f, 0.702f, 0.f},            // 128x128, fetching waves
    {22, 5.72f, 1.37f, 0.497f, 0.684f, 0.047f},         // 128x128, one stage
    {12, 3.14f, 0.28f, 0.440f, 0.463f, 0.f},            // 128x32, two stages
    {24, 7.46f, 0.54f, 0.442f, 0.442f, 0.132f},         // 128x96, one stage
};

constexpr int kTileCostCount = sizeof(kTileCosts) / sizeof(kTileCosts[0]);

// The variant for the n problems of one launch (`shapes` is indexed by variant; tile edges are multiples of 32, at most
// 128), and whether their chunked reductions are spread over blocks (split_mode 1: never, 2 and 3: always).  A list of
// launches built anew asks this for every layer slot, so a problem's tile counts are computed once for all variants and
// both layouts (building the list of a ResNet-shaped call over sixteen subnets: 620 us of host time with each variant and
// layout walking the problems' descriptors, 290 now, 260 before there was a formula to ask).
inline TileChoice pick_tile(const TileWork* ws, size_t n, int split_mode, const TileShape* shapes) {
  const int first = split_mode >= 2;
  double blocks[kTileCostCount][2] = {}, work[kTileCostCount][2] = {}, sums_mb = 0;
  bool bad[kTileCostCount][2] = {}, chunked = false;
  for (size_t i = 0; i < n; ++i) {
    const TileWork& w = ws[i];
    const int per = chunk_steps(w.kt), chunks = per < w.kt ? (w.kt + per - 1) / per : 1;
    const double rows[4] = {(double)((w.M + 31) / 32), (double)((w.M + 63) / 64), (double)((w.M + 95) / 96), (double)((w.M + 127) / 128)};
    const double cols[4] = {(double)((w.K + 31) / 32), (double)((w.K + 63) / 64), (double)((w.K + 95) / 96), (double)((w.K + 127) / 128)};
    if (chunks > 1) sums_mb += 4e-6 * chunks * w.M * w.K;
    chunked = chunked || chunks > 1;
    for (int c = 0; c < kTileCostCount; ++c) {
      const TileCost& k = kTileCosts[c];
      const TileShape& s = shapes[k.variant];
      const double b = rows[s.bm / 32 - 1] * cols[s.bn / 32 - 1];
      const float step = w.taps > 1 ? k.step_taps : k.step;
      blocks[c][0] += b;
      work[c][0] += b * w.kt * (step + (chunks > 1 ? k.walk : 0.f));
      bad[c][0] |= w.kt > s.max_steps;
      if (chunks == 1) {
        blocks[c][1] += b;
        work[c][1] += b * w.kt * step;
        bad[c][1] |= w.kt > s.max_steps;
      } else {
        blocks[c][1] += b * chunks;
        work[c][1] += b * chunks * per * step;
        bad[c][1] |= per > s.max_steps;
      }
    }
  }
  const int last = split_mode == 1 || !(chunked || first) ? 0 : 1;      // nothing to spread: one layout
  TileChoice best{1, first != 0};
  double best_us = 0;
  bool any = false;
  for (int c = 0; c < kTileCostCount; ++c)
    for (int split = first; split <= last; ++split) {
      if (bad[c][split]) continue;
      double per_cu = blocks[c][split] / 256;
      if (per_cu < 4) per_cu = std::ceil(per_cu);
      double us = kTileCosts[c].launch + per_cu * (kTileCosts[c].block + work[c][split] / blocks[c][split]);
      if (split && sums_mb > 0) us += 1.9 + 1.6 * sums_mb;
      if (!any || us < best_us) {
        any = true;
        best_us = us;
        best = {kTileCosts[c].variant, split != 0};
      }
    }
  return best;
}

// The variant that a tuned shape gets, from forwards run with every launch forced to one variant after the other.
// samples[v].ms: the time of the shape's launches that ran with v, one sum per forward; samples[v].launches: how many
// those were.  A shape's launches need not all take a variant (an input scaled on its way takes few), and a variant that
// ran on fewer of them than another is not compared: its sum is of less work.  The variant `without` an entry stays unless
// another is 2 % faster (the least of some thirty noisy medians is often a slower variant's).
struct TuneSample { std::vector<double> ms; int launches = 0; };
inline int measured_variant(const std::vector<TuneSample>& samples, int without) {
  int all = 0, best = -1;
  for (const TuneSample& s : samples) all = std::max(all, s.launches);
  auto median = [](std::vector<double> t) { std::sort(t.begin(), t.end()); return t[t.size() / 2]; };
  auto whole = [&](size_t v) { return v < samples.size() && !samples[v].ms.empty() && samples[v].launches == all; };
  double best_ms = 0;
  for (size_t v = 0; v < samples.size(); ++v) {
    if (!whole(v)) continue;
    const double ms = median(samples[v].ms);
    if (best < 0 || ms < best_ms) { best = (int)v; best_ms = ms; }
  }
  if (best < 0 || (whole((size_t)without) && best_ms > 0.98 * median(samples[without].ms))) return without;
  return best;
}

}  // namespace sna
