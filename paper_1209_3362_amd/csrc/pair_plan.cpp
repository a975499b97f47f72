// Launch planning of the pair kernel (see pair_plan.hpp).
#include "pair_plan.hpp"

#include <algorithm>
#include <limits>

namespace nfs {
namespace {
constexpr int kCus = 256;  // of a GPU
size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
}  // namespace

int pair_simd_load(int count, int waves) {
  const int base = count / waves, extra = count % waves;
  int worst = 0;
  for (int simd = 0; simd < 4; ++simd) {
    int load = 0;
    for (int w = simd; w < waves; w += 4) load += base + (w < extra ? 1 : 0);
    worst = std::max(worst, load);
  }
  return worst;
}

bool plan_group(const std::vector<int32_t>& lags, int first, int count,
                       LagGroup* g) {
  g->first = first;
  g->count = count;
  g->max_lag = lags[first + count - 1];
  g->modes = 0;
  // Two workgroups per CU hide each other's barrier and LDS waits: the first
  // choice is 16 modes per workgroup with LDS for two workgroups, then 16 or
  // 8 modes with LDS for one (the 8-wave kernels with 16 or 8 modes fit the
  // registers of two workgroups per CU).
  const int S = kPairChunk;
  const int H = int(round_up(size_t(g->max_lag + 2 * S), S));
  const struct { int K; size_t budget; } choices[] = {
      {16, size_t(kLdsBytes) / 2}, {16, size_t(kLdsBytes)}, {8, size_t(kLdsBytes)}};
  for (const auto& ch : choices) {
    const size_t lds = size_t(H + kPairMirror) * ch.K * 8;
    if (lds <= ch.budget) {
      g->modes = ch.K;
      g->hist = H;
      g->lds = lds;
      break;
    }
  }
  if (!g->modes) return false;
  // The lags are split over W waves in contiguous slices whose lengths
  // differ by at most one; waves w, w + 4, w + 8 share a SIMD, so pick the
  // W whose busiest SIMD has the fewest lags; ties go to more waves (more
  // waves per SIMD hide each other's LDS and barrier waits: measured on
  // 32-lag groups with one and with two workgroups per CU).
  int best_w = 0, best_cost = std::numeric_limits<int>::max();
  for (int W = 1; W <= kMaxPairWaves; ++W) {
    const int per = (count + W - 1) / W;
    if (per > kMaxLagsPerWave) continue;
    // Workgroups of 12 waves are built for 6 or more lags per wave only.
    if (W > 8 && per < 6) continue;
    const int cost = pair_simd_load(count, W);
    if (cost <= best_cost) {
      best_cost = cost;
      best_w = W;
    }
  }
  g->waves = best_w;
  g->per_wave = best_w ? (count + best_w - 1) / best_w : 0;
  return best_w > 0;
}

std::vector<LagGroup> group_candidates(const std::vector<int32_t>& lags, int first, int count) {
  std::vector<LagGroup> out;
  const int S = kPairChunk;
  const int max_lag = lags[first + count - 1];
  const int H = int(round_up(size_t(max_lag + 2 * S), S));
  for (int K : {16, 8}) {
    const size_t lds = size_t(H + kPairMirror) * K * 8;
    if (lds > size_t(kLdsBytes)) continue;
    for (int W = 1; W <= kMaxPairWaves; ++W) {
      const int per = (count + W - 1) / W;
      if (per > kMaxLagsPerWave) continue;
      if (W > 8 && per < 6) continue;
      LagGroup g;
      g.first = first;
      g.count = count;
      g.max_lag = max_lag;
      g.modes = K;
      g.hist = H;
      g.lds = lds;
      g.waves = W;
      g.per_wave = per;
      out.push_back(g);
    }
  }
  return out;
}

// Where the lines lie (pair sums, history kernel against this one, us; 512 x 512
// frames unless stated). Up to 200 frames this one is never slower: 32 frames and
// 31 lags 67 / 40, 96 and 16 70 / 47, 192 and 32 160 / 130, 96 frames of 2048 x
// 2048 and 16 lags 1021 / 594. Beyond, its loads are a larger part and the
// history kernel overlaps them with the sums: 5 lags over 400 frames 118 / 139,
// 7 over 600 162 / 181, 56 over 500 422 / 471, but 16 over 500 222 / 168 and 32
// over 600 373 / 330; so it takes up to 4 and 9 to 48 lags there (to 40 and from
// 150 frames where a launch has few workgroups: 256 x 256, 48 lags over 298
// frames 51 / 57) and any number where the history leaves the other kernel one
// workgroup per CU (5 lags up to 300 over 600 frames 251 / 160). From 640 frames
// on two workgroups no longer fit a CU: 900 and 16 387 / 538.
// Frames of up to 128 x 128 have fewer workgroups than the chip holds, so the
// waves of one decide: 31 lags over 64 frames of 128 x 128 10 / 14 (10 with 8
// waves), of 256 x 256 25 / 19.
// 32 modes per workgroup read rows in pieces of 256 bytes and waste fewer masked
// targets, as long as four workgroups fit a CU: 64 frames and 32 lags 50 / 72
// us with 32 / 16 modes, 192 frames and 32 lags 198 / 132; with few lags the
// line lies lower (130 frames of 2048 x 2048: 4 lags 445 / 387, 16 702 / 909).
// 8 waves where fewer than four workgroups fit a CU or share it: 448 frames and
// 16 lags 182 / 261 with 8 / 4, 192 frames 109 / 95.
bool window_shape(const LagGroup& group, int64_t n_modes, int64_t T0, int64_t T1,
                  WindowShape* w) {
  if (group.modes == 0 || n_modes < 64 * kCus) return false;
  const int count = group.count;
  w->n_lags = count;
  w->pre = int(std::min<int64_t>(group.max_lag, T0));
  const int64_t rows = w->pre + (T1 - T0);
  if (rows > 640) return false;
  w->modes = rows <= 112 || (rows <= 150 && count > 8) ? 32 : 16;
  const int per_block = 8 * (64 / w->modes);
  const int blocks = int((T1 - T0 + per_block - 1) / per_block);
  const size_t hist = size_t(rows + kWinGuard) * size_t(w->modes) * 8;
  const int64_t at_once = int64_t(kCus) * int64_t(size_t(kLdsBytes) / hist);
  const bool few = (n_modes + w->modes - 1) / w->modes < 2 * at_once;
  if (rows > (few ? 150 : 200) && ((count > 4 && count < 9) || count > (few ? 40 : 48)) &&
      2 * group.lds <= size_t(kLdsBytes))
    return false;
  w->waves = w->modes == 16 && (hist > size_t(kLdsBytes) / 4 || few) ? 8 : 4;
  // The split of the sums with the shortest busiest wave, in units of one lag of
  // one block: 0.4 for a block's target rows, 1 + 0.5 per lag for a task's set-up
  // and the sums it leaves.
  double best = 0.0;
  const int fewest = (group.count + kWinLags - 1) / kWinLags;
  for (int sets = fewest; sets <= std::min(group.count, fewest + w->waves - 1); ++sets)
    for (int slices = 1; slices <= std::min(blocks, w->waves); ++slices) {
      const int per = (group.count + sets - 1) / sets;
      const double task = 1.0 + 0.5 * per + ((blocks + slices - 1) / slices) * (0.4 + per);
      const double cost = ((sets * slices + w->waves - 1) / w->waves) * task;
      if (best == 0.0 || cost < best) {
        best = cost;
        w->sets = sets;
        w->slices = slices;
      }
    }
  w->lds = hist + size_t(w->slices) * size_t(w->modes) * size_t(group.count) * 4;
  return w->lds <= size_t(kLdsBytes) / 2;
}

}  // namespace nfs
