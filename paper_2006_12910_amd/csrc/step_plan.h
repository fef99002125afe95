// step_plan.h -- how the steps of a call are split into launches: the regions
// of the launches of several steps (sweepn_impl.h), what a launch costs, and
// the choice between them.  Host code without HIP (the constants are the
// kernels' too).
#pragma once

#include <algorithm>
#include <cmath>
#include <utility>
#include <vector>

namespace lbk {

enum : int { ST_F64 = 0, ST_F32 = 1, ST_F16 = 2, ST_BF16 = 3 };

// Power-law exponent specialisations.
enum : int { PL_GENERIC = 0, PL_HALF = 1, PL_3Q = 2, PL_3H = 3 };

// Regions of the launches of several steps: columns, rows, threads (a whole
// number of nodes each).  The small
// one has the shortest step (one node a thread, two waves a SIMD) and the
// most tiles; the middle one fills a CU with two workgroups; the large one has
// the least rim, and suits the formats whose LDS leaves room for two.
struct Region {
  int cw, rs, nt;
};
constexpr int REGIONS = 3;
constexpr Region region(int k) {
  return k == 0 ? Region{32, 16, 512} : (k == 1 ? Region{32, 32, 512} : Region{64, 32, 512});
}
// the large region of 8-byte values would take 147 KB of LDS
constexpr bool region_fits(int storage, int k) { return !(storage == ST_F64 && k == 2); }
constexpr int MULTI_MAX = 9;  // most steps a launch takes

// What a domain's collision costs.
struct StepKind {
  int storage;
  bool noise, power;
  int plm;  // with power
};

// Time of a launch of n steps (odd; 1: the single-step sweep) by the model, and
// its region (of one step: 0, or else the single-step sweep); no such launch
// where the time is NEVER.
constexpr double NEVER = 1e300;
struct MultiPlan {
  double us[MULTI_MAX + 1];
  int k[MULTI_MAX + 1] = {};
  MultiPlan() { std::fill(us, us + MULTI_MAX + 1, NEVER); }
};

using Sizes = std::vector<std::pair<int, int>>;  // nx, ny of every domain of a launch

inline int multi_tiles(int k, int n, int nx, int ny) {
  const int ow = region(k).cw - 2 * (n - 1), oh = region(k).rs - 2 * (n - 1);
  return ((nx + ow - 1) / ow) * ((ny + oh - 1) / oh);
}

// Time of a wave-row (one step of 64 nodes) in us of one CU's vector issue.
// n = 1/2 has a closed form, the others iterate: n = 3/4 five times or so with
// a square root of a square root each; thickening fluids (3/2) mostly end at the
// clamp; the generic one calls pow, in FP64 a hundred instructions.
inline double wave_row_us(const StepKind &c) {
  const int s = std::min(c.storage, (int)ST_F16);
  constexpr double plain[3] = {0.069, 0.0525, 0.060}, noise[3] = {0.141, 0.050, 0.059};
  constexpr double power[4][3] = {{0.245, 0.036, 0.034}, {0.070, 0.038, 0.039}, {0.278, 0.167, 0.167},
                                  {0.070, 0.038, 0.039}};
  return plain[s] + (c.noise ? noise[s] : 0.0) + (c.power ? power[c.plm][s] : 0.0);
}

// Time of a launch of n steps over region k in us, or of a single step (n = 1,
// whatever k).  A launch costs 4.7 us from its first load to its last store,
// and then the most of
//  * the chain of its steps in one workgroup: n (6.2, 20, 31) wave-rows;
//  * what the busiest CU issues and what the tiles read and write together, as
//    they overlap only in part: the root of the sum of their squares.  Bytes at
//    8.8 TB/s where the last-level cache holds both buffers, else at 5.3.
// A single step issues a quarter more (shorter runs of independent work; the
// noise is one long run in either), but overlaps the two better.
//
// Fitted to 700 combinations of format, collision and size from 128 x 64 to
// 4096^2, all regions and step counts, in sheared flow: 11 % rms.  The choice
// made by it is 1 % slower than the best of each on average, at worst 20 %
// (FP64 n = 1.3 at 300^2, 4.95 against 4.11 us a step).
inline double launch_us(const StepKind &c, int k, int n, const Sizes &sizes) {
  const double v = wave_row_us(c), bytes = c.storage == ST_F64 ? 8 : c.storage == ST_F32 ? 4 : 2;
  double nodes = 0.0, rows = 0.0;
  for (const auto &s : sizes) {
    nodes += (double)s.first * s.second;
    rows += (double)((s.first + 63) / 64) * s.second;
  }
  const double rate = 18 * bytes * nodes > 256e6 ? 5.3e6 : 8.8e6;  // bytes a us
  if (n == 1) {
    const double issue = (c.noise ? 1.05 : 1.25) * v * rows / 256.0, memory = 18 * bytes * nodes / rate;
    return 4.7 + std::cbrt(issue * issue * issue + memory * memory * memory);
  }
  constexpr double chain[REGIONS] = {6.2, 20.0, 31.0};
  const Region g = region(k);
  double tiles = 0.0, tile_rows = 0.0;
  for (const auto &s : sizes) tiles += multi_tiles(k, n, s.first, s.second);
  for (int s = 0; s < n; ++s) tile_rows += g.cw * (g.rs - 2 * s) / 64.0;
  // two workgroups of region 2 share a CU: one left over runs slower alone
  const double rounds = std::ceil(tiles / 256.0),
               busy = k == 2 ? 0.75 * rounds + 0.5 * std::ceil(tiles / 512.0) : rounds;
  const double moved = tiles * 9 * bytes * (g.cw * g.rs + (g.cw - 2 * (n - 1)) * (g.rs - 2 * (n - 1)));
  return 4.7 + std::max(n * chain[k] * v, std::hypot(busy * tile_rows * v, moved / rate));
}

// Whether the single steps of one domain run over region 0 too: as long as every
// tile has a CU of its own (up to 64 of them the launch also moves the counter
// on, k_multi_one), and up to 17 rounds of the chip and the last-level cache,
// unless more than a third of the rows of the tiles lie outside.  Us a call of
// one step, single-step sweep / region 0: 128 x 64 6.5 / 4.0, 724 x 700 FP16 with
// noise 12.2 / 9.2, 1031 x 1000 FP64 23.3 / 22.4, 1448^2 FP16 16.6 / 15.9, 2048^2 FP16
// with noise 38.4 / 42.1; 20000 x 20 FP32 8.6 / 11.3.
inline bool single_in_region(const StepKind &c, int nx, int ny) {
  const double bytes = c.storage == ST_F64 ? 8 : c.storage == ST_F32 ? 4 : 2;
  const int tiles = multi_tiles(0, 1, nx, ny);
  return tiles <= 256 || (tiles <= 17 * 256 && 18 * bytes * nx * ny <= 256e6 &&
                          tiles * 8.0 <= 1.35 * ((nx + 63) / 64) * ny);
}

// The launches for the domains of one launch, each over the region that takes
// the least time.
inline MultiPlan plan_multi(const StepKind &c, const Sizes &sizes) {
  MultiPlan p;
  p.us[1] = launch_us(c, 0, 1, sizes);
  p.k[1] = sizes.size() == 1 && single_in_region(c, sizes[0].first, sizes[0].second) ? 0 : 1;
  for (int n = 3; n <= MULTI_MAX; n += 2)
    for (int k = 0; k < REGIONS; ++k) {
      if (!region_fits(c.storage, k) || std::min(region(k).cw, region(k).rs) - 2 * (n - 1) < 4) continue;
      const double t = launch_us(c, k, n, sizes);
      if (t < p.us[n]) p.us[n] = t, p.k[n] = k;
    }
  return p;
}

// c steps in parts of an odd number of steps each, the longest first: of lo,
// lo + 2 and, beside parts of three and one, five.
struct StepSplit {
  int parts, lo, longer, longest;
  int len(int i) const { return lo + (i < longest ? 4 : i < longest + longer ? 2 : 0); }
  double us(const MultiPlan &p) const {
    return (longest ? longest * p.us[lo + 4] : 0.0) + (longer ? longer * p.us[lo + 2] : 0.0) +
           (parts - longer - longest) * p.us[lo];
  }
};

// The cheapest of the splits into parts of at most 1, 3, .. steps, as few and as
// equal as each of those allows, and of the one into five, three and one in
// which two single steps and a part of three became one of five.  Single steps
// alone where nothing is less: 16-bit formats with noise on lattices that fill
// the chip issue no fewer instructions in a tile than in a single step, and the
// rim comes on top (FP16 2048^2: 41.3 us a step against 38.4).  The five pays for
// FP16 with obstacles at 2048^2, 116 us against 133, but not with noise, 226
// against 204 (always taken it gained 2.5 % on 32 steps of 24 FP16 domains, and
// lost 15 % of 8 steps with noise or a power law).
inline StepSplit split_steps(int c, const MultiPlan &p) {
  StepSplit best{};
  double least = 2 * NEVER;
  auto take = [&](const StepSplit &r) {
    const double t = r.us(p);
    if (t < least) least = t, best = r;
  };
  for (int n = 1; n <= MULTI_MAX; n += 2) {
    if (!(p.us[n] < NEVER)) break;
    StepSplit r{(c + n - 1) / n, 0, 0, 0};
    if ((r.parts ^ c) & 1) ++r.parts;
    r.lo = c / r.parts;
    if (!(r.lo & 1)) --r.lo;
    r.longer = (c - r.parts * r.lo) / 2;
    take(r);
    if (n == 3 && r.lo == 1 && p.us[5] < NEVER) {
      r.longest = std::min(r.longer, (r.parts - r.longer) / 2);
      r.parts -= 2 * r.longest;
      r.longer -= r.longest;
      take(r);
    }
  }
  return best;
}

}  // namespace lbk
