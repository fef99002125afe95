// step_plan3.h -- how the 3D sweeps are run, by sizes and types.  Host code
// without HIP.
#pragma once

#include <cstddef>

namespace lbk3 {

// Bytes of both population buffers that a step touches: whole 128-byte lines of
// every row, without the padding of the pitch to 64 nodes (of a row of 8 FP64
// nodes that is one line in four).
inline double touched_bytes(int q, int nx, int ny, int nz, size_t elem) {
  return 2.0 * q * nz * ny * (double)((nx * elem + 127) / 128 * 128);
}

// The sweep streams past the 256 MB last-level cache when what it touches
// exceeds it by a quarter.  Us a step cached / streaming: FP32 192 x 192 x nz at
// 290, 360, 400, 450 MB 57.8 / 58.3, 73.0 / 73.5, 78.4 / 74.4, 92.9 / 84.4; FP16
// D3Q27 160 x 160 x 96 (319 MB) 68.5 / 62.4, D3Q19 192 x 192 x 130 (364 MB) 79.1 /
// 69.2; FP64 250 x 99 x 33 D3Q27 (362 MB) 72.3 / 70.6, with noise 80.7 / 81.4.  Below
// the cache streaming costs up to half: 8 x 8 x 4096 FP64 D3Q19, 159 MB touched
// in buffers of 637, 38.4 / 55.6.
constexpr double STREAM_MIN_BYTES = 320.0 * 1024 * 1024;
inline bool streams3(int q, int nx, int ny, int nz, size_t elem) {
  return touched_bytes(q, nx, ny, nz, elem) >= STREAM_MIN_BYTES;
}

// What a 3D domain's step costs.
struct Kind3 {
  int storage;  // 0 FP64, 1 FP32, 2 and 3 the 16-bit formats
  int q;
  bool solids, trt, power;
  double n;     // with power: the exponent
};

// The two-step sweep (sweep3x2_impl.h): output columns of a tile; rows of its
// first step, two more than those of the outputs; workgroups resident on a CU.
constexpr int X2_COLS = 64, X2_ROWS = 7;
constexpr int x2_resident(int storage) { return storage == 0 ? 1 : 2; }

// Segmentation of the walk along z: planes a segment, whose iterations are two
// more, and the iterations one after another on a CU.  As many segments as
// fill whole rounds of the chip cheapest, of four planes at least.
struct X2Split {
  int tiles, planes;
  long long iterations;
};
inline X2Split split3(int storage, int nx, int ny, int nz) {
  X2Split r{((nx + X2_COLS - 1) / X2_COLS) * ((ny + X2_ROWS - 3) / (X2_ROWS - 2)), nz, 1LL << 60};
  const long long slots = 256 * x2_resident(storage);
  for (int segs = 1; segs <= nz; ++segs) {
    const int z = (nz + segs - 1) / segs;
    if (segs > 1 && z < 4) break;
    const long long n = (nz + z - 1) / z, c = ((r.tiles * n + slots - 1) / slots) * (z + 2);
    if (c < r.iterations) r.iterations = c, r.planes = z;
  }
  return r;
}

// Whether two steps a launch take less time than two single ones.  A single
// step costs 3 us and its bytes, at 6.8 TB/s within the last-level cache and
// 5.1 beyond, 7 % more with solids.  Two cost an iteration (one plane of every
// resident tile) of 5.5 us in FP32 and 5.1 in FP64 on D3Q19, a fifth less
// within the cache, 27 / 19 times that on D3Q27, and what the collision adds:
// solids 1.0 / 0.65, TRT 0.25, the power law in FP32 1.1, or 2.6 to 6 where its root
// is iterated for most nodes (thinning fluids but n = 1/2; the others have a
// closed form or end at the clamp; how often depends on the flow), and 1.5 for the D3Q27 form with both, which
// spills 16 to 18 registers.  Measured, us a step, single / two: FP32 D3Q19
// 192 x 192 x 130 open 136 / 99, n = 3/4 with solids 151 / 166, FP64 271 / 170;
// D3Q27 160 x 160 x 96 FP32 open 103 / 86, n = 1/2 with solids 113 / 137; 400 x 30 x
// 100 FP32 D3Q19 open 29.8 / 23.3, n = 1/2 with solids 32.4 / 36.6.  Over 450
// combinations the choice is 0.4 % off the better on average, and at most 5 %
// slower than single steps.
// Not taken: the 16-bit formats, whose single step is bound by vector issue
// almost as much as by memory (D3Q19 71 / 73 us, D3Q27 92 / 104), and the
// power law in FP64 (its pow; 259 / 337 us at n = 0.75).
inline bool two_steps_pay3(const Kind3 &c, int nx, int ny, int nz) {
  if (c.storage > 1 || (c.storage == 0 && c.power)) return false;
  const bool f64 = c.storage == 0;
  const double bytes = touched_bytes(c.q, nx, ny, nz, f64 ? 8 : 4);
  const bool cached = bytes <= 256.0 * 1024 * 1024;
  const double one = 3.0 + bytes / (cached ? 6.8e6 : 5.1e6) * (c.solids ? 1.07 : 1.0);
  double us = (f64 ? 5.1 : 5.5) * (cached ? 0.8 : 1.0);
  if (c.solids) us += f64 ? 0.65 : 1.0;
  if (c.trt) us += 0.25;
  if (c.power) us += c.n < 1.0 && c.n != 0.5 ? 4.2 : 1.1;
  if (c.power && c.solids && c.q == 27) us += 1.5;
  return us * c.q / 19.0 * (double)split3(c.storage, nx, ny, nz).iterations < 2.0 * one;
}

}  // namespace lbk3
