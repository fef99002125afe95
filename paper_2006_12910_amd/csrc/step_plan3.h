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

}  // namespace lbk3
