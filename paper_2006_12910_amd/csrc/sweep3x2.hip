// The two-step 3D sweep: instantiations and launch.
#include "launch3.h"
#include "sweep3x2_impl.h"

namespace lbk3 {
namespace {

// Rows of a tile's first step, and workgroups resident on a CU (waves per
// SIMD the registers are bounded to; both leave no spills).
constexpr int X2_ROWS = 7;
constexpr int x2_waves(int st) { return st == 0 ? 2 : 4; }

// Segmentation of the walk along z: workgroups, planes a segment (its
// iterations are two more), and rounds of the chip's 256 CUs.  As many
// segments as fill whole rounds cheapest, of four planes at least.
struct X2Split {
  int tiles, sz;
  long long iterations;  // one after another on a CU
};
X2Split split(const Dom3 &h) {
  X2Split r;
  r.tiles = ((h.nx + X2_COLS - 1) / X2_COLS) * ((h.ny + X2_ROWS - 3) / (X2_ROWS - 2));
  r.sz = h.nz;
  r.iterations = 1LL << 60;
  const long long slots = 256 * (x2_waves(h.storage) / 2);
  for (int segs = 1; segs <= h.nz; ++segs) {
    const int z = (h.nz + segs - 1) / segs;
    if (segs > 1 && z < 4) break;
    const long long n = (h.nz + z - 1) / z, c = ((r.tiles * n + slots - 1) / slots) * (z + 2);
    if (c < r.iterations) r.iterations = c, r.sz = z;
  }
  return r;
}

template <int ST, bool SOLIDS, int Q, bool PL, int TR>
void go(const Dom3 &h, int kstep, int which, hipStream_t s) {
  const X2Split p = split(h);
  const int tiles = p.tiles, sz = p.sz;
  const dim3 g((unsigned)(tiles * ((h.nz + sz - 1) / sz))), b(64 * (X2_ROWS + 1));
  hipLaunchKernelGGL((k_sweep3x2<ST, SOLIDS, Q, PL, TR, X2_ROWS, x2_waves(ST)>), g, b, 0, s, h, kstep,
                     which, sz);
}

template <int ST, int Q, bool PL> void go_kind(const Dom3 &h, int kstep, int which, hipStream_t s) {
  if (h.nodew) {
    if (h.trt) go<ST, true, Q, PL, 1>(h, kstep, which, s);
    else go<ST, true, Q, PL, 0>(h, kstep, which, s);
  } else {
    if (h.trt) go<ST, false, Q, PL, 1>(h, kstep, which, s);
    else go<ST, false, Q, PL, 0>(h, kstep, which, s);
  }
}
template <int ST, int Q> void go_st(const Dom3 &h, int kstep, int which, hipStream_t s) {
  if constexpr (ST == 1) {
    if (h.pl) return go_kind<ST, Q, true>(h, kstep, which, s);
  }
  go_kind<ST, Q, false>(h, kstep, which, s);
}

}  // namespace

// Both storage formats that take it, and their cost: an iteration (one plane
// of every resident tile) takes 6.8 us in FP32 on D3Q19 and 5.6 in FP64 (one
// workgroup a CU), 27 / 19 times that on D3Q27; a single step its bytes at 5
// TB/s and 3 us.  192 x 192 x 130, a step of the two-step sweep against the
// single one: FP32 91.8 / 127.6 us (D3Q19) and 137.7 / 190.5 (D3Q27), FP64
// 163 / 270 and 237 / 395; with solids, 256 x 160 x 128, FP32 122 / 164 and
// 181 / 244, FP64 203 / 311 and 289 / 433.  Small lattices are latency-bound
// walks: 96^3 FP32 26.2 / 24.7, 33 x 33 x 17 10.3 / 4.6.
// Not taken: the 16-bit formats, whose single step is bound by vector issue
// almost as much as by memory (D3Q19 71 / 73 us, D3Q27 104 / 92), and the
// power law in FP64 (its pow; 337 / 259 us at n = 0.75; FP32 106 / 127).
bool sweep3x2_pays(const Dom3 &h, int q) {
  if (h.storage > 1 || (h.storage == 0 && h.pl)) return false;
  const double us = (h.storage == 0 ? 5.6 : 6.8) * q / 19.0 * (double)split(h).iterations;
  const double bytes = 2.0 * q * (h.storage == 0 ? 8 : 4) * ((double)h.nx * h.ny * h.nz);
  return us < 2.0 * (bytes / 5e6 + 3.0);
}

void launch_sweep3x2(const Dom3 &h, int q, int kstep, int which, hipStream_t s) {
  if (h.storage == 0) {
    if (q == 27) go_st<0, 27>(h, kstep, which, s);
    else go_st<0, 19>(h, kstep, which, s);
  } else {
    if (q == 27) go_st<1, 27>(h, kstep, which, s);
    else go_st<1, 19>(h, kstep, which, s);
  }
}

}  // namespace lbk3
