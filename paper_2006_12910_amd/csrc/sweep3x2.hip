// The two-step 3D sweep: instantiations and launch.
#include "launch3.h"
#include "sweep3x2_impl.h"

namespace lbk3 {
namespace {

template <int ST, bool SOLIDS, int Q, bool PL, int TR>
void go(const Dom3 &h, int planes, int kstep, int which, hipStream_t s) {
  const int tiles = ((h.nx + X2_COLS - 1) / X2_COLS) * ((h.ny + X2_ROWS - 3) / (X2_ROWS - 2));
  const dim3 g((unsigned)(tiles * ((h.nz + planes - 1) / planes))), b(64 * (X2_ROWS + 1));
  // registers: two workgroups a CU in FP32, one in FP64.  No form spills but
  // FP32 D3Q27 with the power law and solids, 16 to 18 of them.
  hipLaunchKernelGGL((k_sweep3x2<ST, SOLIDS, Q, PL, TR, X2_ROWS, 2 * x2_resident(ST)>), g, b, 0, s, h, kstep,
                     which, planes);
}

template <int ST, int Q, bool PL> void go_kind(const Dom3 &h, int planes, int kstep, int which, hipStream_t s) {
  if (h.nodew) {
    if (h.trt) go<ST, true, Q, PL, 1>(h, planes, kstep, which, s);
    else go<ST, true, Q, PL, 0>(h, planes, kstep, which, s);
  } else {
    if (h.trt) go<ST, false, Q, PL, 1>(h, planes, kstep, which, s);
    else go<ST, false, Q, PL, 0>(h, planes, kstep, which, s);
  }
}
template <int ST, int Q> void go_st(const Dom3 &h, int planes, int kstep, int which, hipStream_t s) {
  if constexpr (ST == 1) {
    if (h.pl) return go_kind<ST, Q, true>(h, planes, kstep, which, s);
  }
  go_kind<ST, Q, false>(h, planes, kstep, which, s);
}

}  // namespace

void launch_sweep3x2(const Dom3 &h, int q, int planes, int kstep, int which, hipStream_t s) {
  if (h.storage == 0) {
    if (q == 27) go_st<0, 27>(h, planes, kstep, which, s);
    else go_st<0, 19>(h, planes, kstep, which, s);
  } else {
    if (q == 27) go_st<1, 27>(h, planes, kstep, which, s);
    else go_st<1, 19>(h, planes, kstep, which, s);
  }
}

}  // namespace lbk3
