// kern3_st.h -- instantiates the single-step 3D sweeps of one storage format
// (LBK3_ST) and launches them.  Included once per kern3_*.hip file so the
// formats compile in parallel.
#pragma once

#include "launch3.h"

namespace lbk3 {
namespace {

constexpr int ST = LBK3_ST;

struct Call {
  const Dom3 *dd;
  bool wide;
  unsigned blocks;
  int k;
  hipStream_t s;
};

template <bool SOLIDS, int Q, bool PL, int NZ> void go_mode(const Dom3 &h, const Call &c) {
  const dim3 g(c.blocks), b(256);
  if (c.wide)
    hipLaunchKernelGGL((k_sweep3<ST, SOLIDS, M3_WIDE, Q, PL, NZ>), g, b, 0, c.s, c.dd, c.k);
  else if (h.stream)
    hipLaunchKernelGGL((k_sweep3<ST, SOLIDS, M3_STREAM, Q, PL, NZ>), g, b, 0, c.s, c.dd, c.k);
  else
    hipLaunchKernelGGL((k_sweep3<ST, SOLIDS, M3_CACHED, Q, PL, NZ>), g, b, 0, c.s, c.dd, c.k);
}
template <int Q, bool PL, int NZ> void go_solids(const Dom3 &h, const Call &c) {
  if (h.nodew) go_mode<true, Q, PL, NZ>(h, c);
  else go_mode<false, Q, PL, NZ>(h, c);
}
template <int Q, bool PL> void go_noise(const Dom3 &h, const Call &c) {
  // noise kind: none, with BGK, with TRT (the last needs more registers)
  if (!h.noise) go_solids<Q, PL, 0>(h, c);
  else if (h.trt) go_solids<Q, PL, 2>(h, c);
  else go_solids<Q, PL, 1>(h, c);
}
template <int Q> void go_power(const Dom3 &h, const Call &c) {
  if (h.pl) go_noise<Q, true>(h, c);
  else go_noise<Q, false>(h, c);
}

}  // namespace

void LBK3_ENTRY(const Dom3 &h, const Dom3 *dd, int q, bool wide, unsigned blocks, int kstep,
                hipStream_t s) {
  const Call c{dd, wide, blocks, kstep, s};
  if (q == 27) go_power<27>(h, c);
  else go_power<19>(h, c);
}

}  // namespace lbk3
