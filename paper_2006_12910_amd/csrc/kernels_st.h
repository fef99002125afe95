// kernels_st.h -- instantiates the kernels of one storage format (LBK_ST) and
// exposes them through a KernelSet.  Included once per kern_*.hip file so the
// formats compile in parallel.
#pragma once

#include "aux_impl.h"
#include "discn_impl.h"
#include "launch.h"
#include "particles_impl.h"
#include "sweep_impl.h"
#include "sweepn_impl.h"

namespace lbk {
namespace {

constexpr int ST = LBK_ST;

template <int FEAT, int PLM, int WIDE>
void sweep_l(const DevDomain *doms, const int *prefix, int ndom, int kstep, int blocks, int part,
             hipStream_t s) {
  hipLaunchKernelGGL((k_sweep<ST, FEAT, PLM, WIDE>), dim3(blocks), dim3(256), 0, s, doms, prefix,
                     ndom, kstep, part);
}
template <int FEAT, int PLM>
void multi_one_l(const DevDomain *one, uint32_t *arrived, int kstep, int nsteps, int advance, int blocks,
                 hipStream_t s) {
  hipLaunchKernelGGL((k_multi_one<ST, FEAT, PLM, 0>), dim3(blocks), dim3(region(0).nt), 0, s, *one,
                     arrived, kstep, nsteps, advance);
}
template <int FEAT, int PLM>
void multi_l(const DevDomain *doms, const int *prefix, int ndom, int k, int kstep, int nsteps, int blocks,
             hipStream_t s) {
  if (k == 0) {
    hipLaunchKernelGGL((k_multi<ST, FEAT, PLM, 0>), dim3(blocks), dim3(multi_threads(ST, 0, FEAT)), 0, s, doms,
                       prefix, ndom, kstep, nsteps);
  } else if (k == 1 || !region_fits(ST, 2)) {
    hipLaunchKernelGGL((k_multi<ST, FEAT, PLM, 1>), dim3(blocks), dim3(multi_threads(ST, 1, FEAT)), 0, s, doms,
                       prefix, ndom, kstep, nsteps);
  } else {
    if constexpr (region_fits(ST, 2))
      hipLaunchKernelGGL((k_multi<ST, FEAT, PLM, 2>), dim3(blocks), dim3(multi_threads(ST, 2, FEAT)), 0, s, doms,
                         prefix, ndom, kstep, nsteps);
  }
}
template <int FEAT, int PLM>
void multi_disc_l(const DevDomain *doms, const int *prefix, int ndom, const PItem *items, int nitems,
                  const DevDomain *one, int kstep, int blocks, hipStream_t s) {
  constexpr int K = disc_region(ST);
  static const DevDomain none{};
  hipLaunchKernelGGL((k_multi_disc<ST, FEAT, PLM, K>), dim3(nitems + blocks), dim3(region(K).nt), 0, s,
                     doms, prefix, ndom, items, nitems, one != nullptr ? *one : none, kstep);
}
template <int FEAT, int PLM, int WIDE>
void init_l(const DevDomain *dom, const double *rho, const double *ux, const double *uy, int row0,
            int nrows, int pitch, hipStream_t s) {
  const long long n = (long long)nrows * pitch;
  hipLaunchKernelGGL((k_init<ST, FEAT, PLM, WIDE>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     dom, rho, ux, uy, row0, nrows);
}

#ifndef LBK_GENERIC_POWER_FILE
void pre_l(const DevDomain *doms, const PItem *items, int nitems, int kstep, hipStream_t s) {
  hipLaunchKernelGGL((k_pre<ST>), dim3(nitems), dim3(PT), 0, s, doms, items, kstep);
}
void post_l(const DevDomain *doms, const PItem *items, int nitems, int kstep, hipStream_t s) {
  hipLaunchKernelGGL((k_post<ST>), dim3(nitems), dim3(PT), 0, s, doms, items, kstep);
}
void post_pre_l(const DevDomain *doms, const PItem *items, int nitems, int kstep, hipStream_t s) {
  hipLaunchKernelGGL((k_post_pre<ST>), dim3(nitems), dim3(PT), 0, s, doms, items, kstep);
}
void mass_l(const DevDomain *doms, const int *prefix, int ndom, int blocks, double *alt,
            hipStream_t s) {
  hipLaunchKernelGGL((k_mass_partial<ST>), dim3(blocks), dim3(256), 0, s, doms, prefix, ndom, alt);
}
void moments_l(const DevDomain &dom, double *rho, double *ux, double *uy, int row0, int nrows,
               hipStream_t s) {
  const long long n = (long long)nrows * dom.nx;
  hipLaunchKernelGGL((k_moments<ST>), dim3((unsigned)((n + 511) / 512)), dim3(256), 0, s, dom, rho, ux,
                     uy, row0, nrows);
}
void export_l(const DevDomain *dom, double *out, int row0, int nrows, int nx, hipStream_t s) {
  const long long n = (long long)nrows * nx;
  hipLaunchKernelGGL((k_export<ST>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dom, out,
                     row0, nrows);
}
void import_l(const DevDomain *dom, const double *in, int row0, int nrows, int nx,
              hipStream_t s) {
  const long long n = (long long)nrows * nx;
  hipLaunchKernelGGL((k_import<ST>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dom, in,
                     row0, nrows);
}

void mirror_l(const DevDomain *dom, int nx, int ny, hipStream_t s) {
  const long long n = (long long)nx * ny;
  hipLaunchKernelGGL((k_mirror<ST>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dom);
}
#endif

// The kernels that collide.
template <int FEAT, int PLM, int WIDE> void fill_steps(KernelSet *k) {
  k->sweep = sweep_l<FEAT, PLM, WIDE>;
  // several steps a launch: every set in native arithmetic but the power law
  // without a label plane or with noise
  k->multi = nullptr;
  k->multi_one = nullptr;
  if constexpr (WIDE == 0 && ((FEAT & F_POWER) == 0 ||
                              ((FEAT & F_LABELS) != 0 && (FEAT & F_NOISE) == 0))) {
    k->multi = multi_l<FEAT, PLM>;
    k->multi_one = multi_one_l<FEAT, PLM>;
  }
  k->multi_disc = nullptr;
  if constexpr (WIDE == 0 && (FEAT & F_LABELS) != 0 && !((FEAT & F_POWER) != 0 && (FEAT & F_NOISE) != 0))
    k->multi_disc = multi_disc_l<FEAT, PLM>;
  k->init = init_l<FEAT, PLM, WIDE>;
}

#ifndef LBK_GENERIC_POWER_FILE

void fill_rest(KernelSet *k) {
  k->pre = pre_l;
  k->post = post_l;
  k->post_pre = post_pre_l;
  k->mass_partial = mass_l;
  k->moments = moments_l;
  k->export_f = export_l;
  k->import_f = import_l;
  k->mirror = mirror_l;
}

template <int FEAT, int PLM, int WIDE> void fill(KernelSet *k) {
  fill_steps<FEAT, PLM, WIDE>(k);
  fill_rest(k);
}

template <int BASE, int WIDE> bool pick_power(int feat, int plm, KernelSet *k) {
  if (!(feat & F_POWER)) { fill<BASE, PL_GENERIC, WIDE>(k); return true; }
  switch (plm) {
#ifdef LBK_GENERIC_POWER
    case PL_GENERIC: fill_rest(k); return LBK_GENERIC_POWER(feat, k);
#else
    case PL_GENERIC: fill<BASE | F_POWER, PL_GENERIC, WIDE>(k); return true;
#endif
    case PL_HALF: fill<BASE | F_POWER, PL_HALF, WIDE>(k); return true;
    case PL_3Q: fill<BASE | F_POWER, PL_3Q, WIDE>(k); return true;
    case PL_3H: fill<BASE | F_POWER, PL_3H, WIDE>(k); return true;
  }
  return false;
}

template <int WIDE> bool pick(int feat, int plm, KernelSet *k) {
  switch (feat & (F_LABELS | F_NOISE | F_TRT)) {
    case 0: return pick_power<0, WIDE>(feat, plm, k);
    case F_LABELS: return pick_power<F_LABELS, WIDE>(feat, plm, k);
    case F_NOISE: return pick_power<F_NOISE, WIDE>(feat, plm, k);
    case F_LABELS | F_NOISE: return pick_power<F_LABELS | F_NOISE, WIDE>(feat, plm, k);
    case F_TRT: return pick_power<F_TRT, WIDE>(feat, plm, k);
    case F_LABELS | F_TRT: return pick_power<F_LABELS | F_TRT, WIDE>(feat, plm, k);
  }
  return false;  // TRT with noise is refused at validation
}

#endif  // LBK_GENERIC_POWER_FILE

}  // namespace

#ifndef LBK_GENERIC_POWER_FILE
bool LBK_GETTER(int feat, int plm, int wide, KernelSet *k) {
  if (ST == ST_F64 || !wide) return pick<0>(feat, plm, k);
  return pick<1>(feat, plm, k);
}
#else
// The kernels that collide with the power law of any exponent.
bool LBK_GETTER(int feat, KernelSet *k) {
  switch (feat & (F_LABELS | F_NOISE | F_TRT)) {
    case 0: fill_steps<F_POWER, PL_GENERIC, 0>(k); return true;
    case F_LABELS: fill_steps<F_POWER | F_LABELS, PL_GENERIC, 0>(k); return true;
    case F_NOISE: fill_steps<F_POWER | F_NOISE, PL_GENERIC, 0>(k); return true;
    case F_LABELS | F_NOISE: fill_steps<F_POWER | F_LABELS | F_NOISE, PL_GENERIC, 0>(k); return true;
    case F_TRT: fill_steps<F_POWER | F_TRT, PL_GENERIC, 0>(k); return true;
    case F_LABELS | F_TRT: fill_steps<F_POWER | F_LABELS | F_TRT, PL_GENERIC, 0>(k); return true;
  }
  return false;
}
#endif

}  // namespace lbk
