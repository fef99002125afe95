// particles_impl.h -- particle coupling kernels (Sec. 3).
//
// Per step, for the state at time T (post-collision populations f*(T), labels
// G(T), particle state P(T)), two kernels with one workgroup per particle
// bracket the sweep:
//   k_pre    before the sweep: list the nodes of the particle's bounding box
//            with exterior pulls that cross its surface; for each such link
//            add the momentum exchange of Eq. MP1 and its torque (Eq. MP4) in
//            FP64 and write the moving-wall bounce-back (Eqs. MP7-MP8) into
//            the link's two pull slots, so the sweep pulls unconditionally;
//            the repulsion from solid nodes and from the
//            other particles (Eq. MP2, one lane per particle pair) is summed
//            beside it; then one lane takes the Newton-Euler step of Eqs.
//            MP5-MP6 into P(T+1).
//   k_post   after the sweep: the covered/uncovered-node force (Eq. MP3) of
//            the nodes whose label changes from G(T) to G(T+1), and G(T+1)
//            written into the label plane.
// Both are chains of dependent loads and FP64 steps on one workgroup: what
// counts is the length of the chain and the instructions a wave issues on it.
// 16 discs of R = 8 in 2048 x 1024: k_pre 11.7 -> 8.7 us, k_post 7.0 -> 6.2,
// from a list of single links that two block scans and one lane a link made,
// sums by shuffles, and a division in every periodic image.
// All reductions run in a fixed order, so results are bit-reproducible.
#pragma once

#include "lb_device.h"

namespace lbk {

constexpr int PT = 512;  // threads per particle
// The host admits no particle whose box side W = 2 reach + 2 has W^2 above
// 6144 (W <= 78), so the box with a one-node rim fits 80 x 80 labels.
constexpr int LAB_BOX = 80 * 80;
constexpr uint8_t LBL_OUT = 0xff;  // rim or box node outside a non-periodic domain

// v plus the value that a DPP move brings to the lane (zero where it brings none).
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, true);
  return v + __hiloint2double(hi, lo);
}

// Sum of NV values over the PT threads of a block, fixed order; result valid
// in every thread.  Within a wave by DPP moves (shifts within the rows of 16,
// then the rows' last lanes broadcast on), which cost a quarter of shuffles
// through LDS; lane 63 holds the wave's sum.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double (*scratch)[NV]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    v[k] = dpp_add<0x111, 0xf>(v[k]);  // row_shr 1, 2, 4, 8
    v[k] = dpp_add<0x112, 0xf>(v[k]);
    v[k] = dpp_add<0x114, 0xf>(v[k]);
    v[k] = dpp_add<0x118, 0xf>(v[k]);
    v[k] = dpp_add<0x142, 0xa>(v[k]);  // row_bcast 15, 31
    v[k] = dpp_add<0x143, 0xc>(v[k]);
  }
  if (lane == 63) {
#pragma unroll
    for (int k = 0; k < NV; ++k) scratch[w][k] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k)
    v[k] = ((scratch[0][k] + scratch[1][k]) + (scratch[2][k] + scratch[3][k])) +
           ((scratch[4][k] + scratch[5][k]) + (scratch[6][k] + scratch[7][k]));
  __syncthreads();
}

// Exclusive prefix sum of one int per thread over the first 256 threads of the
// block (fixed order).
__device__ __forceinline__ int block_exscan(int v, int *sh, int &total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63 && w < 4) sh[w] = incl;
  __syncthreads();
  int base = 0;
  for (int k = 0; k < min(w, 4); ++k) base += sh[k];
  total = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return base + incl - v;
}

// Map a box coordinate into the domain: any integer on a periodic axis (so a
// corrupted particle position can never index outside the planes), rejected
// outside a non-periodic axis.
__device__ __forceinline__ bool wrap_coord(int &v, int n, bool periodic) {
  if (v < 0 || v >= n) {
    if (!periodic) return false;
    v %= n;
    if (v < 0) v += n;
  }
  return true;
}

// Not inlined: pow's registers and constants would be taken for the whole of
// the kernels that rarely come here.
__device__ __attribute__((noinline)) double lj_power(double r) { return pow(r, -13.0); }

__device__ __forceinline__ double lj_mag(const DevDomain &D, double gap) {
  const double g = gap < D.lj_floor ? D.lj_floor : gap;
  return D.lj_psi * lj_power(g / D.lj_rit);
}

struct PDisc {
  double x, y, radius;
};

// One of two particle records, chosen field by field (a select of the whole
// record by a runtime condition would go through private memory).
__device__ __forceinline__ PState pick_state(bool second, const PState &a, const PState &b) {
  PState r;
  r.x = second ? b.x : a.x;
  r.y = second ? b.y : a.y;
  r.ux = second ? b.ux : a.ux;
  r.uy = second ? b.uy : a.uy;
  r.omega = second ? b.omega : a.omega;
  r.radius = second ? b.radius : a.radius;
  r.mass = second ? b.mass : a.mass;
  r.inertia = second ? b.inertia : a.inertia;
  r.rho_ratio = second ? b.rho_ratio : a.rho_ratio;
  r.fx = second ? b.fx : a.fx;
  r.fy = second ? b.fy : a.fy;
  r.torque = second ? b.torque : a.torque;
  r.flags = second ? b.flags : a.flags;
  r.pad = 0;
  r.pad2[0] = r.pad2[1] = r.pad2[2] = 0.0;
  return r;
}

// Repulsion on particle p from particle q (Eq. MP2), both from P(T): zero
// for q == p or beyond the interaction range.
__device__ __forceinline__ void pair_repulsion(const DevDomain &D, const PState &P,
                                               const PDisc &Q, double &lx, double &ly) {
  const bool perx = D.bc_x == BC_PERIODIC, pery = D.bc_y == BC_PERIODIC;
  const double dx = min_image(P.x - Q.x, D.nx, perx), dy = min_image(P.y - Q.y, D.ny, pery);
  const double dist = sqrt(dx * dx + dy * dy);
  const double gap = dist - P.radius - Q.radius;
  if (gap > D.lj_rit || !(dist > 0.0)) return;
  const double m = lj_mag(D, gap);
  lx += m * dx / dist;
  ly += m * dy / dist;
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Newton-Euler step (Eqs. MP5-MP6) of a particle: P(T+1) from its state
// P = P(T), its link, cover and solid-repulsion forces F and its
// particle-particle repulsion (lx, ly); with F_FAVG the update takes the mean
// of this step's total force and torque and the previous step's, which P(T)
// holds.  fast: the new velocity is outside what the coupling covers.  Called
// by whole waves, whose lanes hold the same values: the three divisions, of
// many instructions each, run in three lanes at once.
__device__ __forceinline__ PState newton_euler(const DevDomain &D, const PState &P, const PForce &F,
                                               double lx, double ly, bool &fast) {
  const bool perx = D.bc_x == BC_PERIODIC, pery = D.bc_y == BC_PERIODIC;
  const double fx = F.fx + F.cx_ + (lx + F.ljx);
  const double fy = F.fy + F.cy_ + (ly + F.ljy);
  const double tq = F.torque + F.ctorque;
  // optional: the mean of this and the previous step's totals (kept in P)
  const bool avg = (D.feat & F_FAVG) != 0;
  const double fxu = avg ? 0.5 * (fx + P.fx) : fx;
  const double fyu = avg ? 0.5 * (fy + P.fy) : fy;
  const double tqu = avg ? 0.5 * (tq + P.torque) : tq;
  PState N = P;
  N.fx = fx;
  N.fy = fy;
  N.torque = tq;
  fast = false;
  if (!(P.flags & 1)) {
    const double buoy = 1.0 - D.rho0 / (P.rho_ratio * D.rho0);
    const int lane = threadIdx.x & 63;
    const double q = (lane == 0 ? fxu : lane == 1 ? fyu : tqu) / (lane < 2 ? P.mass : P.inertia);
    N.ux = P.ux + lane_value(q, 0) + buoy * D.gx;
    N.uy = P.uy + lane_value(q, 1) + buoy * D.gy;
    N.omega = P.omega + lane_value(q, 2);
    N.x = P.x + P.ux;
    N.y = P.y + P.uy;
    if (perx) { if (N.x >= D.nx) N.x -= D.nx; if (N.x < 0.0) N.x += D.nx; }
    if (pery) { if (N.y >= D.ny) N.y -= D.ny; if (N.y < 0.0) N.y += D.ny; }
    fast = !(fabs(N.ux) < 0.5 && fabs(N.uy) < 0.5);
  }
  return N;
}

// Repulsion on a particle from the solid node (x, y) within lim of its centre.
__device__ __forceinline__ void solid_repulsion(const DevDomain &D, const PState &P, double lim, int x,
                                                int y, double &ljx, double &ljy) {
  const bool perx = D.bc_x == BC_PERIODIC, pery = D.bc_y == BC_PERIODIC;
  const double dx = min_image(P.x - x, D.nx, perx), dy = min_image(P.y - y, D.ny, pery);
  const double dist = sqrt(dx * dx + dy * dy);
  if (dist <= lim && dist > 0.0) {
    const double m = lj_mag(D, dist - P.radius);
    ljx += m * dx / dist;
    ljy += m * dy / dist;
  }
}

// The multiple of the period that min_image takes off d.
__device__ __forceinline__ double image_shift(double d, double len, bool periodic) {
  if (!periodic || fabs(d) < 0.49 * len) return 0.0;
  return len * floor(d / len + 0.5);
}

// j / w for box positions (j < 8192, w < 128), inv = 1.0f / w.
__device__ __forceinline__ int box_row(int j, float inv) { return (int)((j + 0.5f) * inv); }

// Exterior nodes with a link, box position and mask of the directions (bit
// i - 1: the pull along i comes out of the particle): those of an annulus of
// width sqrt(2) around the disc.
template <int CAP> struct LinkList {
  uint32_t rec[CAP];
  int count[PT / 64];
};

// The links of the particle P in its box of W x W nodes.  First every thread
// takes nodes of the box: mask(bi, bk) is a node's mask of links (and adds a
// solid node's repulsion); the nodes that have some are listed in a fixed
// order.  Then wave d takes the links along direction d + 1 of all of them,
// a lane each: most of the box has none, and a wave that met its few nodes in
// place would run the code of all eight directions for them (1.5 us more for
// three steps of a disc of R = 5).  For each link the momentum exchange and torque go onto acc[0 .. 2]
// and the bounce-back into its two slots: load(x, y, bi, bk, i, k) and put(...,
// v) are the value of direction i at the node (k = 0) or at its source x - e_k.
// A link's surface point is half a node from (x, y), a disc's radius from the
// centre, so both have the same periodic image.
template <int CAP, class Mask, class At, class Load, class Put>
__device__ __forceinline__ void box_links(const DevDomain &D, const PState &P, int W, int bx0, int by0,
                                          LinkList<CAP> &list, double (&acc)[7], Mask mask, At at,
                                          Load load, Put put) {
  const bool perx = D.bc_x == BC_PERIODIC, pery = D.bc_y == BC_PERIODIC;
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nbox = W * W;
  const float inv = 1.0f / (float)W;
  uint64_t m0 = 0, m1 = 0;  // masks of the thread's nodes, at most 12 (6144 / PT)
  int cnt = 0;
  for (int j = tid, it = 0; it * PT < nbox; j += PT, ++it) {
    uint32_t m = 0;
    if (j < nbox) {
      const int bk = box_row(j, inv);
      m = mask(j - bk * W, bk);
    }
    cnt += __popcll(__ballot(m != 0));
    if (it < 8) m0 |= (uint64_t)m << (8 * it);
    else m1 |= (uint64_t)m << (8 * (it - 8));
  }
  if (lane == 0) list.count[wave] = cnt;
  __syncthreads();
  int pos = 0, total = 0;
#pragma unroll
  for (int k = 0; k < PT / 64; ++k) {
    const int c = list.count[k];
    pos += k < wave ? c : 0;
    total += c;
  }
  for (int j = tid, it = 0; it * PT < nbox; j += PT, ++it) {
    const uint32_t m = (uint32_t)((it < 8 ? m0 >> (8 * it) : m1 >> (8 * (it - 8))) & 255u);
    const uint64_t b = __ballot(m != 0);
    const int mine = pos + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
    if (m && mine < CAP) list.rec[mine] = ((uint32_t)j << 8) | m;
    pos += __popcll(b);
  }
  __syncthreads();
  if (total > CAP && tid == 0) atomicOr(D.health, HEALTH_LINK_OVERFLOW);
  total = min(total, CAP);
  const int dir = wave + 1, o = opp(dir);
  const int dcx = cx(dir), dcy = cy(dir);
  const double w = dir <= 4 ? wgt<double>(1) : wgt<double>(5);
  for (int e = lane; e < total; e += 64) {
    const uint32_t rec = list.rec[e];
    if (!((rec >> wave) & 1u)) continue;
    const int j = (int)(rec >> 8), bk = box_row(j, inv), bi = j - bk * W;
    int x = bx0 + bi, y = by0 + bk;
    wrap_coord(x, D.nx, perx);
    wrap_coord(y, D.ny, pery);
    const auto here = at(x, y, bi, bk, 0, 0), so = at(x, y, bi, bk, dcx, dcy);
    const double a = load(here, o), b = load(so, dir);
    const double fopp = w * D.rho0 + a;
    const double sx = image_shift(x - P.x, D.nx, perx), sy = image_shift(y - P.y, D.ny, pery);
    const double rx = (x - 0.5 * dcx - P.x) - sx, ry = (y - 0.5 * dcy - P.y) - sy;
    const double vx = P.ux - P.omega * ry, vy = P.uy + P.omega * rx;
    const double ue = vx * dcx + vy * dcy;
    const double M = 6.0 * D.rho0 * w * ue;
    const double mag = 2.0 * fopp + M;
    const double dpx = -dcx * mag, dpy = -dcy * mag;
    acc[0] += dpx;
    acc[1] += dpy;
    acc[2] += rx * dpy - ry * dpx;
    put(so, dir, a + M);
    put(here, o, b - M);
  }
}

// Force and torque of a node (x, y) that the particle P covers (sign 1) or
// uncovers (-1), load(i) its populations' deviations, onto acc.
template <class Load>
__device__ __forceinline__ void cover_term(const DevDomain &D, const PState &P, int x, int y,
                                           double sign, double (&acc)[3], Load load) {
  const bool perx = D.bc_x == BC_PERIODIC, pery = D.bc_y == BC_PERIODIC;
  double drho = 0.0, jx = 0.0, jy = 0.0;
  for (int i = 0; i < 9; ++i) {
    const double v = load(i);
    drho += v;
    jx += v * cx(i);
    jy += v * cy(i);
  }
  const double rho = D.rho0 + drho;
  const double ux = jx / rho - 0.5 * D.gx, uy = jy / rho - 0.5 * D.gy;
  const double fx = sign * rho * (ux - P.ux), fy = sign * rho * (uy - P.uy);
  const double rx = min_image(x - P.x, D.nx, perx), ry = min_image(y - P.y, D.ny, pery);
  acc[0] += fx;
  acc[1] += fy;
  acc[2] += rx * fy - ry * fx;
}

// Before the sweep of step T -> T+1, one workgroup per particle p.
//
// Links: an exterior fluid node x and an interior node s = x - e_d of p.  The
// pull into x along d and the pull into s along -e_d both bounce off the
// surface point r_b = x - e_d/2 moving at u_b = U + Omega z x (r_b - r_c):
//   f_d(x)  <- f*_{-d}(x) + M,   f_{-d}(s) <- f*_d(s) - M,   M = 6 rho0 w_d (u_b . e_d).
// The slots those two pulls read -- (d, s) and (-d, x) -- are read by no other
// pull and by no other link (s lies inside one particle only), so each link's
// thread reads f*_{-d}(x) for the force and writes the bounced values there
// in place, and the sweep pulls every direction unconditionally.
template <int ST>
__device__ __forceinline__ void pre_body(const DevDomain *__restrict__ doms,
                                         const PItem *__restrict__ items, int kstep) {
  using S = Store<ST>;
  using T = typename S::T;
  using RS = typename S::R;
  __shared__ double red[PT / 64][7];
  __shared__ LinkList<1024> links;
  // labels G(T) of the box and a one-node rim (out of the domain: LBL_OUT)
  __shared__ uint8_t lab[LAB_BOX];
  const PItem it = items[blockIdx.x];
  const DevDomain &D = doms[it.dom];
  // The step counter, this particle's record in both state buffers, its force
  // record (read by the update at the end) and, one per lane, the other
  // particles' records in both buffers are requested together: none depends
  // on another, so choosing the buffer by the step's parity afterwards costs
  // no extra round trip through memory (this kernel is a latency chain).
  const uint64_t T0 = *D.tstep + (uint64_t)kstep;
  const PState Pa = D.pstate[0][it.p], Pb = D.pstate[1][it.p];
  const PForce Fpre = D.pforce[it.p];
  const int qme = (int)threadIdx.x;  // np <= MAX_PARTICLES <= 256: one particle per lane
  const bool pair_lane = D.lj_psi > 0.0 && qme < D.np && qme != it.p;
  PDisc qa{0.0, 0.0, 0.0}, qb{0.0, 0.0, 0.0};
  if (pair_lane) {
    const PState &A = D.pstate[0][qme], &B = D.pstate[1][qme];
    qa = PDisc{A.x, A.y, A.radius};
    qb = PDisc{B.x, B.y, B.radius};
  }
  static_assert(MAX_PARTICLES <= 256, "one particle per lane");
  const PState P = pick_state((T0 & 1) != 0, Pa, Pb);
  T *f = (T *)D.f[T0 & 1];
  const size_t plane = (size_t)D.ny * D.pitch;
  const bool perx = D.bc_x == BC_PERIODIC, pery = D.bc_y == BC_PERIODIC;
  const uint8_t mine = (uint8_t)(LBL_PART0 + it.p);
  const int reach = max((int)ceil(P.radius) + 2, (int)ceil(P.radius + D.lj_rit) + 1);
  const int W = 2 * reach + 2;
  const int bx0 = (int)floor(P.x) - reach, by0 = (int)floor(P.y) - reach;
  const double lim = P.radius + D.lj_rit;

  // stage the labels: box position (i, k) -> lab[(k + 1) * WR + i + 1]
  const int WR = W + 2;
  const float invr = 1.0f / (float)WR;
  for (int j = threadIdx.x; j < WR * WR; j += PT) {
    const int k = box_row(j, invr);
    int x = bx0 - 1 + j - k * WR, y = by0 - 1 + k;
    const bool in = wrap_coord(x, D.nx, perx) && wrap_coord(y, D.ny, pery);
    lab[j] = in ? D.label[(size_t)y * D.pitch + x] : LBL_OUT;
  }
  __syncthreads();
  auto lab_at = [&](int i, int k) { return lab[(k + 1) * WR + i + 1]; };

  // repulsion from the other particles, one lane per pair
  double plx = 0.0, ply = 0.0;
  if (pair_lane) {
    const bool odd = (T0 & 1) != 0;
    const PDisc Q{odd ? qb.x : qa.x, odd ? qb.y : qa.y, odd ? qb.radius : qa.radius};
    pair_repulsion(D, P, Q, plx, ply);
  }
  double acc[7] = {0.0, 0.0, 0.0, 0.0, 0.0, plx, ply};
  box_links<1024>(
      D, P, W, bx0, by0, links, acc,
      [&](int bi, int bk) -> uint32_t {
        const uint8_t lx = lab_at(bi, bk);
        if (lx == LBL_SOLID) {
          int x = bx0 + bi, y = by0 + bk;
          wrap_coord(x, D.nx, perx);
          wrap_coord(y, D.ny, pery);
          solid_repulsion(D, P, lim, x, y, acc[3], acc[4]);
        }
        if (lx != LBL_FLUID) return 0u;
        uint32_t m = 0;
#pragma unroll
        for (int i = 1; i < 9; ++i) m |= (uint32_t)(lab_at(bi - cx(i), bk - cy(i)) == mine) << (i - 1);
        return m;
      },
      [&](int x, int y, int, int, int dx, int dy) {
        int sx = x - dx, sy = y - dy;
        wrap_coord(sx, D.nx, perx);
        wrap_coord(sy, D.ny, pery);
        return (size_t)((uint32_t)sy * D.pitch + sx);
      },
      [&](size_t at, int i) { return (double)S::load(f + i * plane, at, i); },
      [&](size_t at, int i, double v) { S::put(f + i * plane, at, i, (RS)v, 0u); });
  block_sum<7>(acc, red);
  if (threadIdx.x < 64) {
    PForce F = Fpre;
    F.fx = acc[0];
    F.fy = acc[1];
    F.torque = acc[2];
    F.ljx = acc[3];
    F.ljy = acc[4];
    bool fast;
    const PState N = newton_euler(D, P, F, acc[5], acc[6], fast);
    if (threadIdx.x == 0) {
      D.pforce[it.p] = F;
      D.pstate[(T0 + 1) & 1][it.p] = N;
      if (fast) atomicOr(D.health, HEALTH_FAST_PARTICLE);
    }
  }
}

// Label of node (x, y) from the particle discs Pn (PState, or PDisc staged in
// LDS): first particle (in index order) whose disc strictly contains the
// node, else fluid.
template <class Disc>
__device__ __forceinline__ uint8_t new_label(const DevDomain &D, const Disc *Pn, int x, int y) {
  const bool perx = D.bc_x == BC_PERIODIC, pery = D.bc_y == BC_PERIODIC;
  for (int q = 0; q < D.np; ++q) {
    const double dx = min_image((double)x - Pn[q].x, D.nx, perx);
    const double dy = min_image((double)y - Pn[q].y, D.ny, pery);
    if (dx * dx + dy * dy < Pn[q].radius * Pn[q].radius) return (uint8_t)(LBL_PART0 + q);
  }
  return LBL_FLUID;
}
// The same rule over the candidate discs cand[0 .. n) (ascending indices):
// the particles that can hold a node of the caller's box.
__device__ __forceinline__ uint8_t label_among(const DevDomain &D, const PDisc *Pn, const int *cand,
                                               int n, int x, int y) {
  const bool perx = D.bc_x == BC_PERIODIC, pery = D.bc_y == BC_PERIODIC;
  for (int k = 0; k < n; ++k) {
    const int q = cand[k];
    const double dx = min_image((double)x - Pn[q].x, D.nx, perx);
    const double dy = min_image((double)y - Pn[q].y, D.ny, pery);
    if (dx * dx + dy * dy < Pn[q].radius * Pn[q].radius) return (uint8_t)(LBL_PART0 + q);
  }
  return LBL_FLUID;
}

// After the sweep of step T -> T+1, one workgroup per particle p, over a box
// around P(T+1) that holds every node p leaves or enters (particles move less
// than half a node per step).  G(T) and G(T+1) of a non-solid node are the
// first-particle rule applied to P(T) and P(T+1), so no workgroup reads the
// label plane while others rewrite it (overlapping boxes write identical
// values).  Covered node (enters p): F = +rho (u - U_p); uncovered node:
// -rho (u - U_p), with rho and u = j/rho + g/2 the moments of f(T+1)
// (recovered from f*(T+1): j(f*) = j(f) + rho g), applied in the next step
// (Eq. MP3).
template <int ST>
__device__ __forceinline__ void post_body(const DevDomain *__restrict__ doms,
                                          const PItem *__restrict__ items, int kstep) {
  using S = Store<ST>;
  using T = typename S::T;
  __shared__ double red[PT / 64][3];
  __shared__ int scan_sh[4];
  // discs of P(T) and P(T+1) that can reach a node of this box, in index
  // order (so the first-particle rule is unchanged)
  __shared__ PDisc disc0[MAX_PARTICLES], disc1[MAX_PARTICLES];
  __shared__ int cand[MAX_PARTICLES];
  const PItem it = items[blockIdx.x];
  const DevDomain &D = doms[it.dom];
  // the step counter and the discs in both state buffers (this particle's
  // record, and one other particle per lane) are requested together, then
  // sorted into old and new by the step's parity: no dependent round trip
  const uint64_t T1 = *D.tstep + (uint64_t)kstep + 1;
  const PState Pa = D.pstate[0][it.p], Pb = D.pstate[1][it.p];
  const int qme = (int)threadIdx.x;  // MAX_PARTICLES <= 256: one disc per lane
  PDisc qa{0.0, 0.0, 0.0}, qb{0.0, 0.0, 0.0};
  if (qme < D.np) {
    const PState &A = D.pstate[0][qme], &B = D.pstate[1][qme];
    qa = PDisc{A.x, A.y, A.radius};
    qb = PDisc{B.x, B.y, B.radius};
  }
  const bool odd = (T1 & 1) != 0;
  const PState P = pick_state(odd, Pa, Pb);  // P(T+1)
  const T *src = (const T *)D.f[T1 & 1];
  const size_t plane = (size_t)D.ny * D.pitch;
  const bool perx = D.bc_x == BC_PERIODIC, pery = D.bc_y == BC_PERIODIC;
  const uint8_t mine = (uint8_t)(LBL_PART0 + it.p);
  const int reach = (int)ceil(P.radius) + 3;
  const int W = 2 * reach + 2;
  const int bx0 = (int)floor(P.x) - reach, by0 = (int)floor(P.y) - reach;
  int ncand;
  {
    static_assert(MAX_PARTICLES <= 256, "one candidate test per lane");
    // a node of the box lies within (W - 1) / 2 of the box centre on each
    // axis, so a disc holding one has its centre within r + W / 2 + 1
    const int q = qme;
    int hit = 0;
    if (q < D.np) {
      const double bcx = bx0 + 0.5 * (W - 1), bcy = by0 + 0.5 * (W - 1), h = 0.5 * W + 1.0;
      const PDisc A{odd ? qa.x : qb.x, odd ? qa.y : qb.y, odd ? qa.radius : qb.radius};  // P(T)
      const PDisc B{odd ? qb.x : qa.x, odd ? qb.y : qa.y, odd ? qb.radius : qa.radius};  // P(T+1)
      disc0[q] = A;
      disc1[q] = B;
      hit = (fabs(min_image(A.x - bcx, D.nx, perx)) < h + A.radius &&
             fabs(min_image(A.y - bcy, D.ny, pery)) < h + A.radius) ||
            (fabs(min_image(B.x - bcx, D.nx, perx)) < h + B.radius &&
             fabs(min_image(B.y - bcy, D.ny, pery)) < h + B.radius);
    }
    const int pos = block_exscan(hit, scan_sh, ncand);
    if (hit) cand[pos] = q;
    __syncthreads();
  }
  double acc[3] = {0.0, 0.0, 0.0};
  const float inv = 1.0f / (float)W;
  for (int j = threadIdx.x; j < W * W; j += PT) {
    const int k = box_row(j, inv);
    int x = bx0 + j - k * W, y = by0 + k;
    if (!wrap_coord(x, D.nx, perx) || !wrap_coord(y, D.ny, pery)) continue;
    const uint32_t here = (uint32_t)y * D.pitch + x;
    if (D.nodew[here] & NODE_SOLID) continue;
    const uint8_t l0 = label_among(D, disc0, cand, ncand, x, y);
    const uint8_t l1 = label_among(D, disc1, cand, ncand, x, y);
    if (l1 != l0) D.label[here] = l1;
    if ((l0 == mine) == (l1 == mine)) continue;
    const double sign = l1 == mine ? 1.0 : -1.0;
    cover_term(D, P, x, y, sign, acc,
               [&](int i) { return (double)S::load(src + i * plane, here, i); });
  }
  block_sum<3>(acc, red);
  if (threadIdx.x == 0) {
    PForce &F = D.pforce[it.p];
    F.cx_ = acc[0];
    F.cy_ = acc[1];
    F.ctorque = acc[2];
  }
}

template <int ST>
__global__ __launch_bounds__(PT) void k_pre(const DevDomain *__restrict__ doms,
                                             const PItem *__restrict__ items, int kstep) {
  pre_body<ST>(doms, items, kstep);
}

template <int ST>
__global__ __launch_bounds__(PT) void k_post(const DevDomain *__restrict__ doms,
                                              const PItem *__restrict__ items, int kstep) {
  post_body<ST>(doms, items, kstep);
}

// k_post of step kstep and k_pre of step kstep + 1 in one launch, for
// launches in which no domain holds more than one particle.  Then each
// workgroup's particle is alone in its domain: no other workgroup touches
// its labels, populations or records, and the barrier between the two
// halves orders everything the second half reads (the labels and the cover
// force just written, the populations the first half read before the
// bounce-back writes).  One launch less per step, the same results.  With
// two or more particles in a domain the halves of different workgroups
// would race (a disc's bounce-back writes can reach nodes a neighbour's
// cover force still reads), so those launches keep the two kernels.
template <int ST>
__global__ __launch_bounds__(PT) void k_post_pre(const DevDomain *__restrict__ doms,
                                                  const PItem *__restrict__ items, int kstep) {
  post_body<ST>(doms, items, kstep);
  __syncthreads();
  pre_body<ST>(doms, items, kstep + 1);
}

#ifdef LBK_COMMON_KERNELS
// Labels of the current particle state inside each particle's box, from the
// label plane's own values (used once the particles are added).
__global__ __launch_bounds__(256) void k_relabel(const DevDomain *__restrict__ doms,
                                                 const PItem *__restrict__ items) {
  const PItem it = items[blockIdx.x];
  const DevDomain &D = doms[it.dom];
  const PState *Pn = D.pstate[*D.tstep & 1];
  const PState P = Pn[it.p];
  const bool perx = D.bc_x == BC_PERIODIC, pery = D.bc_y == BC_PERIODIC;
  const int reach = (int)ceil(P.radius) + 3;
  const int W = 2 * reach + 2;
  const int bx0 = (int)floor(P.x) - reach, by0 = (int)floor(P.y) - reach;
  for (int j = threadIdx.x; j < W * W; j += 256) {
    int x = bx0 + j % W, y = by0 + j / W;
    if (!wrap_coord(x, D.nx, perx) || !wrap_coord(y, D.ny, pery)) continue;
    const size_t here = (size_t)y * D.pitch + x;
    const uint8_t l0 = D.label[here];
    if (l0 == LBL_SOLID) continue;
    const uint8_t l1 = new_label(D, Pn, x, y);
    if (l1 != l0) D.label[here] = l1;
  }
}

// [a0, a1] meets [b0, b1] (inclusive node ranges; b may reach past the
// domain, whose periodic images count on a periodic axis)
__device__ __forceinline__ bool ranges_meet(int a0, int a1, int b0, int b1, int n, bool periodic) {
  if (b0 <= a1 && a0 <= b1) return true;
  if (!periodic) return false;
  return (b0 - n <= a1 && a0 <= b1 - n) || (b0 + n <= a1 && a0 <= b1 + n);
}

// Sweep tiles that the particle coupling around the state T = tstep + kstep
// touches: k_post of the step before (labels in a box of reach ceil(R) + 3
// around P(T)) and k_pre (link slots within one node of a box of reach
// max(ceil(R) + 2, ceil(R + r_it) + 1) around P(T)).  A tile is flagged when
// its nodes or the nodes its pulls read (one-node halo) come within two nodes
// of the larger box, into near_tiles[T & 1].  One thread per tile.
__global__ __launch_bounds__(256) void k_near_tiles(const DevDomain *__restrict__ Dp, int kstep) {
  const DevDomain &D = *Dp;
  const int t = (int)(blockIdx.x * 256 + threadIdx.x);
  if (t >= D.tiles_x * D.tiles_y) return;
  const uint64_t T = *D.tstep + (uint64_t)kstep;
  const PState *P = D.pstate[T & 1];
  const int th = (256 / D.tile_w) * D.rows_per_thread;
  const int ty = t / D.tiles_x, tx = t - ty * D.tiles_x;
  const int x0 = tx * D.tile_w - 1, x1 = min((tx + 1) * D.tile_w, D.nx);
  const int y0 = ty * th - 1, y1 = min((ty + 1) * th, D.ny);
  const bool perx = D.bc_x == BC_PERIODIC, pery = D.bc_y == BC_PERIODIC;
  uint8_t hit = 0;
  for (int p = 0; p < D.np && !hit; ++p) {
    const PState &Q = P[p];
    const int reach =
        max((int)ceil(Q.radius) + 3, (int)ceil(Q.radius + D.lj_rit) + 1) + 2;
    const int cx0 = (int)floor(Q.x), cy0 = (int)floor(Q.y);
    hit = ranges_meet(x0, x1, cx0 - reach, cx0 + reach + 1, D.nx, perx) &&
          ranges_meet(y0, y1, cy0 - reach, cy0 + reach + 1, D.ny, pery);
  }
  D.near_tiles[T & 1][t] = hit;
}
#endif  // LBK_COMMON_KERNELS

}  // namespace lbk
