// discn_impl.h -- several time steps per launch for domains with one particle.
//
// A step of such a domain is a chain of two launches, k_post_pre on one
// workgroup (14 us, dependent loads and block sums) and the sweep (7.6 us at
// 512^2); neither fills the chip.  Here one launch takes DISC_STEPS steps: a
// workgroup of its own per particle holds the region around it in LDS and runs
// the whole of k_pre, sweep and k_post on it, step by step, beside the tiles of
// sweepn_impl.h, which sweep the domain as if there were no particle and leave
// the nodes around it, where that matters, to its workgroup.
//
// Measured, FP32 with noise, R = 5, us a step: 512^2 22 -> 8.8, bound by the
// particle's workgroup (a launch of three steps takes 26 us with it, 12
// without: 7 for its loads and stores, then a third each for the links, the
// sweep of its nodes by one CU, and the labels and sums); 32 domains of 128^2
// to 1024^2 123 -> 74, bound by the tiles.  More steps a launch would not help
// the first and make the region and its rim larger.
//
// What that rests on, with n = 3 steps, offsets counted from the node of P(T),
// the region at offsets -H .. H - 1, a radius R and a drift of less than half a
// node a step:
//  * the links and covered nodes of state T + j lie within R + 2 + j / 2, and
//    the region is valid to H - 1 - j;
//  * the particle's workgroup stores the nodes at least n inside the region.
//    Any other node is at offset H - n or more, reads state T + j from offset
//    H - 2 n + j on, and the slots that the links rewrite end before
//    R + 2 + j / 2.
// H = ceil(R) + 8 keeps both.  A particle faster than half a node a step
// latches the health flag, as in k_pre; its boxes are clamped to the region,
// so that nothing is accessed out of range.
//
// Every node, link, sum and update goes through the code of k_pre, k_post and
// the sweep in the same order (the sums: PT threads over the same box), so the
// results are bit-identical to single steps.
#pragma once

#include "particles_impl.h"
#include "sweepn_impl.h"

namespace lbk {

constexpr int DISC_DRIFT = DISC_STEPS;
constexpr int DISC_LINKS = 256;  // nodes of an annulus of sqrt(2) around a radius of 8: about 80
constexpr int DW = DISC_SIDE;  // row length of the region in LDS, whatever its side

// What the particle's workgroup holds on chip, in the memory that the tiles of
// region K use for theirs where it is large enough.
template <int ST> struct DiscShared {
  typename Store<ST>::T f[9][DW * DW];
  uint16_t nodew[DW * DW];
  uint8_t lab[DISC_BOX * DISC_BOX];
  LinkList<DISC_LINKS> links;
  double red7[PT / 64][7], red3[PT / 64][3];
  PState p[2];  // P(T + s) in p[s & 1]
  PForce force;
  int changed;  // some label changed in this step
};

// Nodes that the particle's workgroup stores, from P(T).
__device__ __forceinline__ SkipRect disc_rect(const DevDomain &D, uint64_t T0) {
  const PState *const ps0 = D.pstate[0];
  const PState *const ps1 = D.pstate[1];
  const bool odd = (T0 & 1) != 0;
  const double xa = gbl(ps0)->x, xb = gbl(ps1)->x, ya = gbl(ps0)->y, yb = gbl(ps1)->y;
  const double ra = gbl(ps0)->radius, rb = gbl(ps1)->radius;
  const int x = __builtin_amdgcn_readfirstlane((int)floor(odd ? xb : xa));
  const int y = __builtin_amdgcn_readfirstlane((int)floor(odd ? yb : ya));
  const int side = disc_side(__builtin_amdgcn_readfirstlane((int)ceil(odd ? rb : ra)));
  const int in = DISC_STEPS - side / 2, len = side - 2 * DISC_STEPS;
  return SkipRect{wrap(wrap(x, D.nx) + in, D.nx), wrap(wrap(y, D.ny) + in, D.ny), len, len};
}

template <int ST, int FEAT, int PLM, int NT>
__device__ __forceinline__ void disc_body(const DevDomain &D, DiscShared<ST> &sh, uint64_t T0) {
  using S = Store<ST>;
  using T = typename S::T;
  using R = CompT<ST, 0>;
  using RS = typename S::R;
  constexpr int NODES = DW * DW, U = NODES / NT;
  static_assert(NODES % NT == 0 && NT == PT, "whole nodes per thread");
  constexpr uint32_t B = sizeof(T);
  const int nx = D.nx, ny = D.ny, pitch = D.pitch;
  const bool perx = D.bc_x == BC_PERIODIC, pery = D.bc_y == BC_PERIODIC;
  const uint32_t pitchB = (uint32_t)pitch * B, planeB = (uint32_t)ny * pitchB;
  void *const f0 = D.f[0];
  void *const f1 = D.f[1];
  const BufRes src = pop_buffer((T0 & 1) ? f1 : f0, 9u * planeB);
  const BufRes dst = pop_buffer((T0 & 1) ? f0 : f1, 9u * planeB);
  const bool sr = (ST == ST_F16 || ST == ST_BF16) && (D.feat & F_STOCH);
  const int tid = (int)threadIdx.x;
  const PState *const ps0 = D.pstate[0];
  const PState *const ps1 = D.pstate[1];
  const bool odd = (T0 & 1) != 0;
  const double xa = gbl(ps0)->x, xb = gbl(ps1)->x, ya = gbl(ps0)->y, yb = gbl(ps1)->y;
  const double ra = gbl(ps0)->radius, rb = gbl(ps1)->radius;
  if (tid < (int)sizeof(PState) / 8) {
    const double *q = (const double *)(odd ? ps1 : ps0);
    ((double *)&sh.p[0])[tid] = gbl(q)[tid];
  } else if (tid >= 64 && tid < 64 + (int)sizeof(PForce) / 8) {
    ((double *)&sh.force)[tid - 64] = gbl((const double *)D.pforce)[tid - 64];
  }
  const int cx0 = wrap(__builtin_amdgcn_readfirstlane((int)floor(odd ? xb : xa)), nx);
  const int cy0 = wrap(__builtin_amdgcn_readfirstlane((int)floor(odd ? yb : ya)), ny);
  const uint8_t mine = LBL_PART0;
  const double rad = odd ? rb : ra;
  const double lim = rad + D.lj_rit;
  const int rceil = __builtin_amdgcn_readfirstlane((int)ceil(rad));
  const int reach =
      max(rceil + 2, __builtin_amdgcn_readfirstlane((int)ceil(rad + D.lj_rit)) + 1);
  const int SBH = reach + 1 + DISC_DRIFT, SB = disc_box(reach);
  const int side = disc_side(rceil), half = side / 2;
  const float invb = 1.0f / (float)SB;
  bool bad = false;

  // The region's populations f*(T), its node words, and the labels G(T) of the
  // box, row by row, all loads in flight together.
  {
    T raw[U][9];
    uint16_t nw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = tid + u * NT, r = k / DW, c = k % DW;
      const int x = wrap_near(cx0 - half + (c < side ? c : 0), nx);
      const int y = wrap_near(cy0 - half + (r < side ? r : 0), ny);
      const uint32_t at = (uint32_t)y * pitchB + (uint32_t)x * B;
#pragma unroll
      for (int i = 0; i < 9; ++i) raw[u][i] = bload<T>(src, at, (uint32_t)i * planeB);
      nw[u] = gbl(D.nodew)[(uint32_t)y * pitch + x];
    }
    for (int j = tid; j < SB * SB; j += NT) {
      const int k = box_row(j, invb), x = cx0 - SBH + j - k * SB, y = cy0 - SBH + k;
      const bool in = (perx || (x >= 0 && x < nx)) && (pery || (y >= 0 && y < ny));
      sh.lab[j] = in ? gbl(D.label)[(size_t)wrap_near(y, ny) * pitch + wrap_near(x, nx)] : LBL_OUT;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < 9; ++i) sh.f[i][tid + u * NT] = raw[u][i];
      sh.nodew[tid + u * NT] = nw[u];
    }
  }
  // The nodes are numbered from the inside out for the steps: the square that
  // the last one leaves, then the rings around it, so that those of every step
  // are the first (side - 2 s)^2 and fill whole waves.
  int id[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int k = tid + u * NT;
    int m = side - 2 * DISC_STEPS, c, r;
    if (k < m * m) {
      r = box_row(k, 1.0f / (float)m);
      c = k - r * m;
      r += DISC_STEPS;
      c += DISC_STEPS;
    } else {
      int t = DISC_STEPS - 1;  // ring t nodes from the edge
      while (t > 0 && k >= (m + 2) * (m + 2)) {
        m += 2;
        --t;
      }
      const int e = k - m * m, q = m + 2;
      if (e < 2 * q) {
        r = e < q ? t : t + q - 1;
        c = t + (e < q ? e : e - q);
      } else {
        const int g = e - 2 * q;
        r = t + 1 + (g >> 1);
        c = (g & 1) ? t + q - 1 : t;
      }
    }
    id[u] = k < side * side ? r * DW + c : 0;
  }
  // how far the particle's node is from (cx0, cy0), inside the drift
  auto offset = [](double v, int c, int n, bool per) {
    int o = (int)floor(v) - c;
    if (per) o = o > n / 2 ? o - n : (o < -(n / 2) ? o + n : o);
    return min(max(o, -DISC_DRIFT), DISC_DRIFT);
  };
  __syncthreads();
  // its place in the domain, from its place in the region
  auto place = [&](int at, int &x, int &y) {
    x = wrap_near(cx0 - half + at % DW, nx);
    y = wrap_near(cy0 - half + at / DW, ny);
  };

#pragma unroll 1
  for (int s = 1; s <= DISC_STEPS; ++s) {
    const uint32_t step = (uint32_t)(T0 + (uint64_t)s);
    const PState &Q = sh.p[(s - 1) & 1];  // P(T + s - 1)
    PState &P = sh.p[s & 1];              // P(T + s)
    // ---- k_pre of state T + s - 1
    {
      const int ox = offset(Q.x, cx0, nx, perx), oy = offset(Q.y, cy0, ny, pery);
      const int W = 2 * reach + 2;
      const uint8_t *lab0 = sh.lab + (SBH + oy - reach) * SB + SBH + ox - reach;
      const int x0 = cx0 + ox - reach, y0 = cy0 + oy - reach;
      const int gx0 = half + ox - reach, gy0 = half + oy - reach;
      double acc[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      box_links<DISC_LINKS>(
          D, Q, W, x0, y0, sh.links, acc,
          [&](int bi, int bk) -> uint32_t {
            const uint8_t *lab = lab0 + bk * SB + bi;
            const uint8_t lx = *lab;
            if (lx == LBL_SOLID)
              solid_repulsion(D, Q, lim, wrap_near(x0 + bi, nx), wrap_near(y0 + bk, ny), acc[3], acc[4]);
            const int gx = gx0 + bi, gy = gy0 + bk;
            if (lx != LBL_FLUID || gx < 1 || gx >= side - 1 || gy < 1 || gy >= side - 1) return 0u;
            uint32_t m = 0;
#pragma unroll
            for (int i = 1; i < 9; ++i) m |= (uint32_t)(lab[-cy(i) * SB - cx(i)] == mine) << (i - 1);
            return m;
          },
          [&](int, int, int bi, int bk, int dx, int dy) { return (gy0 + bk - dy) * DW + gx0 + bi - dx; },
          [&](int at, int i) { return (double)S::dec(sh.f[i][at], i); },
          [&](int at, int i, double v) { sh.f[i][at] = S::enc((RS)v, i, 0u); });
      block_sum<7>(acc, sh.red7);
      // P(T + s), by the wave with the fewest nodes beside the others' sweep
      if (tid >= NT - 64) {
        PForce F = sh.force;
        F.fx = acc[0];
        F.fy = acc[1];
        F.torque = acc[2];
        F.ljx = acc[3];
        F.ljy = acc[4];
        bool fast;
        const PState N = newton_euler(D, Q, F, 0.0, 0.0, fast);
        if (tid == NT - 64) {
          sh.force = F;
          sh.changed = 0;
          P = N;
          if (fast) atomicOr(D.health, HEALTH_FAST_PARTICLE);
        }
      }
    }
    // ---- the sweep of the nodes at least s inside the region, in place
    {
      Pulled<T> raw[U];
      const int last = (side - 2 * s) * (side - 2 * s);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (tid + u * NT >= last) continue;
        const T *p = &sh.f[0][0] + id[u];
        const uint32_t wu = sh.nodew[id[u]];
        raw[u].set(0, p[0]);
#pragma unroll
        for (int i = 1; i < 9; ++i)
          raw[u].set(i, p[((wu >> (i - 1)) & 1u) ? opp(i) * NODES : i * NODES - cy(i) * DW - cx(i)]);
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (tid + u * NT >= last) continue;
        const bool solid = sh.nodew[id[u]] & NODE_SOLID;
        int x, y;
        place(id[u], x, y);
        const uint32_t node = (uint32_t)y * (uint32_t)nx + (uint32_t)x;
        R e[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) e[i] = solid ? R(0) : (R)S::raw_dec(raw[u].get(i));
        bad = bad || !(fabs(scaled_drho<ST, R>(e)) < R(1e30));
        collide_node<ST, FEAT, PLM, R>(D, e, node, step);
        T q[9];
        if (sr) {
          encode_node<ST, R, true>(D, e, node, step, q);
#pragma unroll
          for (int i = 0; i < 9; ++i) sh.f[i][id[u]] = q[i];
        } else {
          encode_node<ST, R, false>(D, e, node, step, q);
#pragma unroll
          for (int i = 0; i < 9; ++i) sh.f[i][id[u]] = q[i];
        }
      }
      __syncthreads();
    }
    // ---- k_post: labels G(T + s) and the cover force of the changed nodes
    {
      const int ox = offset(P.x, cx0, nx, perx), oy = offset(P.y, cy0, ny, pery);
      const int preach = rceil + 3, W = 2 * preach + 2;
      const float inv = 1.0f / (float)W;
      double acc[3] = {0.0, 0.0, 0.0};
      for (int j = tid; j < W * W; j += PT) {
        const int bk = box_row(j, inv), bi = j - bk * W;
        uint8_t &lab = sh.lab[(SBH + oy - preach + bk) * SB + SBH + ox - preach + bi];
        if (lab == LBL_OUT || lab == LBL_SOLID) continue;
        const int x = wrap_near(cx0 + ox - preach + bi, nx), y = wrap_near(cy0 + oy - preach + bk, ny);
        const double dx0 = min_image((double)x - Q.x, nx, perx), dy0 = min_image((double)y - Q.y, ny, pery);
        const double dx1 = min_image((double)x - P.x, nx, perx), dy1 = min_image((double)y - P.y, ny, pery);
        const bool in0 = dx0 * dx0 + dy0 * dy0 < Q.radius * Q.radius;
        const bool in1 = dx1 * dx1 + dy1 * dy1 < P.radius * P.radius;
        if (in0 == in1) continue;
        lab = in1 ? mine : LBL_FLUID;
        sh.changed = 1;
        const int gx = half + ox - preach + bi, gy = half + oy - preach + bk;
        if (gx < 0 || gx >= side || gy < 0 || gy >= side) continue;
        const T *const p = &sh.f[0][0] + gy * DW + gx;
        cover_term(D, P, x, y, in1 ? 1.0 : -1.0, acc,
                   [&](int i) { return (double)S::dec(p[i * NODES], i); });
      }
      __syncthreads();
      if (sh.changed) block_sum<3>(acc, sh.red3);  // else all zero
      if (tid == NT - 64) {
        sh.force.cx_ = acc[0];
        sh.force.cy_ = acc[1];
        sh.force.ctorque = acc[2];
      }
    }
  }
  // state T + n
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (tid + u * NT >= (side - 2 * DISC_STEPS) * (side - 2 * DISC_STEPS)) continue;
    int x, y;
    place(id[u], x, y);
    const uint32_t here = (uint32_t)y * pitchB + (uint32_t)x * B;
#pragma unroll
    for (int i = 0; i < 9; ++i) bstore<T, false>(dst, here, (uint32_t)i * planeB, sh.f[i][id[u]]);
  }
  for (int j = tid; j < SB * SB; j += NT) {
    const uint8_t l = sh.lab[j];
    if (l == LBL_OUT || l == LBL_SOLID) continue;
    const int k = box_row(j, invb);
    const int x = wrap_near(cx0 - SBH + j - k * SB, nx), y = wrap_near(cy0 - SBH + k, ny);
    gbl(D.label)[(size_t)y * pitch + x] = l;
  }
  if (tid == NT - 64) {
    PState *const nxt = odd ? D.pstate[0] : D.pstate[1];
    static_assert((DISC_STEPS & 1) != 0, "into the other buffer");
    *nxt = sh.p[DISC_STEPS & 1];
    *D.pforce = sh.force;
  }
  if (bad) atomicOr(D.health, HEALTH_NONFINITE);
}

// DISC_STEPS steps of domains that hold at most one particle each: a workgroup
// per particle (items), then the tiles.
template <int ST, int FEAT, int PLM, int K>
__global__ __launch_bounds__(region(K).nt, 4) void k_multi_disc(const DevDomain *__restrict__ doms,
                                                             const int *__restrict__ prefix, int ndom,
                                                             const PItem *__restrict__ items,
                                                             int nitems, const DevDomain one,
                                                             int kstep) {
  using Tile = typename Store<ST>::T[9][region(K).cw * region(K).rs];
  constexpr size_t bytes = sizeof(Tile) > sizeof(DiscShared<ST>) ? sizeof(Tile) : sizeof(DiscShared<ST>);
  __shared__ alignas(16) char mem[bytes];
  if ((int)blockIdx.x < nitems) {
    // a single domain's descriptor comes in the arguments: two dependent loads less
    DevDomain D;
    if (one.nx > 0) D = one;
    else D = doms[items[blockIdx.x].dom];
    disc_body<ST, FEAT, PLM, region(K).nt>(D, *(DiscShared<ST> *)mem, uniform_time(D, kstep));
    return;
  }
  const int b = xcd_remap((int)blockIdx.x - nitems, (int)gridDim.x - nitems);
  const int dix = ndom == 1 ? 0 : find_domain(prefix, ndom, b);
  DevDomain D;  // held in scalar registers across the steps
  if (one.nx > 0) D = one;
  else D = doms[dix];
  const uint64_t T0 = uniform_time(D, kstep);
  multi_body<ST, FEAT, PLM, K, region(K).nt, true>(D, *(Tile *)mem, ndom == 1 ? b : b - prefix[dix], T0, DISC_STEPS,
                                     D.np > 0 ? disc_rect(D, T0) : SkipRect{0, 0, 0, 0});
}

}  // namespace lbk
