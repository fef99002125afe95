// sweepn_impl.h -- several time steps per launch, for the domains that need
// nothing between two steps (no density faces, and no particles but those of
// discn_impl.h): obstacles,
// walls as label rows, either collision, the power law, thermal noise.
//
// A workgroup owns a region of CW x RS nodes.  The first step of the region is
// computed from global memory, exactly as k_sweep does, and kept in LDS,
// rounded to the storage format; each further step pulls from LDS, where the
// nodes whose sources are all inside (one node less on every side) take the
// next step in place; the last one stores its nodes to global memory.  With n
// steps a launch the stored tile is the region less n - 1 nodes on every side,
// and the tiles cover the domain.  Every node of every step goes through the
// same pull, collision and rounding as in k_sweep, so the result is
// bit-identical to n single steps.
//
// What this is for.  Small lattices are bound by the ~4 us that a launch
// costs from its first load to its last store, large ones by the bytes of a
// step: both are paid once per n steps.  What n costs is the rim, computed by
// several workgroups.  step_plan.h has a model of what a launch costs and splits
// the steps of a call by it.
//
// n is odd (3, 5, 7, 9): the launch reads buffer T & 1 and writes the other,
// which is the buffer of step T + n, so any sequence of launches and single
// steps leaves the state where every other kernel expects it.
//
// Measured, us a step, against the two-step tiles this replaced (62 columns
// by 6 to 14 rows, a pair of steps a launch): channel 128 x 64 FP64 3.13 ->
// 1.03, power-law channel 101 x 51 FP32 4.34 -> 1.37, noise 256 x 512 FP32
// 5.08 -> 2.58, 724 x 700 FP32 4.84 -> 3.45, 2048^2 with obstacles FP32 41.0
// -> 23.9, 4096^2 FP32 134 -> 77 (15.7 TB/s of single-step bytes), 3000^2
// FP64 138 -> 76, 4096^2 FP16 80.1 -> 72.5.
#pragma once

#include "sweep_impl.h"

namespace lbk {

// State time, made wave-uniform so that the buffers stay in scalar registers.
__device__ __forceinline__ uint64_t uniform_time(const DevDomain &D, int kstep) {
  const uint64_t ts = *gbl(D.tstep);
  return (((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(ts >> 32)) << 32) |
          __builtin_amdgcn_readfirstlane((uint32_t)ts)) + (uint64_t)kstep;
}

// c mod n, in [0, n)
__device__ __forceinline__ int wrap(int c, int n) {
  c %= n;
  return c < 0 ? c + n : c;
}

// The same for a c less than a period outside.
__device__ __forceinline__ int wrap_near(int c, int n) { return c < 0 ? c + n : (c >= n ? c - n : c); }

// With SKIP, the nodes [skip_x, skip_x + skip_w) x [skip_y, skip_y + skip_h),
// wrapped, are left to another workgroup.
struct SkipRect {
  int x, y, w, h;
};

// ONE: a single step is possible, from global memory to global memory.
template <int ST, int FEAT, int PLM, int K, int NT, bool SKIP = false, bool ONE = false>
__device__ __forceinline__ void multi_body(const DevDomain &D,
                                           typename Store<ST>::T (*lds)[region(K).cw * region(K).rs],
                                           int tile, uint64_t T0, int nsteps,
                                           SkipRect skip = SkipRect{}) {
  using S = Store<ST>;
  using T = typename S::T;
  using R = CompT<ST, 0>;
  constexpr bool LABELS = (FEAT & F_LABELS) != 0;
  constexpr Region G = region(K);
  constexpr int CW = G.cw, RS = G.rs, NODES = CW * RS, U = NODES / NT;
  static_assert(NODES % NT == 0, "whole nodes per thread");
  constexpr uint32_t B = sizeof(T);

  const int nx = D.nx, ny = D.ny, pitch = D.pitch;
  const int rim = nsteps - 1, ow = CW - 2 * rim, oh = RS - 2 * rim;
  const int tiles_x = (nx + ow - 1) / ow;
  const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
  const uint32_t pitchB = (uint32_t)pitch * B, planeB = (uint32_t)ny * pitchB;
  void *const f0 = D.f[0];
  void *const f1 = D.f[1];
  const BufRes src = pop_buffer((T0 & 1) ? f1 : f0, 9u * planeB);
  const BufRes dst = pop_buffer((T0 & 1) ? f0 : f1, 9u * planeB);
  const bool has_lab = LABELS && D.label != nullptr;
  const bool sr = (ST == ST_F16 || ST == ST_BF16) && (D.feat & F_STOCH);
  bool bad = false;

  // this thread's nodes: id = thread + u NT, row id / CW, column id % CW.  Where
  // a wave is one row, the row and its addresses live in scalar registers.
  static_assert(NT % CW == 0, "the same column in every row");
  const int col = (int)threadIdx.x % CW;
  const int row0 = CW == 64 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / CW)
                            : (int)threadIdx.x / CW;
  constexpr int RSTEP = NT / CW;
  uint32_t w[U], node[U], here[U];
  int xu[U], yu[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int x = tx * ow - rim + col, y = ty * oh - rim + row0 + u * RSTEP;
    xu[u] = nx >= CW ? wrap_near(x, nx) : wrap(x, nx);
    yu[u] = ny >= RS ? wrap_near(y, ny) : wrap(y, ny);
    w[u] = has_lab ? gbl(D.nodew)[(uint32_t)yu[u] * pitch + xu[u]] : 0u;
    node[u] = (uint32_t)yu[u] * (uint32_t)nx + (uint32_t)xu[u];
    here[u] = (uint32_t)yu[u] * pitchB + (uint32_t)xu[u] * B;
  }
  // first step: the pulls of all nodes together.  The population plane is
  // the scalar offset, the place in it the vector offset; opposite directions
  // lie two planes apart, so a bounced pull takes the lower one's plane and
  // the vector offset makes up the rest (see pull_node).
  Pulled<T> raw[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int x = xu[u], y = yu[u];
    const uint32_t xo[3] = {(uint32_t)(x + 1 < nx ? x + 1 : 0) * B, (uint32_t)x * B,
                            (uint32_t)(x > 0 ? x - 1 : nx - 1) * B};
    const uint32_t yo[3] = {(uint32_t)(y + 1 < ny ? y + 1 : 0) * pitchB, (uint32_t)y * pitchB,
                            (uint32_t)(y > 0 ? y - 1 : ny - 1) * pitchB};
    raw[u].set(0, bload<T>(src, here[u], 0u));
#pragma unroll
    for (int i = 1; i < 9; ++i) {
      const uint32_t vN = yo[1 + cy(i)] + xo[1 + cx(i)];
      if constexpr (!LABELS) {
        raw[u].set(i, bload<T>(src, vN, (uint32_t)i * planeB));
      } else {
        const bool up = opp(i) > i;
        uint32_t m = (uint32_t)(-(int32_t)((w[u] >> (i - 1)) & 1u));  // all ones: bounces
        __asm__("" : "+v"(m));
        const uint32_t a = up ? vN : vN + 2u * planeB, c = up ? here[u] + 2u * planeB : here[u];
        raw[u].set(i, bload<T>(src, a ^ ((a ^ c) & m), (uint32_t)(up ? i : opp(i)) * planeB));
      }
    }
  }
  // the rounding mode is uniform: each branch keeps its own writes
  auto encode = [&](const R (&e)[9], uint32_t nd, uint32_t step, auto &&put) {
    T q[9];
    if (sr) {
      encode_node<ST, R, true>(D, e, nd, step, q);
#pragma unroll
      for (int i = 0; i < 9; ++i) put(i, q[i]);
    } else {
      encode_node<ST, R, false>(D, e, nd, step, q);
#pragma unroll
      for (int i = 0; i < 9; ++i) put(i, q[i]);
    }
  };
  // A solid node is swept at rest, as in k_sweep, wherever its values are
  // stored to memory: a solid neighbour's next pull would read them.  The first
  // of several steps is only kept in LDS, where nothing reads them (a pull from
  // a solid bounces back), so there it collides whatever it pulled; in either
  // case what a solid holds is not checked.
  const bool stored = ONE && nsteps == 1;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int id = (int)threadIdx.x + u * NT;
    const bool solid = LABELS && (w[u] & NODE_SOLID);
    R e[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) e[i] = stored && solid ? R(0) : (R)S::raw_dec(raw[u].get(i));
    bad = bad || (!solid && !(fabs(scaled_drho<ST, R>(e)) < R(1e30)));
    const uint32_t step = (uint32_t)(T0 + 1);
    collide_node<ST, FEAT, PLM, R>(D, e, node[u], step);
    if (!ONE || nsteps > 1)
      encode(e, node[u], step, [&](int i, T v) { lds[i][id] = v; });
    else if (tx * ow + col < nx && ty * oh + row0 + u * RSTEP < ny)
      encode(e, node[u], step,
             [&](int i, T v) { bstore<T, false>(dst, here[u], (uint32_t)i * planeB, v); });
  }
  // step s: the nodes at least s - 1 inside the region, from LDS, in place
#pragma unroll 1
  for (int s = 2; s <= nsteps; ++s) {
    const int m = s - 1;
    const uint32_t step = (uint32_t)(T0 + (uint64_t)s);
    __syncthreads();
    bool act[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int id = (int)threadIdx.x + u * NT, r = row0 + u * RSTEP;
      act[u] = r >= m && r < RS - m && col >= m && col < CW - m;
      if (!act[u]) continue;
      const T *p = &lds[0][0] + id;
      raw[u].set(0, p[0]);
#pragma unroll
      for (int i = 1; i < 9; ++i) {
        const int kn = i * NODES - cy(i) * CW - cx(i), ko = opp(i) * NODES;
        if constexpr (LABELS) raw[u].set(i, p[((w[u] >> (i - 1)) & 1u) ? ko : kn]);
        else raw[u].set(i, p[kn]);
      }
    }
    __syncthreads();  // every source has been read
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!act[u]) continue;
      const int id = (int)threadIdx.x + u * NT;
      const bool solid = LABELS && (w[u] & NODE_SOLID);
      R e[9];
#pragma unroll
      for (int i = 0; i < 9; ++i) e[i] = solid ? R(0) : (R)S::raw_dec(raw[u].get(i));
      bad = bad || !(fabs(scaled_drho<ST, R>(e)) < R(1e30));
      collide_node<ST, FEAT, PLM, R>(D, e, node[u], step);
      if (s < nsteps)
        encode(e, node[u], step, [&](int i, T v) { lds[i][id] = v; });
      else if (tx * ow + col - rim < nx && ty * oh + row0 + u * RSTEP - rim < ny &&
               !(SKIP && (uint32_t)(xu[u] - skip.x + (xu[u] < skip.x ? nx : 0)) < (uint32_t)skip.w &&
                 (uint32_t)(yu[u] - skip.y + (yu[u] < skip.y ? ny : 0)) < (uint32_t)skip.h))
        // ordinary stores: the lines that two tiles share merge in the cache
        encode(e, node[u], step,
               [&](int i, T v) { bstore<T, false>(dst, here[u], (uint32_t)i * planeB, v); });
    }
  }
  if (bad) atomicOr(D.health, HEALTH_NONFINITE);
}

// One domain, its descriptor in the kernel's arguments: without the load of
// the descriptor the chain of dependent loads is one shorter, 0.6 us of the
// 7 that a launch takes on a small lattice.  A single step also comes here
// (channel 128 x 64 FP64, 20 calls of one step and the moments: 125 -> 89 us).
//
// With `advance`, the launch is the last of its call and also moves the step
// counter on, by the workgroup that arrives last at `arrived` (which it leaves
// at zero): all have read the counter then.  It spares a launch of 2 us; a
// workgroup's arrival is an atomic on one address for the whole device, so
// only small grids do it.
template <int ST, int FEAT, int PLM, int K>
__global__ __launch_bounds__(region(K).nt) void k_multi_one(const DevDomain D, uint32_t *arrived,
                                                            int kstep, int nsteps, int advance) {
  __shared__ typename Store<ST>::T lds[9][region(K).cw * region(K).rs];
  const uint64_t T0 = uniform_time(D, kstep);
  uint32_t place = 0;
  if (advance) {
    __syncthreads();
    if (threadIdx.x == 0)
      place = __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  multi_body<ST, FEAT, PLM, K, region(K).nt, false, true>(D, lds, xcd_remap((int)blockIdx.x, (int)gridDim.x), T0,
                                            nsteps);
  if (advance && threadIdx.x == 0 && place == gridDim.x - 1) {
    *arrived = 0;
    *D.tstep = T0 - (uint64_t)kstep + (uint64_t)advance;
  }
}

// The domains of a batch (prefix: tiles of nsteps-step launches per domain).
template <int ST, int FEAT, int PLM, int K>
__global__ __launch_bounds__(multi_threads(ST, K, FEAT), multi_threads(ST, K, FEAT) / 128) void k_multi(
    const DevDomain *__restrict__ doms, const int *__restrict__ prefix, int ndom, int kstep, int nsteps) {
  __shared__ typename Store<ST>::T lds[9][region(K).cw * region(K).rs];
  const int b = xcd_remap((int)blockIdx.x, (int)gridDim.x);
  const int dix = ndom == 1 ? 0 : find_domain(prefix, ndom, b);
  const DevDomain D = doms[dix];  // held in scalar registers across the steps
  multi_body<ST, FEAT, PLM, K, multi_threads(ST, K, FEAT)>(
      D, lds, ndom == 1 ? b : b - prefix[dix], uniform_time(D, kstep), nsteps);
}

}  // namespace lbk
