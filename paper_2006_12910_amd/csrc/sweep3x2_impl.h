// sweep3x2_impl.h -- two time steps of a D3Q19 / D3Q27 domain per pass over
// the population buffers (FP32 and FP64 storage; BGK or TRT, with or without
// the power law; no noise).
//
// What bounds a single step is memory: 5.0-5.7 TB/s of populations in and
// out, at a quarter of the vector issue rate.  Two steps a pass read and
// write each population once per two steps, plus the rim.
//
// A workgroup owns a column of 64 x (RY - 2) nodes and walks it along z: one
// wave per row of the first step (RY rows: the outputs and one on either
// side) and one more for the two rim columns, so that rows stay 64 aligned
// lanes and every store a whole line (62 output columns with the rim in lanes
// 0 and 63 took a fifth more lanes on nx = 192 and 256).  Every iteration computes the first step of one z plane from global
// memory, exactly as k_sweep3 does, rounds it to the storage format, and
// hands it to the neighbouring columns through LDS.  What a node pulls from
// it completes the output plane behind it (e_z = -1) and starts the next two
// (e_z = 0, +1), which wait in registers; the completed plane is collided a
// second time and stored.  LDS then holds one plane (the e_z = +1 directions
// two, for the walk's second plane and for bounced pulls): 42.5 KB in FP32 on
// D3Q19 at RY = 7, two workgroups a CU; three whole planes would take 105.
// Every node of both steps goes through the same pull, collision and rounding
// as in k_sweep3, so the result is bit-identical to two single steps.
//
// Measured (192 x 192 x 130, us a step, single step / this): FP32 D3Q19 127.6
// / 91.8, D3Q27 190.5 / 137.7, FP64 270 / 163 and 395 / 237.  Without
// collisions FP32 D3Q19 takes 186 us a launch, without loads and stores 98:
// bound by the memory path still.  RY = 15 (one workgroup of 16 waves a CU)
// 95 open, 144 against 129 with solids; RY = 9, 11 between.
//
// A launch leaves the state in the buffer of the other parity, so launches come
// in pairs (`which` = 0 then 1).
#pragma once

#include "step_plan3.h"
#include "sweep3_impl.h"

namespace lbk3 {

// columns of a tile's first step: one more on either side
constexpr int X2_PITCH = X2_COLS + 2;

// LDS planes of one workgroup: the directions with e_z = +1 twice (the plane
// at hand and the one before), the other moving ones once.  A table: the
// loops over directions unroll to constants only if nothing is left to
// evaluate in them.
template <int Q> struct X2Planes {
  int of[Q];   // first LDS plane of direction i
  int up;      // planes of one e_z = +1 set (the second set follows it)
  int total;
};
template <int Q> constexpr X2Planes<Q> x2_planes() {
  X2Planes<Q> m{};
  int n = 0;
  for (int i = 1; i < Q; ++i)
    if (ez(i) > 0) m.of[i] = n++;
  m.up = n;
  n *= 2;
  for (int i = 1; i < Q; ++i)
    if (ez(i) <= 0) m.of[i] = n++;
  m.total = n;
  return m;
}

// RY rows of the first step (RY - 2 of outputs), RY + 1 waves
// TR: 0 BGK, 1 TRT
template <int ST, bool SOLIDS, int Q, bool PL, int TR, int RY, int WAVES>
__global__ __launch_bounds__(64 * (RY + 1), WAVES) void k_sweep3x2(const Dom3 D, int kstep,
                                                                   int which, int sz) {
  static_assert(RY <= 32, "the rim wave holds two columns");
  using S = S3<ST>;
  using T = typename S::T;
  using R = typename S::R;
  constexpr uint32_t E = sizeof(T);
  constexpr X2Planes<Q> M = x2_planes<Q>();
  constexpr int PLANE = RY * X2_PITCH, UP = M.up * PLANE;
  __shared__ T lds[M.total * PLANE];
  const int nx = D.nx, ny = D.ny, nz = D.nz, pitch = D.pitch;
  const int tiles_x = (nx + X2_COLS - 1) / X2_COLS, tiles_y = (ny + RY - 3) / (RY - 2);
  const int b = tile_order3<false>((int)blockIdx.x, (int)gridDim.x);
  const int seg = b / (tiles_x * tiles_y), t = b - seg * (tiles_x * tiles_y);
  const int ty = t / tiles_x, tx = t - ty * tiles_x;
  const int lane = (int)threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int z0 = seg * sz, n = nz - z0 < sz ? nz - z0 : sz;

  auto wrap = [](int c, int m) {
    c %= m;
    return c < 0 ? c + m : c;
  };
  // waves 0 .. RY - 1 hold a row of 64 columns each, the last one the rim
  // columns (left in lanes 0 .., right in lanes 32 ..; lanes without a node
  // repeat the last row's)
  const bool rim = wave == RY;
  const int r = rim ? ((lane & 31) < RY ? (lane & 31) : RY - 1) : wave;
  const int k = rim ? (lane < 32 ? 0 : X2_PITCH - 1) : lane + 1;
  const int xs = tx * X2_COLS + k - 1, ys = ty * (RY - 2) + r - 1;
  const int x = wrap(xs, nx), y = wrap(ys, ny);
  // the second step is taken by the inner rows (wave-uniform)
  const bool inner = wave >= 1 && wave <= RY - 2 && ty * (RY - 2) + wave - 1 < ny;
  const bool out = xs < nx;

  const uint64_t ts = *lbk::gbl(D.tstep);
  const uint64_t T0 =
      (((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(ts >> 32)) << 32) |
       __builtin_amdgcn_readfirstlane((uint32_t)ts)) + (uint64_t)kstep;
  const bool odd = ((T0 + (uint64_t)which) & 1) != 0;
  const uint32_t rowb = (uint32_t)pitch * E, zb = (uint32_t)ny * rowb, popb = (uint32_t)nz * zb;
  const Res3 rs = res3(odd ? D.f[1] : D.f[0], (uint32_t)Q * popb);
  const Res3 rd = res3(odd ? D.f[0] : D.f[1], (uint32_t)Q * popb);
  // byte offsets of the nine nodes around (x, y) in a z plane, by the
  // direction that pulls from there: [1 + e_x][1 + e_y]
  uint32_t off[3][3];
  {
    const int xn[3] = {x + 1 < nx ? x + 1 : 0, x, x > 0 ? x - 1 : nx - 1};
    const int yn[3] = {y + 1 < ny ? y + 1 : 0, y, y > 0 ? y - 1 : ny - 1};
#pragma unroll
    for (int i = 0; i < 9; ++i)
      off[i / 3][i % 3] = (uint32_t)yn[i % 3] * rowb + (uint32_t)xn[i / 3] * E;
  }

  auto word = [&](int z) -> uint32_t {
    if constexpr (SOLIDS) return lbk::gbl(D.nodew)[((uint32_t)z * (uint32_t)ny + (uint32_t)y) * (uint32_t)pitch + (uint32_t)x];
    else return 0u;
  };
  // every pull of node (x, y, z); the scalar offset carries the population
  // and z plane, the vector offset the place in the plane.  A bounced pull
  // reads the node's own opposite slot: opposite directions lie one
  // population plane apart, so which of the two scalar offsets is smaller is
  // known at compile time and the difference rides on the vector offset,
  // picked by a mask (one three-input bitwise instruction).
  auto pull = [&](int z, uint32_t w, T (&raw)[Q]) {
    const uint32_t zo[3] = {(uint32_t)(z + 1 < nz ? z + 1 : 0) * zb, (uint32_t)z * zb,
                            (uint32_t)(z > 0 ? z - 1 : nz - 1) * zb};
    raw[0] = ld3<T>(rs, off[1][1], zo[1]);
#pragma unroll
    for (int i = 1; i < Q; ++i) {
      const uint32_t sN = (uint32_t)i * popb + zo[1 + ez(i)];
      const uint32_t vN = off[1 + ex(i)][1 + ey(i)];
      if constexpr (!SOLIDS) {
        raw[i] = ld3<T>(rs, vN, sN);
      } else {
        const uint32_t sB = (uint32_t)opp(i) * popb + zo[1], vB = off[1][1];
        // all ones where the pull bounces (the empty asm keeps the mux from
        // becoming a compare and a select)
        uint32_t m = (uint32_t)(-(int32_t)((w >> (i - 1)) & 1u));
        const uint32_t d = __builtin_amdgcn_readfirstlane((i & 1) ? sB - sN : sN - sB);
        __asm__("" : "+v"(m));
        const uint32_t a = (i & 1) ? vN : vN + d, c = (i & 1) ? vB + d : vB;
        raw[i] = ld3<T>(rs, a ^ ((a ^ c) & m), (i & 1) ? sN : sB);
      }
    }
  };
  bool bad = false;
  // collision of one node (no noise: the node number and step are unused)
  auto relax = [&](R (&d)[Q], bool solid) {
    collide3<R, Q, PL, 0, TR>(D, d, 0u, 0u);
    bad = bad || (!solid && !(fabs(d[0]) < R(1e30)));
  };

  // what the next output plane already has: c[i] of the directions with
  // e_z >= 0
  T c[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) c[i] = T(0);
  auto next = [&](int k) { return k + 1 < nz ? k + 1 : 0; };
  int z = z0 > 0 ? z0 - 1 : nz - 1, zp = z;
  uint32_t wp = 0u, wc = word(z), wn = word(next(z));
  T raw[Q];
  pull(z, wc, raw);
#pragma unroll
  for (int i = 0; i < Q; ++i) __asm__ volatile("" : "+v"(raw[i]));
#pragma unroll 1
  for (int it = 0; it < n + 2; ++it) {
    const int par = it & 1;
    // this node's place in LDS plane 0, and in the two buffers of the
    // e_z = +1 directions: of this plane, of the one before (hidden from the
    // optimiser, which would keep one address a direction across the loop)
    uint32_t me = (uint32_t)(r * X2_PITCH + k), up_now = me + (uint32_t)(par * UP),
             up_old = me + (uint32_t)((par ^ 1) * UP);
    __asm__ volatile("" : "+v"(me), "+v"(up_now), "+v"(up_old));
    T q0;
    {
      // first step of plane z.  A solid node's values are never read, so it
      // collides whatever it pulled.
      R d[Q];
#pragma unroll
      for (int i = 0; i < Q; ++i) d[i] = S::dec(raw[i], Q, i);
      relax(d, SOLIDS && (wc & NODE_SOLID3));
      __syncthreads();  // the plane before has been read
      q0 = S::enc(d[0], Q, 0, false, 0u);
#pragma unroll
      for (int i = 1; i < Q; ++i)
        lds[(ez(i) > 0 ? up_now : me) + M.of[i] * PLANE] = S::enc(d[i], Q, i, false, 0u);
    }
    // the pulls of the next plane fly while this one is exchanged and the
    // plane before takes its second step
    const int zn = next(z);
    const uint32_t w2 = word(next(zn));
    if (it < n + 1) pull(zn, wn, raw);
    __syncthreads();
    const bool solid = SOLIDS && (wp & NODE_SOLID3);
    R e[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) e[i] = R(0);
    if (inner) {
      // pull i of an output plane: the neighbour's value (its plane's
      // buffer base bn), or, bounced, the node's own opposite one (base bo).
      // The two lie a constant apart.
      auto get = [&](int i, uint32_t bn, uint32_t bo, uint32_t w) -> T {
        const int kn = M.of[i] * PLANE - ey(i) * X2_PITCH - ex(i);
        if constexpr (!SOLIDS) {
          return lds[bn + kn];
        } else {
          const int ko = M.of[opp(i)] * PLANE;
          const bool bounce = ((w >> (i - 1)) & 1u) != 0;
          return lds[bounce ? bo + ko : bn + kn];
        }
      };
      if (it >= 2) {
#pragma unroll
        for (int i = 0; i < Q; ++i) e[i] = S::dec(ez(i) >= 0 ? c[i] : get(i, me, up_old, wp), Q, i);
        relax(e, solid);
      }
      c[0] = q0;
#pragma unroll
      for (int i = 1; i < Q; ++i) {
        if (ez(i) == 0) c[i] = get(i, me, me, wc);
        if (ez(i) > 0) c[i] = get(i, up_old, me, wc);
      }
    }
    // The pulls have landed by now.  Waited for here, on every path, they
    // leave nothing to wait for behind the stores (loads and stores complete
    // in one order, so a wait at the top of the loop would be for both).
#pragma unroll
    for (int i = 0; i < Q; ++i) __asm__ volatile("" : "+v"(raw[i]));
    if (inner && it >= 2 && out) {
      // a solid node stores zero deviations
      auto store = [&](auto nt) {
#pragma unroll
        for (int i = 0; i < Q; ++i)
          st3<T, decltype(nt)::value>(rd, off[1][1], (uint32_t)i * popb + (uint32_t)zp * zb,
                                      solid ? T(0) : S::enc(e[i], Q, i, false, 0u));
      };
      if (D.stream) store(std::true_type{});
      else store(std::false_type{});
    }
    wp = wc;
    wc = wn;
    wn = w2;
    zp = z;
    z = zn;
  }
  if (bad) atomicOr(D.health, 1u);
}

}  // namespace lbk3
