// Two red-black sweeps on cubes held in LDS, for levels whose plane march is
// latency-bound: W = sweep(sweep(S (+ P x_c))), one launch, bitwise the result
// of two fused sweeps.
//
// The marching kernels (gmg_sweep.h, gmg_sweep2.h) pay one memory latency and
// one barrier per plane of their march: 10-13 us a launch on 64^3 and 32^3
// whatever the tile, with data that sits in the caches.  Here a workgroup
// loads an 8 x 8 x 8 cube of cells and its halo of four cells at once (one
// memory latency), does the four half-sweeps in place in LDS, each one cell
// ring narrower than the one before (a colour's cells depend only on the
// other colour), and stores the cube.  The halo is recomputed by neighbouring
// cubes: 8 times the cells, which costs less than the march on levels of few
// cubes (cube_level has the measurements).
//
// A thread owns an x-pair column of four planes: x lives in LDS, sigma and the
// faces of its eight cells in registers.  Cells outside a wall hold zeros
// (their faces are zero and relax_cell leaves them at their input), as in the
// other kernels, and every update is relax_cell on the same operands.
#pragma once

#include <type_traits>

#include "gmg_sweep.h"  // wrap_coord, ldv, ldLv (and gmg_device.h)

namespace gmg {

constexpr int CU_B = 8;                // cube edge
constexpr int CU_H = 4;                // halo
constexpr int CU_R = CU_B + 2 * CU_H;  // edge of the loaded region
constexpr int CU_P = CU_R / 2;         // x-pairs per row
constexpr int CU_G = 4;                // groups of planes, one per thread of a column
constexpr int CU_NT = CU_P * CU_R * CU_G;  // 512 threads

template <typename T, int RZ>
struct CubeSmem {
  T x[RZ][CU_R][CU_R + 2];
};

// VEC = 2 for an even nx (a pair never straddles the edge: 2-wide loads and
// stores), else 1.  BZ: planes of the cube, 8 or 4; half cubes where whole ones
// leave CUs idle, since the half-sweeps' arithmetic is most of a launch (FP64
// above all, which divides): a launch on 32^3 FP64 takes 8.7 us with halves, 10
// with whole cubes, on 30x22x18 FP32 7-9 and 8-10.
// SPARE: the cycles recorded for a refinement step, of which most may find its
// solve finished: a finished slot of 256 x 64 x 64 takes 42 us with the test of the
// flag behind the loads, 25 with it in front.  Behind them it shares their latency,
// which a solve's few slots beyond its end do not outweigh (solve 32^3 FP64 641 us
// so, 649 in front; a run-time choice costs a launch 0.3 us).
template <typename T, typename TL, int VEC, bool PROL, int BZ, bool SPARE>
__global__ __launch_bounds__(CU_NT) void k_rb_cube(
    Geom g, Roles<T> X, int rs, int rd, const T* __restrict__ sigma, const TL* __restrict__ L,
    const T* __restrict__ xc, const uint8_t* __restrict__ active, Geom gc, int cx, int cy, int cz,
    const double* omega_p, const int* done) {
  constexpr int RZ = BZ + 2 * CU_H, CU_Z = RZ / CU_G;  // region planes, planes per thread
  static_assert(RZ % CU_G == 0, "planes divide among the groups");
  if constexpr (SPARE)
    if (stopped(done)) return;
  __shared__ CubeSmem<T, RZ> sm;
  const T* __restrict__ S = X.get(rs);
  T* const W = X.get(rd);
  const int nbx = (g.nx + CU_B - 1) / CU_B, nby = (g.ny + CU_B - 1) / CU_B;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int i0 = (t % nbx) * CU_B, j0 = (t / nbx) % nby * CU_B, k0 = t / (nbx * nby) * BZ;
  // a wave holds eight rows of one parity, so that the colour of a half-sweep
  // picks the same element of every lane's pair
  const int p = threadIdx.x % CU_P, rr = threadIdx.x / CU_P % CU_R;
  const int par = __builtin_amdgcn_readfirstlane(rr / (CU_R / 2));
  const int r = 2 * (rr % (CU_R / 2)) + par;
  // the thread's first plane of the region, the same for a wave
  const int z0 = __builtin_amdgcn_readfirstlane(threadIdx.x / (CU_P * CU_R)) * CU_Z;
  const int xa = i0 - CU_H + 2 * p, y = j0 - CU_H + r;
  // in-plane offsets of the pair (-1 outside a wall), of the column to its
  // east and of the row above
  const int jj = wrap_coord(y, g.ny, g.py), jn = wrap_coord(y + 1, g.ny, g.py);
  const int ii0 = wrap_coord(xa, g.nx, g.px), ii1 = wrap_coord(xa + 1, g.nx, g.px);
  const int ie = wrap_coord(xa + 2, g.nx, g.px);
  const TL* const Lx = L;
  const TL* const Ly = L + g.n;
  const TL* const Lz = L + 2 * g.n;
  T s[CU_Z][2], sg[CU_Z][2], lx[CU_Z][2], lxe[CU_Z], ly[CU_Z][2], lyh[CU_Z][2], lz[CU_Z + 1][2];
  // Every load is issued, at a clamped in-domain address where its cell lies
  // outside a wall; the value is then taken as zero.
  const int cj = jj >= 0 ? jj : 0, cn = jn >= 0 ? jn : 0;
  const int c0 = ii0 >= 0 ? ii0 : 0, c1 = ii1 >= 0 ? ii1 : 0, ce = ie >= 0 ? ie : 0;
  const bool in0 = jj >= 0 && ii0 >= 0, in1 = jj >= 0 && ii1 >= 0;
  const bool n0 = jn >= 0 && ii0 >= 0, n1 = jn >= 0 && ii1 >= 0, ine = jj >= 0 && ie >= 0;
  const long long o0 = (long long)cj * g.sy + c0, o1 = (long long)cj * g.sy + c1;
  const long long m0 = (long long)cn * g.sy + c0, m1 = (long long)cn * g.sy + c1;
  const long long oe = (long long)cj * g.sy + ce;
#pragma unroll
  for (int z = 0; z < CU_Z; ++z) {
    const int kw = wrap_coord(k0 - CU_H + z0 + z, g.nz, g.pz);
    const bool zin = kw >= 0;
    const long long zo = (long long)(zin ? kw : 0) * g.sz;
    if constexpr (VEC == 2) {
      ldv<T, 2>(S, zo + o0, s[z]);
      ldv<T, 2>(sigma, zo + o0, sg[z]);
      ldLv<T, 2>(Lx, zo + o0, lx[z]);
      ldLv<T, 2>(Ly, zo + o0, ly[z]);
      ldLv<T, 2>(Ly, zo + m0, lyh[z]);
      ldLv<T, 2>(Lz, zo + o0, lz[z]);
    } else {
      s[z][0] = S[zo + o0];
      s[z][1] = S[zo + o1];
      sg[z][0] = sigma[zo + o0];
      sg[z][1] = sigma[zo + o1];
      lx[z][0] = ldL<T>(Lx, zo + o0);
      lx[z][1] = ldL<T>(Lx, zo + o1);
      ly[z][0] = ldL<T>(Ly, zo + o0);
      ly[z][1] = ldL<T>(Ly, zo + o1);
      lyh[z][0] = ldL<T>(Ly, zo + m0);
      lyh[z][1] = ldL<T>(Ly, zo + m1);
      lz[z][0] = ldL<T>(Lz, zo + o0);
      lz[z][1] = ldL<T>(Lz, zo + o1);
    }
    lxe[z] = ldL<T>(Lx, zo + oe);
    s[z][0] = zin && in0 ? s[z][0] : T(0);
    s[z][1] = zin && in1 ? s[z][1] : T(0);
    sg[z][0] = zin && in0 ? sg[z][0] : T(0);
    sg[z][1] = zin && in1 ? sg[z][1] : T(0);
    lx[z][0] = zin && in0 ? lx[z][0] : T(0);
    lx[z][1] = zin && in1 ? lx[z][1] : T(0);
    lxe[z] = zin && ine ? lxe[z] : T(0);
    ly[z][0] = zin && in0 ? ly[z][0] : T(0);
    ly[z][1] = zin && in1 ? ly[z][1] : T(0);
    lyh[z][0] = zin && n0 ? lyh[z][0] : T(0);
    lyh[z][1] = zin && n1 ? lyh[z][1] : T(0);
    lz[z][0] = zin && in0 ? lz[z][0] : T(0);
    lz[z][1] = zin && in1 ? lz[z][1] : T(0);
    if constexpr (PROL) {
      const long long crow = (long long)((zin ? kw : 0) >> (cz >> 1)) * gc.sz +
                             (long long)(cj >> (cy >> 1)) * gc.sy;
      const T p0 = xc[crow + (c0 >> (cx >> 1))], p1 = xc[crow + (c1 >> (cx >> 1))];
      const bool a0 = active[zo + o0] != 0, a1 = active[zo + o1] != 0;
      if (zin && in0 && a0) s[z][0] += p0;
      if (zin && in1 && a1) s[z][1] += p1;
    }
  }
  {  // the z faces above the last plane
    const int kw = wrap_coord(k0 - CU_H + z0 + CU_Z, g.nz, g.pz);
    const long long zo = (long long)(kw >= 0 ? kw : 0) * g.sz;
    if constexpr (VEC == 2) {
      ldLv<T, 2>(Lz, zo + o0, lz[CU_Z]);
    } else {
      lz[CU_Z][0] = ldL<T>(Lz, zo + o0);
      lz[CU_Z][1] = ldL<T>(Lz, zo + o1);
    }
    lz[CU_Z][0] = kw >= 0 && in0 ? lz[CU_Z][0] : T(0);
    lz[CU_Z][1] = kw >= 0 && in1 ? lz[CU_Z][1] : T(0);
  }
  const T omega = (T)(*omega_p);
  if (stopped(done)) return;
#pragma unroll
  for (int z = 0; z < CU_Z; ++z) {
    sm.x[z0 + z][r][2 * p] = s[z][0];
    sm.x[z0 + z][r][2 * p + 1] = s[z][1];
  }
  __syncthreads();
  // half-sweep h: colour h & 1, the cube grown by 3 - h cells.  Region origins
  // are even: x + y + z of element e on the thread's plane z has the parity of
  // e + par + z0 + z, parc that of par + z0.
  auto half = [&](auto hc, auto parc) {
    constexpr int h = decltype(hc)::value;
    // region coordinates updated: [lo, hi), planes [lo, hz)
    constexpr int lo = 1 + h, hi = CU_R - 1 - h, hz = RZ - 1 - h;
    if (r < lo || r >= hi) return;
#pragma unroll
    for (int z = 0; z < CU_Z; ++z) {
      constexpr int SY = CU_R + 2, SZ = CU_R * SY;
      const int e = (decltype(parc)::value + z + h) & 1;  // known at compile time
      const int zr = z0 + z, c = 2 * p + e;
      if (zr < lo || zr >= hz || c < lo || c >= hi) continue;
      T* const q = &sm.x[zr][r][c];
      q[0] = relax_cell<T>(q[0], q[1], q[-1], q[SY], q[-SY], q[SZ], q[-SZ], lx[z][e],
                           e ? lxe[z] : lx[z][1], ly[z][e], lyh[z][e], lz[z][e], lz[z + 1][e],
                           sg[z][e], omega);
    }
  };
  auto sweeps = [&](auto parc) {
    half(std::integral_constant<int, 0>{}, parc);
    __syncthreads();
    half(std::integral_constant<int, 1>{}, parc);
    __syncthreads();
    half(std::integral_constant<int, 2>{}, parc);
    __syncthreads();
    half(std::integral_constant<int, 3>{}, parc);
  };
  if ((par + z0) & 1)
    sweeps(std::integral_constant<int, 1>{});
  else
    sweeps(std::integral_constant<int, 0>{});
  // the cube: each thread stores the cells it updated
  if (r < CU_H || r >= CU_H + CU_B || p < CU_H / 2 || p >= (CU_H + CU_B) / 2 || y >= g.ny) return;
#pragma unroll
  for (int z = 0; z < CU_Z; ++z) {
    const int zr = z0 + z, k = k0 - CU_H + zr;
    if (zr < CU_H || zr >= CU_H + BZ || k >= g.nz) continue;
    const long long q = (long long)k * g.sz + (long long)y * g.sy + xa;
    if constexpr (VEC == 2) {
      if (xa >= g.nx) continue;
      if constexpr (sizeof(T) == 4)
        *reinterpret_cast<float2*>(W + q) =
            make_float2(sm.x[zr][r][2 * p], sm.x[zr][r][2 * p + 1]);
      else
        *reinterpret_cast<double2*>(W + q) =
            make_double2(sm.x[zr][r][2 * p], sm.x[zr][r][2 * p + 1]);
    } else {
      if (xa < g.nx) W[q] = sm.x[zr][r][2 * p];
      if (xa + 1 < g.nx) W[q + 1] = sm.x[zr][r][2 * p + 1];
    }
  }
}

}  // namespace gmg
