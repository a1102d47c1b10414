// Coarse tail of the V-cycle in one workgroup.
//
// Below some size a level's sweep is pure latency: a fused-sweep launch on a
// 16^3 grid costs about as much as one on 128^3, and a V-cycle visits the
// small levels with a dozen launches.  Here one workgroup of kTailThreads
// threads runs everything from the first tail level down: pre-sweeps,
// residual restriction, the coarsest-level smoothing, prolongation +
// correction and post-sweeps, with workgroup barriers in place of kernel
// boundaries.  Tail levels (x, sigma, faces, active mask) are held in LDS for
// the whole launch and x and sigma go back to global memory at the end; a
// level too large for LDS (only ever the coarsest one, alone) is worked on
// in global memory by the same code.
//
// The coarsest level is smoothed either by nu_coarse sweeps or, with
// coarse_rtol > 0, in groups of nu_coarse sweeps until its residual norm has
// fallen to coarse_rtol times its value on entry (at most coarse_max): the paper's
// anisotropic coarsening (Sec. 3.2) reaches a coarsest grid on which the
// smoother alone removes the lowest wavenumbers, and this rule lets it do
// so.  The rule first removes the mean of the level's right-hand side over
// its active cells (zero in exact arithmetic on these singular levels; what
// rounding leaves there no sweep can remove), and its norms are FP64 sums in
// a fixed order.
//
// Arithmetic is that of the grid-wide kernels: the same relax_cell per cell,
// colour by colour (a colour's cells depend only on the other colour, so an
// in-place half-sweep equals the simultaneous one), the residual from
// stencil_Ax, and the restriction sum of each coarse cell taken in the order
// of the tiled restriction kernel (z first per fine column, then x-pairs,
// then y-pairs).  With one workgroup per problem the same body serves a batch
// of independent problems (k_tail_batch).
#pragma once

#include "gmg_device.h"

namespace gmg {

constexpr int kTailThreads = 1024;
constexpr int kTailMax = 8;                // levels the tail can hold
constexpr int kTailLds = 156 * 1024;       // LDS budget of the tail (bytes)

template <typename T, typename TL>
struct TailLevel {
  Geom g;
  T* x;             // global x (written back at the end)
  T* sigma;         // global sigma (read for the first level, written back)
  const TL* L;      // global faces
  const uint8_t* active;
  int cx, cy, cz;   // factors to the next level
  int ox, os, oL, oa;  // byte offsets of x, sigma, faces, mask in LDS
  int reg;          // pairs per thread of the register-resident smoothing (0: from LDS)
};

template <typename T, typename TL>
struct TailArgs {
  TailLevel<T, TL> lv[kTailMax];
  int nl;  // levels in the tail; the last is the coarsest
  int nu_pre, nu_post, nu_coarse;
  double coarse_rtol;  // > 0: the coarsest-level stopping rule (see above)
  int coarse_max;
  const double* omega;  // relaxation factor (device)
  const int* done;      // solve finished: the launch is a no-op (may be NULL)
  int* sweeps;          // receives the coarsest level's sweep count (may be NULL)
};

// LDS bytes of one level: x, sigma (T), three faces (TL), mask, each part
// rounded up to 16 bytes.
__host__ __device__ inline int tail_round16(long long b) { return (int)((b + 15) & ~15LL); }
template <typename T, typename TL>
__host__ __device__ inline int tail_level_bytes(long long n) {
  return 2 * tail_round16(n * (long long)sizeof(T)) + tail_round16(3 * n * (long long)sizeof(TL)) +
         tail_round16(n);
}

// a / b for 0 <= a < 2^22, b >= 1, from a float reciprocal and one fix-up.
__device__ __forceinline__ int tail_div(int a, int b, float rb) {
  int q = (int)((float)a * rb);
  const int r = a - q * b;
  if (r < 0) --q;
  else if (r >= b) ++q;
  return q;
}

template <typename T, typename TL>
struct TailView {  // one level in LDS
  Geom g;
  T* x;
  T* s;
  TL* L;
  uint8_t* a;
};

// GLOBAL: the level is used in place in global memory; otherwise it lives in
// LDS at its offsets.  A compile-time choice, so that the LDS pointers are
// known to be LDS pointers and the accesses become LDS instructions.
template <typename T, typename TL, bool GLOBAL>
__device__ __forceinline__ TailView<T, TL> tail_view(char* lds, const TailLevel<T, TL>& v) {
  if constexpr (GLOBAL)
    return TailView<T, TL>{v.g, v.x, v.sigma, const_cast<TL*>(v.L),
                           const_cast<uint8_t*>(v.active)};
  return TailView<T, TL>{v.g, (T*)(lds + v.ox), (T*)(lds + v.os), (TL*)(lds + v.oL),
                         (uint8_t*)(lds + v.oa)};
}

// One half-sweep of colour `colour` ((i + j + k) mod 2), in place: thread
// work items are x-pairs of a row, each holding exactly one cell per colour.
template <typename T, typename TL>
__device__ __forceinline__ void tail_half_sweep(const TailView<T, TL>& v, int colour, T omega) {
  const Geom& g = v.g;
  const int nx = g.nx, ny = g.ny;
  const int sy = nx, sz = nx * ny, n = sz * g.nz;
  const int pr = (nx + 1) >> 1;
  const int np = pr * ny * g.nz;
  const float rpr = 1.0f / (float)pr, rny = 1.0f / (float)ny;
  const TL* Lx = v.L;
  const TL* Ly = v.L + n;
  const TL* Lz = v.L + 2 * n;
  T* x = v.x;
  for (int p = threadIdx.x; p < np; p += kTailThreads) {
    const int row = tail_div(p, pr, rpr);
    const int m = p - row * pr;
    const int k = tail_div(row, ny, rny);
    const int j = row - k * ny;
    const int i = 2 * m + ((j + k + colour) & 1);
    if (i >= nx) continue;
    const int q = row * nx + i;
    // neighbours: wrap when periodic; outside a wall value and high face are 0
    const bool xe_in = i + 1 < nx || g.px, xw_in = i > 0 || g.px;
    const bool yn_in = j + 1 < ny || g.py, ys_in = j > 0 || g.py;
    const bool zt_in = k + 1 < g.nz || g.pz, zb_in = k > 0 || g.pz;
    const int qe = (i + 1 < nx) ? q + 1 : q - (nx - 1);
    const int qw = (i > 0) ? q - 1 : q + (nx - 1);
    const int qn = (j + 1 < ny) ? q + sy : q - (ny - 1) * sy;
    const int qs = (j > 0) ? q - sy : q + (ny - 1) * sy;
    const int qt = (k + 1 < g.nz) ? q + sz : q - (g.nz - 1) * sz;
    const int qb = (k > 0) ? q - sz : q + (g.nz - 1) * sz;
    x[q] = relax_cell<T>(x[q], xe_in ? x[qe] : T(0), xw_in ? x[qw] : T(0), yn_in ? x[qn] : T(0),
                         ys_in ? x[qs] : T(0), zt_in ? x[qt] : T(0), zb_in ? x[qb] : T(0),
                         ldL<T>(Lx, q), xe_in ? ldL<T>(Lx, qe) : T(0), ldL<T>(Ly, q),
                         yn_in ? ldL<T>(Ly, qn) : T(0), ldL<T>(Lz, q),
                         zt_in ? ldL<T>(Lz, qt) : T(0), v.s[q], omega);
  }
  __syncthreads();
}

template <typename T, typename TL>
__device__ __forceinline__ void tail_sweeps(const TailView<T, TL>& v, int nsw, T omega) {
  for (int s = 0; s < nsw; ++s) {
    tail_half_sweep<T, TL>(v, 0, omega);
    tail_half_sweep<T, TL>(v, 1, omega);
  }
}

// Sum over the cz fine planes of coarse plane K of the residual of fine
// column (i, j), active cells only.
template <typename T, typename TL>
__device__ __forceinline__ T tail_column_residual(const TailView<T, TL>& f, int cz, int i, int j,
                                                  int K) {
  const Geom& g = f.g;
  T acc = T(0);
  for (int dz = 0; dz < cz; ++dz) {
    const int k = K * cz + dz;
    const long long idx = (long long)k * g.sz + (long long)j * g.sy + i;
    const T xc = f.x[idx];
    T D;
    const T ax = stencil_Ax<T, TL>(g, f.x, f.L, idx, i, j, k, xc, D);
    if (D != T(0)) acc += f.s[idx] - ax;
  }
  return acc;
}

// sigma_c = R (sigma - A x) on the next level and x_c = 0.
template <typename T, typename TL>
__device__ __forceinline__ void tail_restrict(const TailView<T, TL>& f, const TailLevel<T, TL>& fl,
                                              const TailView<T, TL>& c) {
  const Geom& gc = c.g;
  const int ncell = (int)gc.n;
  const float rnx = 1.0f / (float)gc.nx, rny = 1.0f / (float)gc.ny;
  for (int q = threadIdx.x; q < ncell; q += kTailThreads) {
    const int row = tail_div(q, gc.nx, rnx);
    const int I = q - row * gc.nx;
    const int K = tail_div(row, gc.ny, rny);
    const int J = row - K * gc.ny;
    T r[2];
    for (int dy = 0; dy < fl.cy; ++dy) {
      const int j = J * fl.cy + dy;
      T a = tail_column_residual<T, TL>(f, fl.cz, I * fl.cx, j, K);
      if (fl.cx == 2) a += tail_column_residual<T, TL>(f, fl.cz, I * fl.cx + 1, j, K);
      r[dy] = a;
    }
    c.s[q] = (fl.cy == 2) ? r[0] + r[1] : r[0];
    c.x[q] = T(0);
  }
  __syncthreads();
}

// x += P x_c on active cells.
template <typename T, typename TL>
__device__ __forceinline__ void tail_prolong(const TailView<T, TL>& f, const TailLevel<T, TL>& fl,
                                             const TailView<T, TL>& c) {
  const Geom& g = f.g;
  const int ncell = (int)g.n;
  const float rnx = 1.0f / (float)g.nx, rny = 1.0f / (float)g.ny;
  for (int q = threadIdx.x; q < ncell; q += kTailThreads) {
    if (!f.a[q]) continue;
    const int row = tail_div(q, g.nx, rnx);
    const int i = q - row * g.nx;
    const int k = tail_div(row, g.ny, rny);
    const int j = row - k * g.ny;
    f.x[q] += c.x[(k / fl.cz) * (int)c.g.sz + (j / fl.cy) * (int)c.g.sy + i / fl.cx];
  }
  __syncthreads();
}

// A level is smoothed by a group of threads: the workgroup's first wavefront
// alone when the coarsest level's cells fill no more (between two half-sweeps
// a wavefront needs only its own memory operations completed: a fence, no
// barrier), else the whole workgroup.  The group's stride STRIDE names it; the
// mean of a level of at most kWaveCells cells is always taken by the wavefront.
constexpr int kWave = 64;
constexpr int kWaveCells = 256;

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

template <int STRIDE>
__device__ __forceinline__ void grp_sync() {
  if constexpr (STRIDE == kWave)
    wave_sync();
  else
    __syncthreads();
}

// Sum over the wavefront, the same fixed order in every lane's result.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// Sum over the group, the result in every thread (red: one LDS double).
template <int STRIDE>
__device__ __forceinline__ double grp_sum(double v, double* red) {
  if constexpr (STRIDE == kWave) {
    return wave_sum(v);
  } else {
    const double s = block_sum(v, threadIdx.x, STRIDE);
    if (threadIdx.x == 0) *red = s;
    __syncthreads();
    const double out = *red;
    __syncthreads();  // *red is reused by the next sum
    return out;
  }
}

// Sum over the wavefront in every lane's result: within rows of 16 lanes by
// DPP moves, then the four rows in order.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const int lo = (int)(uint32_t)u, hi = (int)(uint32_t)(u >> 32);
  const uint32_t l2 = (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
  const uint32_t h2 = (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
  return v + __builtin_bit_cast(double, (uint64_t)h2 << 32 | l2);
}
__device__ __forceinline__ double wave_sum_rows(double v) {
  v = dpp_add<0xB1>(v);   // quad: lanes 1 0 3 2
  v = dpp_add<0x4E>(v);   // quad: lanes 2 3 0 1
  v = dpp_add<0x141>(v);  // half row mirrored
  v = dpp_add<0x140>(v);  // row mirrored
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const int lo = (int)(uint32_t)u, hi = (int)(uint32_t)(u >> 32);
  double s = 0.0;
#pragma unroll
  for (int r = 0; r < kWave; r += 16)
    s += __builtin_bit_cast(double,
                            (uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi, r) << 32 |
                                (uint32_t)__builtin_amdgcn_readlane(lo, r));
  return s;
}

// Residual of cell q of a tail level (dtype arithmetic); `act` is D != 0.
template <typename T, typename TL>
__device__ __forceinline__ T tail_cell_residual(const TailView<T, TL>& v, int q, float rnx,
                                                float rny, bool& act) {
  const Geom& g = v.g;
  const int row = tail_div(q, g.nx, rnx);
  const int i = q - row * g.nx;
  const int k = tail_div(row, g.ny, rny);
  const int j = row - k * g.ny;
  T D;
  const T ax = stencil_Ax<T, TL>(g, v.x, v.L, q, i, j, k, v.x[q], D);
  act = D != T(0);
  return act ? v.s[q] - ax : T(0);
}

// ||sigma - A x||_2 over the active cells: FP64 squares of the dtype
// residuals summed per thread in cell order, then over the workgroup.
template <typename T, typename TL>
__device__ __forceinline__ double tail_resnorm(const TailView<T, TL>& v, double* red) {
  const Geom& g = v.g;
  const int ncell = (int)g.n;
  const float rnx = 1.0f / (float)g.nx, rny = 1.0f / (float)g.ny;
  double s2 = 0.0;
  for (int q = threadIdx.x; q < ncell; q += kTailThreads) {
    bool act;
    const T r = tail_cell_residual<T, TL>(v, q, rnx, rny, act);
    if (act) s2 += (double)r * (double)r;
  }
  return sqrt(grp_sum<kTailThreads>(s2, red));
}

// sigma -= its mean over the active cells (FP64 sum and mean, the
// difference rounded once to the dtype).  With walls and periodic
// directions only, every level is singular (constants are in the null
// space) and a right-hand side is solvable only with zero mean; the
// restricted residual has it in exact arithmetic, and this removes what
// rounding left, which the smoother could not reduce and which would drift
// the level's iterate along the null space.
template <typename T, typename TL, int STRIDE>
__device__ __forceinline__ void grp_project(const TailView<T, TL>& v, double* red) {
  const int ncell = (int)v.g.n;
  double s = 0.0, c = 0.0;
  for (int q = threadIdx.x; q < ncell; q += STRIDE)
    if (v.a[q]) {
      s += (double)v.s[q];
      c += 1.0;
    }
  s = grp_sum<STRIDE>(s, red);
  c = grp_sum<STRIDE>(c, red);
  const double mean = c > 0.0 ? s / c : 0.0;
  for (int q = threadIdx.x; q < ncell; q += STRIDE)
    if (v.a[q]) v.s[q] = (T)((double)v.s[q] - mean);
  grp_sync<STRIDE>();
}

// Smoothing of the coarsest level by the workgroup from LDS or global memory,
// for levels too large for registers: nu_coarse sweeps, or with coarse_rtol >
// 0 the right-hand side projected to zero mean, then sweeps in groups of
// max(1, nu_coarse), the residual norm checked after each, until it is at most
// coarse_rtol times its value on entry or coarse_max sweeps are done (the last
// group cut to fit).  Returns the number of sweeps.
template <typename T, typename TL>
__device__ __forceinline__ int plain_coarsest(const TailView<T, TL>& v, int nu_coarse,
                                              double coarse_rtol, int coarse_max, T omega,
                                              double* red) {
  if (!(coarse_rtol > 0.0)) {
    tail_sweeps<T, TL>(v, nu_coarse, omega);
    return nu_coarse;
  }
  grp_project<T, TL, kTailThreads>(v, red);
  const double lim = coarse_rtol * tail_resnorm<T, TL>(v, red);
  const int group = nu_coarse > 1 ? nu_coarse : 1;
  int n = 0;
  while (n < coarse_max) {
    const int k = min(group, coarse_max - n);
    tail_sweeps<T, TL>(v, k, omega);
    n += k;
    if (n < coarse_max && tail_resnorm<T, TL>(v, red) <= lim) break;
  }
  return n;
}

// Register-resident smoothing of a level by a group of STRIDE threads, for
// levels of at most NS x STRIDE x-pairs: each thread owns NS pairs, one cell of
// each colour, and keeps their x, faces, sigma, diagonal and neighbour addresses
// in registers from the first sweep to the last; x is also kept in LDS, one
// array per colour indexed by pair, so that a half-sweep reads five neighbours
// of the other colour at consecutive addresses (the sixth is the thread's own)
// and writes one value.  A half-sweep is bound by instruction issue of the one
// workgroup: working indices, wraps and faces out of LDS each time took about
// three times as long.  Measured on a V-cycle with a 15 x 11 x 9 coarsest level:
// tail 61 -> 27 us; on the tails of a batch of 64 problems 111 -> 34 us.  Every
// update rounds as relax_cell on the same operands, so the iterates are
// bitwise those of the plain half-sweeps.
constexpr int kRegPairsWave = 2 * kWave;        // pairs one wavefront takes
constexpr int kRegSlots = 2;                    // most pairs of a workgroup's thread
constexpr int kRegPad = 4;                      // the zero read beyond a wall, and padding
constexpr int kRegPairs = kRegSlots * kTailThreads;
__host__ __device__ constexpr int reg_colour(int slots, int stride) {  // elements of one colour
  return slots * stride + kRegPad;
}

template <typename T>
using LdsPtr = __attribute__((address_space(3))) T*;

template <typename T>
struct TailPair {
  LdsPtr<T> own;                // colour 0's entry of this pair
  LdsPtr<const T> n, s, t, b;   // colour 0's entries of the y and z neighbours
  LdsPtr<const T> ext[2];       // by colour: the x neighbour in another pair
  T f[2][6];                    // by colour: low x, high x, low y, high y, low z, high z
  T sg[2], rd[2], x[2];         // rd: FP32 1 / D as relax_cell takes it, FP64 D
  int q;                        // the pair's first cell, -1: none
  bool first;                   // the first cell of the pair has colour 0
  bool two;                     // the pair has a second cell
  bool on[2];                   // by colour: the cell exists and D != 0
};

template <typename T, typename TL, int NS, int STRIDE>
struct TailRegs {
  static constexpr int CS = reg_colour(NS, STRIDE);
  TailPair<T> a[NS];

  // Takes the level's x (with the prolonged correction x += P x_c on active
  // cells if PROL), faces and sigma; x's place in LDS (xs) may be v.x itself.
  template <bool PROL>
  __device__ __forceinline__ void load(const TailView<T, TL>& v, T* xs,
                                       const TailLevel<T, TL>* fl, const TailView<T, TL>* cv) {
    const Geom& g = v.g;
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const int sy = nx, sz = nx * ny, n = sz * nz;
    const int pr = (nx + 1) >> 1, pz = pr * ny;
    const float rpr = 1.0f / (float)pr, rny = 1.0f / (float)ny;
    const LdsPtr<T> c0 = (LdsPtr<T>)xs;
    const LdsPtr<const T> zero = c0 + (CS - 1);
#pragma unroll
    for (int it = 0; it < NS; ++it) {
      TailPair<T>& P = a[it];
      const int p = threadIdx.x + it * STRIDE;
      P.q = -1;
      P.two = false;
      P.first = true;
      P.own = c0 + p;
      P.n = P.s = P.t = P.b = P.ext[0] = P.ext[1] = zero;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        P.on[c] = false;
        P.x[c] = P.sg[c] = P.rd[c] = T(0);
#pragma unroll
        for (int d = 0; d < 6; ++d) P.f[c][d] = T(0);
      }
      if (p >= pz * nz) continue;
      const int row = tail_div(p, pr, rpr);
      const int m = p - row * pr;
      const int k = tail_div(row, ny, rny);
      const int j = row - k * ny;
      P.q = row * nx + 2 * m;
      P.two = 2 * m + 1 < nx;
      P.first = ((j + k) & 1) == 0;
      // neighbours in the pair grid (periodic sizes are even); beyond a wall the zero
      const bool ny_in = j + 1 < ny || g.py, sy_in = j > 0 || g.py;
      const bool tz_in = k + 1 < nz || g.pz, bz_in = k > 0 || g.pz;
      if (ny_in) P.n = P.own + (j + 1 < ny ? pr : -(ny - 1) * pr);
      if (sy_in) P.s = P.own + (j > 0 ? -pr : (ny - 1) * pr);
      if (tz_in) P.t = P.own + (k + 1 < nz ? pz : -(nz - 1) * pz);
      if (bz_in) P.b = P.own + (k > 0 ? -pz : (nz - 1) * pz);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const bool lo = P.first == (c == 0);  // the pair's first cell
        if (!lo && !P.two) continue;
        const int i = 2 * m + (lo ? 0 : 1);
        const int q = row * nx + i;
        const bool e_in = i + 1 < nx || g.px, w_in = i > 0 || g.px;
        if (lo && w_in) P.ext[c] = P.own + (m > 0 ? -1 : pr - 1);
        if (!lo && e_in) P.ext[c] = P.own + (m + 1 < pr ? 1 : -(pr - 1));
        const int qe = (i + 1 < nx) ? q + 1 : q - (nx - 1);
        const int qn = (j + 1 < ny) ? q + sy : q - (ny - 1) * sy;
        const int qt = (k + 1 < nz) ? q + sz : q - (nz - 1) * sz;
        T* f = P.f[c];
        f[0] = ldL<T>(v.L, q);
        f[1] = e_in ? ldL<T>(v.L, qe) : T(0);
        f[2] = ldL<T>(v.L + n, q);
        f[3] = ny_in ? ldL<T>(v.L + n, qn) : T(0);
        f[4] = ldL<T>(v.L + 2 * n, q);
        f[5] = tz_in ? ldL<T>(v.L + 2 * n, qt) : T(0);
        const T s = ((f[0] + f[1]) + (f[2] + f[3])) + (f[4] + f[5]);
        P.on[c] = !(s == T(0));
        if constexpr (sizeof(T) == 4)
          P.rd[c] = __builtin_amdgcn_rcpf(-s);
        else
          P.rd[c] = -s;
        P.sg[c] = v.s[q];
        P.x[c] = v.x[q];
        if constexpr (PROL)
          if (v.a[q])
            P.x[c] += cv->x[(k >> (fl->cz >> 1)) * (int)cv->g.sz +
                            (j >> (fl->cy >> 1)) * (int)cv->g.sy + (i >> (fl->cx >> 1))];
      }
    }
    grp_sync<STRIDE>();  // v.x is read before its place is used
#pragma unroll
    for (int it = 0; it < NS; ++it) {
      a[it].own[0] = a[it].x[0];
      a[it].own[CS] = a[it].x[1];
    }
    if (threadIdx.x == 0) c0[CS - 1] = c0[2 * CS - 1] = T(0);
    grp_sync<STRIDE>();
  }

  // A x of the pair's cell of colour c, summed as relax_cell and stencil_Ax do.
  __device__ __forceinline__ static T flux(const TailPair<T>& P, int c) {
    const int o = (1 - c) * CS;
    const T xc = P.x[c];
    const bool lo = P.first == (c == 0);
    const T ex = P.ext[c][o], in = P.x[1 - c];
    const T xe = lo ? in : ex, xw = lo ? ex : in;
    T ax = T(0);
    ax += P.f[c][1] * (xe - xc);
    ax += P.f[c][0] * (xw - xc);
    ax += P.f[c][3] * (P.n[o] - xc);
    ax += P.f[c][2] * (P.s[o] - xc);
    ax += P.f[c][5] * (P.t[o] - xc);
    ax += P.f[c][4] * (P.b[o] - xc);
    return ax;
  }

  __device__ __forceinline__ void sweep(T omega) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
      for (int it = 0; it < NS; ++it) {
        TailPair<T>& P = a[it];
        if (!P.on[c]) continue;
        const T ax = flux(P, c);
        if constexpr (sizeof(T) == 4)
          P.x[c] = P.x[c] + omega * (P.sg[c] - ax) * P.rd[c];
        else
          P.x[c] = P.x[c] + omega * (P.sg[c] - ax) / P.rd[c];
        P.own[c * CS] = P.x[c];
      }
      grp_sync<STRIDE>();
    }
  }

  // ||sigma - A x||_2 over the active cells, the same in every thread; FP64
  // squares of the dtype residuals in a fixed order.  red: STRIDE / 64 doubles,
  // not read again until a sweep has passed.
  __device__ __forceinline__ double norm(double* red) const {
    double s2 = 0.0;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int it = 0; it < NS; ++it)
        if (a[it].on[c]) {
          const T r = a[it].sg[c] - flux(a[it], c);
          s2 += (double)r * (double)r;
        }
    s2 = wave_sum_rows(s2);
    if constexpr (STRIDE > kWave) {
      if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = s2;
      __syncthreads();
      s2 = 0.0;
#pragma unroll
      for (int w = 0; w < STRIDE / kWave; ++w) s2 += red[w];
    }
    return sqrt(s2);
  }

  // Puts val(pair, colour) of every cell in its place in the level's x.
  template <typename F>
  __device__ __forceinline__ void put(T* x, F&& val) const {
#pragma unroll
    for (int it = 0; it < NS; ++it) {
      const TailPair<T>& P = a[it];
      if (P.q < 0) continue;
      const T v0 = val(P, 0), v1 = val(P, 1);
      x[P.q] = P.first ? v0 : v1;
      if (P.two) x[P.q + 1] = P.first ? v1 : v0;
    }
  }
  __device__ __forceinline__ void store(const TailView<T, TL>& v) const {
    put(v.x, [](const TailPair<T>& P, int c) { return P.x[c]; });
    grp_sync<STRIDE>();
  }
};

// The coarsest level's smoothing (see plain_coarsest) from registers.
template <typename T, typename TL, int NS, int STRIDE>
__device__ __forceinline__ int reg_coarsest(const TailView<T, TL>& v, T* xs, int nu_coarse,
                                            double coarse_rtol, int coarse_max, T omega,
                                            double* red) {
  TailRegs<T, TL, NS, STRIDE> r;
  r.template load<false>(v, xs, nullptr, nullptr);
  int n = 0;
  if (!(coarse_rtol > 0.0)) {
    for (; n < nu_coarse; ++n) r.sweep(omega);
  } else {
    const double lim = coarse_rtol * r.norm(red);
    const int group = nu_coarse > 1 ? nu_coarse : 1;
    while (n < coarse_max) {
      const int k = min(group, coarse_max - n);
      for (int s = 0; s < k; ++s) r.sweep(omega);
      n += k;
      if (n < coarse_max && r.norm(red) <= lim) break;
    }
  }
  r.store(v);
  return n;
}

// The coarsest level's smoothing by the first wavefront or the workgroup;
// returns the number of sweeps to every thread.
template <typename T, typename TL>
__device__ __forceinline__ int tail_coarsest(const TailView<T, TL>& v, T* xs, int reg,
                                             int nu_coarse, double coarse_rtol, int coarse_max,
                                             T omega, int* count) {
  __shared__ double red[kTailThreads / kWave];
  const int pairs = ((v.g.nx + 1) >> 1) * v.g.ny * v.g.nz;
  const bool one_wave = pairs <= kRegPairsWave || v.g.n <= kWaveCells;
  if (reg > 0) {
    if (coarse_rtol > 0.0) {
      if (one_wave) {
        if (threadIdx.x < kWave) grp_project<T, TL, kWave>(v, red);
        __syncthreads();
      } else {
        grp_project<T, TL, kTailThreads>(v, red);
      }
    }
    int n = 0;
    if (pairs <= kRegPairsWave) {
      if (threadIdx.x < kWave)
        n = reg_coarsest<T, TL, kRegPairsWave / kWave, kWave>(v, xs, nu_coarse, coarse_rtol,
                                                              coarse_max, omega, red);
    } else if (reg == 1) {
      n = reg_coarsest<T, TL, 1, kTailThreads>(v, xs, nu_coarse, coarse_rtol, coarse_max, omega,
                                               red);
    } else {
      n = reg_coarsest<T, TL, 2, kTailThreads>(v, xs, nu_coarse, coarse_rtol, coarse_max, omega,
                                               red);
    }
    if (threadIdx.x == 0) *count = n;
  } else {
    const int n =
        plain_coarsest<T, TL>(v, nu_coarse, coarse_rtol, coarse_max, omega, red);
    if (threadIdx.x == 0) *count = n;
  }
  __syncthreads();
  return *count;
}

// Pre-smoothing and restriction of a level from registers: the residuals take
// x's place while the coarse cells sum them, in the order of tail_restrict.
template <typename T, typename TL, int NS>
__device__ __forceinline__ void reg_down(const TailView<T, TL>& f, T* xs,
                                         const TailLevel<T, TL>& fl, const TailView<T, TL>& c,
                                         int nsw, T omega) {
  TailRegs<T, TL, NS, kTailThreads> r;
  r.template load<false>(f, xs, nullptr, nullptr);
  for (int s = 0; s < nsw; ++s) r.sweep(omega);
  T res[NS][2];
#pragma unroll
  for (int it = 0; it < NS; ++it)
#pragma unroll
    for (int col = 0; col < 2; ++col)
      res[it][col] = r.a[it].on[col] ? r.a[it].sg[col] - r.flux(r.a[it], col) : T(0);
  __syncthreads();
  r.put(f.x, [&](const TailPair<T>& P, int col) { return res[&P - r.a][col]; });
  __syncthreads();
  const Geom& gc = c.g;
  const int sy = f.g.nx, sz = f.g.nx * f.g.ny;
  const float rnx = 1.0f / (float)gc.nx, rny = 1.0f / (float)gc.ny;
  for (int q = threadIdx.x; q < (int)gc.n; q += kTailThreads) {
    const int row = tail_div(q, gc.nx, rnx);
    const int I = q - row * gc.nx;
    const int K = tail_div(row, gc.ny, rny);
    const int J = row - K * gc.ny;
    auto column = [&](int i, int j) {
      T acc = T(0);
      for (int dz = 0; dz < fl.cz; ++dz) acc += f.x[(K * fl.cz + dz) * sz + j * sy + i];
      return acc;
    };
    T rr[2];
    for (int dy = 0; dy < fl.cy; ++dy) {
      const int j = J * fl.cy + dy;
      T acc = column(I * fl.cx, j);
      if (fl.cx == 2) acc += column(I * fl.cx + 1, j);
      rr[dy] = acc;
    }
    c.s[q] = (fl.cy == 2) ? rr[0] + rr[1] : rr[0];
    c.x[q] = T(0);
  }
  __syncthreads();
  r.store(f);
}

// Correction and post-smoothing of a level from registers.
template <typename T, typename TL, int NS>
__device__ __forceinline__ void reg_up(const TailView<T, TL>& f, T* xs, const TailLevel<T, TL>& fl,
                                       const TailView<T, TL>& c, int nsw, T omega) {
  TailRegs<T, TL, NS, kTailThreads> r;
  r.template load<true>(f, xs, &fl, &c);
  for (int s = 0; s < nsw; ++s) r.sweep(omega);
  r.store(f);
}

// Copy n elements between global memory and LDS in 16-byte pieces, several
// in flight per thread (both ends 16-byte aligned), then the remaining bytes.
template <typename T>
__device__ __forceinline__ void tail_copy(T* dst, const T* src, int n) {
  const int nb = n * (int)sizeof(T);
  const int n16 = nb >> 4;
  uint4* d16 = reinterpret_cast<uint4*>(dst);
  const uint4* s16 = reinterpret_cast<const uint4*>(src);
  int q = threadIdx.x;
  for (; q + 3 * kTailThreads < n16; q += 4 * kTailThreads) {
    const uint4 a = s16[q], b = s16[q + kTailThreads], c = s16[q + 2 * kTailThreads],
                d = s16[q + 3 * kTailThreads];
    d16[q] = a;
    d16[q + kTailThreads] = b;
    d16[q + 2 * kTailThreads] = c;
    d16[q + 3 * kTailThreads] = d;
  }
  for (; q < n16; q += kTailThreads) d16[q] = s16[q];
  uint8_t* d1 = reinterpret_cast<uint8_t*>(dst);
  const uint8_t* s1 = reinterpret_cast<const uint8_t*>(src);
  for (int b = (n16 << 4) + (int)threadIdx.x; b < nb; b += kTailThreads) d1[b] = s1[b];
}

// The whole tail of one problem (see the top of this file).  GLOBAL: the
// tail is one level (the coarsest), used in place in global memory.
template <typename T, typename TL, bool GLOBAL>
__device__ __forceinline__ void tail_run(const TailArgs<T, TL>& a, char* tail_lds) {
  __shared__ int count;
  const T omega = (T)(*a.omega);
  const int last = a.nl - 1;
  // stage the levels in LDS (x and sigma of the first level come from the
  // restriction that precedes this launch; deeper levels are produced here)
  if constexpr (!GLOBAL) {
    for (int l = 0; l < a.nl; ++l) {
      const TailLevel<T, TL>& v = a.lv[l];
      const TailView<T, TL> w = tail_view<T, TL, false>(tail_lds, v);
      const int n = (int)v.g.n;
      tail_copy<TL>(w.L, v.L, 3 * n);
      tail_copy<uint8_t>(w.a, v.active, n);
      if (l == 0) {
        tail_copy<T>(w.x, v.x, n);
        tail_copy<T>(w.s, v.sigma, n);
      }
    }
    __syncthreads();
  }
  for (int l = 0; l < last; ++l) {
    const TailView<T, TL> f = tail_view<T, TL, GLOBAL>(tail_lds, a.lv[l]);
    const TailView<T, TL> c = tail_view<T, TL, GLOBAL>(tail_lds, a.lv[l + 1]);
    T* const xs = (T*)(tail_lds + a.lv[l].ox);
    if (a.lv[l].reg == 1) {
      reg_down<T, TL, 1>(f, xs, a.lv[l], c, a.nu_pre, omega);
    } else if (a.lv[l].reg == 2) {
      reg_down<T, TL, 2>(f, xs, a.lv[l], c, a.nu_pre, omega);
    } else {
      tail_sweeps<T, TL>(f, a.nu_pre, omega);
      tail_restrict<T, TL>(f, a.lv[l], c);
    }
  }
  const int nc = tail_coarsest<T, TL>(tail_view<T, TL, GLOBAL>(tail_lds, a.lv[last]),
                                      (T*)(tail_lds + a.lv[last].ox), a.lv[last].reg, a.nu_coarse,
                                      a.coarse_rtol, a.coarse_max, omega, &count);
  if (a.sweeps && threadIdx.x == 0) *a.sweeps = nc;
  for (int l = last - 1; l >= 0; --l) {
    const TailView<T, TL> f = tail_view<T, TL, GLOBAL>(tail_lds, a.lv[l]);
    const TailView<T, TL> c = tail_view<T, TL, GLOBAL>(tail_lds, a.lv[l + 1]);
    T* const xs = (T*)(tail_lds + a.lv[l].ox);
    if (a.lv[l].reg == 1) {
      reg_up<T, TL, 1>(f, xs, a.lv[l], c, a.nu_post, omega);
    } else if (a.lv[l].reg == 2) {
      reg_up<T, TL, 2>(f, xs, a.lv[l], c, a.nu_post, omega);
    } else {
      tail_prolong<T, TL>(f, a.lv[l], c);
      tail_sweeps<T, TL>(f, a.nu_post, omega);
    }
  }
  if constexpr (!GLOBAL) {
    for (int l = 0; l < a.nl; ++l) {
      const TailLevel<T, TL>& v = a.lv[l];
      const TailView<T, TL> w = tail_view<T, TL, false>(tail_lds, v);
      tail_copy<T>(v.x, w.x, (int)v.g.n);
      tail_copy<T>(v.sigma, w.s, (int)v.g.n);
    }
  }
}

template <typename T, typename TL, bool GLOBAL>
__global__ __launch_bounds__(kTailThreads) void k_tail(TailArgs<T, TL> a) {
  if (a.done != nullptr && *a.done) return;
  extern __shared__ __align__(16) char tail_lds[];
  tail_run<T, TL, GLOBAL>(a, tail_lds);
}

// One workgroup per problem of a batch, each with its own tail.
template <typename T, typename TL, bool GLOBAL>
__global__ __launch_bounds__(kTailThreads) void k_tail_batch(
    const TailArgs<T, TL>* __restrict__ args) {
  const TailArgs<T, TL>& a = args[blockIdx.x];
  if (a.done != nullptr && *a.done) return;
  extern __shared__ __align__(16) char tail_lds[];
  tail_run<T, TL, GLOBAL>(a, tail_lds);
}

}  // namespace gmg
