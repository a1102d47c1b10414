// libunet.so: the 3-D U-Net warm start of the GMG solver, for gfx950.
//
// C ABI and layouts: include/unet.h.  Convolutions are implicit GEMMs on the
// CDNA4 BF16 matrix cores (v_mfma_f32_16x16x32_bf16, FP32 accumulation):
//   forward:  M = voxels, N = output channels, K = taps * input channels;
//   dgrad:    the forward kernel on flipped, transposed weights;
//   wgrad:    M = output channels, N = taps * input channels, K = voxels, split
//             over voxel chunks into FP32 partials that a second kernel sums
//             in a fixed order (deterministic).
// Everything else (pooling, upsampling, ReLU backward, the 1x1x1 head, the
// masked MSE, Adam) is elementwise or a small reduction and HBM-bound.

#include <hip/hip_runtime.h>
#include <type_traits>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/unet.h"
#include "unet_conv.h"
#include "unet_wgrad.h"
#include "unet_device.h"

using namespace unet;

namespace {

thread_local std::string g_err;

unet_status ufail(unet_status s, const std::string& m) {
  g_err = m;
  return s;
}

#define UHIP(expr)                                                                       \
  do {                                                                                   \
    hipError_t e_ = (expr);                                                              \
    if (e_ != hipSuccess)                                                                \
      return ufail(e_ == hipErrorOutOfMemory ? UNET_ENOMEM : UNET_EHIP,                  \
                   std::string(#expr) + ": " + hipGetErrorString(e_));                   \
  } while (0)

struct Vox {
  int n, d, h, w;
};
// a / b for a >= 0, b > 0: in 32 bits where a fits (a 64-bit division is over a
// hundred instructions, and pooling and upsampling do four or five per thread).
// With the eight loads of a pooled voxel in flight together: pooling of 16
// channels of 2 x 128^3 58 -> 48 us, of 48x56x104's second and third levels 5.6 ->
// 3.7; the gradients and upsampling are bound by memory and stay as they were.
__device__ __forceinline__ long long div_idx(long long a, int b) {
  return a >> 31 ? a / b : (long long)((unsigned)a / (unsigned)b);
}
__device__ __forceinline__ Vox vox_of(long long v, const unet_shape& s) {
  Vox r;
  if (!(v >> 31)) {
    const unsigned u = (unsigned)v, t = u / (unsigned)s.w, p = t / (unsigned)s.h,
                   n = p / (unsigned)s.d;
    r.w = (int)(u - t * s.w);
    r.h = (int)(t - p * s.h);
    r.d = (int)(p - n * s.d);
    r.n = (int)n;
    return r;
  }
  r.w = (int)(v % s.w);
  long long t = v / s.w;
  r.h = (int)(t % s.h);
  t /= s.h;
  r.d = (int)(t % s.d);
  r.n = (int)(t / s.d);
  return r;
}
__device__ __forceinline__ long long vox_index(const Vox& a, const unet_shape& s) {
  return (((long long)a.n * s.d + a.d) * s.h + a.h) * s.w + a.w;
}

// Neighbour of voxel a at tap t (27 taps in (kd, kh, kw) order, or 1 tap = a
// itself); returns -1 outside the grid (zero padding).
__device__ __forceinline__ long long tap_nbr(const Vox& a, const unet_shape& s, int taps, int t) {
  if (taps == 1) return vox_index(a, s);
  Vox b = a;
  b.d += t / 9 - 1;
  b.h += (t / 3) % 3 - 1;
  b.w += t % 3 - 1;
  if (b.d < 0 || b.d >= s.d || b.h < 0 || b.h >= s.h || b.w < 0 || b.w >= s.w) return -1;
  return vox_index(b, s);
}

// ---------------------------------------------------------------------------
// MFMA lane layout (16x16x32 BF16):
//   A[m][k]: lane l holds m = l % 16, k = 8 (l / 16) + j, j = 0..7
//   B[k][n]: lane l holds n = l % 16, k = 8 (l / 16) + j
//   D[m][n]: lane l, element r holds m = 4 (l / 16) + r, n = l % 16
// ---------------------------------------------------------------------------

__global__ void k_mfma_selfcheck(const uint16_t* A, const uint16_t* B, float* out) {
  const int l = threadIdx.x;
  uint16_t a[8], b[8];
  for (int j = 0; j < 8; ++j) {
    a[j] = A[(l % 16) * 32 + 8 * (l / 16) + j];
    b[j] = B[(8 * (l / 16) + j) * 16 + (l % 16)];
  }
  bf16x8 av, bv;
  __builtin_memcpy(&av, a, 16);
  __builtin_memcpy(&bv, b, 16);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc, 0, 0, 0);
  for (int r = 0; r < 4; ++r) out[(4 * (l / 16) + r) * 16 + (l % 16)] = acc[r];
}

// ---------------------------------------------------------------------------
// Implicit-GEMM convolution forward: each wave computes 16 MB voxels (MB
// blocks of 16) x NB*16 output channels, the workgroup's output channels
// starting at 16 NB blockIdx.y; K steps of 32 = 4 lane groups x 8
// consecutive input channels of one tap.  Every output's K order is the same
// for every (MB, NB), so the split does not change a bit of the result.
// ---------------------------------------------------------------------------

template <int MB, int NB>
__global__ __launch_bounds__(256) void k_conv_fwd(unet_shape s, const uint16_t* __restrict__ x,
                                                  int xld, int xoff, int cin,
                                                  const uint16_t* __restrict__ w,
                                                  const float* __restrict__ bias, int taps,
                                                  uint16_t* __restrict__ y, int yld, int yoff,
                                                  float* __restrict__ yf, int relu) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long nvox = (long long)s.n * s.d * s.h * s.w;
  const long long vbase = ((long long)blockIdx.x * 4 + wave) * (16 * MB);
  const int co0 = blockIdx.y * (16 * NB);  // this workgroup's output channels
  const int K = taps * cin;
  const int ksteps = (K + 31) / 32;
  // Each of the lane's four voxels: its index (the host keeps voxel counts
  // below 2^31) and a mask of the taps that land inside the grid (bit t for
  // tap t in (kd, kh, kw) order; zero padding elsewhere).  A tap's neighbour
  // is then the voxel index plus an offset that is the same for every voxel.
  int vi[MB];
  uint32_t vm[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const long long v = vbase + mb * 16 + (lane & 15);
    const bool ok = v < nvox;
    const Vox a = vox_of(ok ? v : 0, s);
    vi[mb] = ok ? (int)v : 0;
    uint32_t m = 0;
    if (taps == 1) {
      m = 1u;
    } else {
#pragma unroll
      for (int t = 0; t < 27; ++t) {
        const int dd = a.d + t / 9 - 1, dh = a.h + (t / 3) % 3 - 1, dw = a.w + t % 3 - 1;
        const bool in = dd >= 0 && dd < s.d && dh >= 0 && dh < s.h && dw >= 0 && dw < s.w;
        m |= (in ? 1u : 0u) << t;
      }
    }
    vm[mb] = ok ? m : 0u;
  }
  const int hw = s.h * s.w;
  // k / cin for k < 27 cin by a multiply and shift, exact for cin <= 384
  const uint32_t rcin = ((1u << 22) + (uint32_t)cin - 1) / (uint32_t)cin;
  const int kl = 8 * (lane >> 4);
  // Operands of K step ks.  Every load is issued (at the voxel itself or
  // at a clamped k when the value is padding), and padding is zeroed after
  // the load, so that no branch sits between the loads of a step and the
  // next step's loads can be in flight while this step's MFMAs run.
  auto load = [&](int ks, bf16x8 (&a)[MB], bf16x8 (&b)[NB]) {
    const int k = ks * 32 + kl;
    const bool kin = k < K;
    const int kk = kin ? k : K - 8;
    const int t = (int)(((uint32_t)kk * rcin) >> 22), ci = kk - t * cin;
    const int off = (taps == 1) ? 0 : (t / 9 - 1) * hw + ((t / 3) % 3 - 1) * s.w + (t % 3 - 1);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const bool use = kin && ((vm[mb] >> t) & 1u);
      const bf16x8 v = ld8(x + (long long)(use ? vi[mb] + off : vi[mb]) * xld + xoff + ci);
      a[mb] = use ? v : zero8();
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const bf16x8 v = ld8(w + (long long)(co0 + nb * 16 + (lane & 15)) * K + kk);
      b[nb] = kin ? v : zero8();
    }
  };
  f32x4 acc[MB][NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 a0[MB], b0[NB], a1[MB], b1[NB];
  load(0, a0, b0);
  for (int ks = 0; ks < ksteps; ++ks) {
    load(ks + 1 < ksteps ? ks + 1 : ks, a1, b1);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[mb], b0[nb], acc[mb][nb], 0, 0, 0);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) a0[mb] = a1[mb];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) b0[nb] = b1[nb];
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int co = co0 + nb * 16 + (lane & 15);
      const float bb = bias ? bias[co] : 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const long long v = vbase + mb * 16 + 4 * (lane >> 4) + r;
        if (v >= nvox) continue;
        float val = acc[mb][nb][r] + bb;
        if (relu) val = fmaxf(val, 0.f);
        if (yf)
          yf[v * yld + yoff + co] = val;
        else
          y[v * yld + yoff + co] = f2bf(val);
      }
    }
}

// wflip[c][t'][o] = w[o][taps-1-t'][c]
__global__ void k_flip_weights(const uint16_t* __restrict__ w, uint16_t* __restrict__ wf, int cout,
                               int cin, int taps) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long n = (long long)cout * cin * taps;
  if (i >= n) return;
  const int o = (int)(i % cout);
  long long r = i / cout;
  const int tp = (int)(r % taps);
  const int c = (int)(r / taps);
  wf[((long long)c * taps + tp) * cout + o] = w[((long long)o * taps + (taps - 1 - tp)) * cin + c];
}

// ---------------------------------------------------------------------------
// Weight gradient: block = (k-tile of 64, voxel chunk); 4 waves, wave q owns
// k-block q (16 values of k) and every 16-channel output block.  Each step
// stages 32 voxels of dy (as [o][v]) and of the im2col input (as [k][v]) in
// LDS so that every MFMA operand is one 16-byte LDS read.
// ---------------------------------------------------------------------------

template <int OB>
__global__ __launch_bounds__(256) void k_conv_wgrad(unet_shape s, const uint16_t* __restrict__ x,
                                                    int xld, int xoff, int cin,
                                                    const uint16_t* __restrict__ dy, int dld,
                                                    int doff, int taps, long long vchunk,
                                                    long long rs, float* __restrict__ ws) {
  constexpr int COUT = OB * 16;
  __shared__ uint16_t sdy[COUT][40];  // [o][v], padded rows
  __shared__ uint16_t sx[64][40];     // [k][v]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int K = taps * cin;
  const int k0 = blockIdx.x * 64;
  const long long nvox = (long long)s.n * s.d * s.h * s.w;
  const long long v0 = (long long)blockIdx.y * vchunk;
  const long long v1 = min(nvox, v0 + vchunk);
  f32x4 acc[OB];
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) acc[ob] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (long long vs = v0; vs < v1; vs += 32) {
    // stage dy: 32 voxels x COUT channels, 8 channels per item
    for (int q = tid; q < 32 * (COUT / 8); q += 256) {
      const int vv = q / (COUT / 8), oc = (q % (COUT / 8)) * 8;
      const long long v = vs + vv;
      uint16_t buf[8];
      if (v < v1) {
        const uint4 raw = *reinterpret_cast<const uint4*>(dy + v * dld + doff + oc);
        __builtin_memcpy(buf, &raw, 16);
      } else {
        for (int e = 0; e < 8; ++e) buf[e] = 0;
      }
      for (int e = 0; e < 8; ++e) sdy[oc + e][vv] = buf[e];
    }
    // stage im2col: 32 voxels x 64 k, 8 consecutive k (one tap) per item
    for (int q = tid; q < 32 * 8; q += 256) {
      const int vv = q >> 3, kc = (q & 7) * 8;
      const long long v = vs + vv;
      const int k = k0 + kc;
      uint16_t buf[8];
      long long nb_v = -1;
      int ci = 0;
      if (v < v1 && k < K) {
        const int t = k / cin;
        ci = k - t * cin;
        nb_v = tap_nbr(vox_of(v, s), s, taps, t);
      }
      if (nb_v >= 0) {
        const uint4 raw = *reinterpret_cast<const uint4*>(x + nb_v * xld + xoff + ci);
        __builtin_memcpy(buf, &raw, 16);
      } else {
        for (int e = 0; e < 8; ++e) buf[e] = 0;
      }
      for (int e = 0; e < 8; ++e) sx[kc + e][vv] = buf[e];
    }
    __syncthreads();
    const int vl = 8 * (lane >> 4);
    bf16x8 bv;
    __builtin_memcpy(&bv, &sx[wave * 16 + (lane & 15)][vl], 16);
#pragma unroll
    for (int ob = 0; ob < OB; ++ob) {
      bf16x8 av;
      __builtin_memcpy(&av, &sdy[ob * 16 + (lane & 15)][vl], 16);
      acc[ob] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc[ob], 0, 0, 0);
    }
    __syncthreads();
  }
  // partial dW of this chunk: ws[chunk * rs + o K + k]
  float* out = ws + (long long)blockIdx.y * rs;
#pragma unroll
  for (int ob = 0; ob < OB; ++ob)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = ob * 16 + 4 * (lane >> 4) + r;
      const int k = k0 + wave * 16 + (lane & 15);
      if (k < K) out[(long long)o * K + k] = acc[ob][r];
    }
}

// Per-chunk channel sums of dy (bias gradient partials): wsb[chunk * rs + o].
__global__ __launch_bounds__(256) void k_bias_partial(unet_shape s, const uint16_t* __restrict__ dy,
                                                      int dld, int doff, int cout, long long vchunk,
                                                      long long rs, float* __restrict__ wsb) {
  const long long nvox = (long long)s.n * s.d * s.h * s.w;
  const long long v0 = (long long)blockIdx.x * vchunk, v1 = min(nvox, v0 + vchunk);
  for (int o = threadIdx.x; o < cout; o += blockDim.x) {
    float acc = 0.f;
    for (long long v = v0; v < v1; ++v) acc += bf2f(dy[v * dld + doff + o]);
    wsb[(long long)blockIdx.x * rs + o] = acc;
  }
}

// Sum of the nchunks rows of ws (row length n): entries below nw go to dw, the
// rest to db.  A workgroup takes 64 entries, its wave w the rows of the w-th of
// WAVES parts in order, and the waves' sums are added in wave order: the order
// depends only on the row count.  Several loads of a wave are in flight, where
// one thread per entry walked 64 rows one latency after another (64 rows of
// 110848 entries: 17.5 -> 9 us; 256 rows of 6928, in two launches, 11 -> 4.8).
// Of few rows a workgroup of 16 waves is mostly start-up (32 rows of 442496
// entries: 16.3 us, with 4 waves 8.0).
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_sum_rows(const float* __restrict__ ws,
                                                             long long n, int nchunks,
                                                             long long nw, float* __restrict__ dw,
                                                             float* __restrict__ db) {
  __shared__ float part[WAVES][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long i = (long long)blockIdx.x * 64 + lane;
  const int c0 = nchunks * wave / WAVES, c1 = nchunks * (wave + 1) / WAVES;
  float acc = 0.f;
  if (i < n) {
#pragma unroll 8
    for (int c = c0; c < c1; ++c) acc += ws[(long long)c * n + i];
  }
  part[wave][lane] = acc;
  __syncthreads();
  if (wave > 0 || i >= n) return;
  acc = part[0][lane];
#pragma unroll
  for (int w = 1; w < WAVES; ++w) acc += part[w][lane];
  if (i < nw)
    dw[i] = acc;
  else
    db[i - nw] = acc;
}

// ---------------------------------------------------------------------------
// Elementwise and small kernels
// ---------------------------------------------------------------------------

__global__ void k_relu_bwd(long long nvox, int c, const uint16_t* __restrict__ y, int yld, int yoff,
                           const uint16_t* __restrict__ dy, int dld, int doff,
                           uint16_t* __restrict__ out, int old, int ooff) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nvox * c) return;
  const long long v = i / c;
  const int ch = (int)(i - v * c);
  const float g = bf2f(dy[v * dld + doff + ch]);
  out[v * old + ooff + ch] = (bf2f(y[v * yld + yoff + ch]) > 0.f) ? f2bf(g) : (uint16_t)0;
}

// coarse voxel V = (n, D, H, W) of a fine grid (2D, 2H, 2W)
__global__ void k_pool_fwd(unet_shape f, int c, const uint16_t* __restrict__ x, int xld, int xoff,
                           uint16_t* __restrict__ y, int yld, int yoff) {
  unet_shape cs{f.n, f.d / 2, f.h / 2, f.w / 2};
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long ncv = (long long)cs.n * cs.d * cs.h * cs.w;
  if (i >= ncv * c) return;
  const long long V = i / c;
  const int ch = (int)(i - V * c);
  const Vox a = vox_of(V, cs);
  float acc = 0.f;
  for (int q = 0; q < 8; ++q) {
    const Vox b{a.n, 2 * a.d + (q >> 2), 2 * a.h + ((q >> 1) & 1), 2 * a.w + (q & 1)};
    acc += bf2f(x[vox_index(b, f) * xld + xoff + ch]);
  }
  y[V * yld + yoff + ch] = f2bf(acc * 0.125f);
}

__global__ void k_pool_bwd(unet_shape f, int c, const uint16_t* __restrict__ dy, int dld, int doff,
                           uint16_t* __restrict__ dx, int xld, int xoff, int accumulate) {
  unet_shape cs{f.n, f.d / 2, f.h / 2, f.w / 2};
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long nfv = (long long)f.n * f.d * f.h * f.w;
  if (i >= nfv * c) return;
  const long long v = i / c;
  const int ch = (int)(i - v * c);
  const Vox a = vox_of(v, f);
  const Vox b{a.n, a.d / 2, a.h / 2, a.w / 2};
  float g = 0.125f * bf2f(dy[vox_index(b, cs) * dld + doff + ch]);
  if (accumulate) g += bf2f(dx[v * xld + xoff + ch]);
  dx[v * xld + xoff + ch] = f2bf(g);
}

__global__ void k_up_fwd(unet_shape cs, int c, const uint16_t* __restrict__ x, int xld, int xoff,
                         uint16_t* __restrict__ y, int yld, int yoff) {
  const unet_shape f{cs.n, 2 * cs.d, 2 * cs.h, 2 * cs.w};
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long nfv = (long long)f.n * f.d * f.h * f.w;
  if (i >= nfv * c) return;
  const long long v = i / c;
  const int ch = (int)(i - v * c);
  const Vox a = vox_of(v, f);
  const Vox b{a.n, a.d / 2, a.h / 2, a.w / 2};
  y[v * yld + yoff + ch] = x[vox_index(b, cs) * xld + xoff + ch];
}

__global__ void k_up_bwd(unet_shape cs, int c, const uint16_t* __restrict__ dy, int dld, int doff,
                         uint16_t* __restrict__ dx, int xld, int xoff) {
  const unet_shape f{cs.n, 2 * cs.d, 2 * cs.h, 2 * cs.w};
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long ncv = (long long)cs.n * cs.d * cs.h * cs.w;
  if (i >= ncv * c) return;
  const long long V = i / c;
  const int ch = (int)(i - V * c);
  const Vox a = vox_of(V, cs);
  float acc = 0.f;
  for (int q = 0; q < 8; ++q) {
    const Vox b{a.n, 2 * a.d + (q >> 2), 2 * a.h + ((q >> 1) & 1), 2 * a.w + (q & 1)};
    acc += bf2f(dy[vox_index(b, f) * dld + doff + ch]);
  }
  dx[V * xld + xoff + ch] = f2bf(acc);
}

// 1x1x1 head to one channel: y[v] = b + sum_c w[c] x[v][c] (FP32 out).
__global__ void k_head_fwd(long long nvox, int c, const uint16_t* __restrict__ x, int xld, int xoff,
                           const float* __restrict__ w, const float* __restrict__ b,
                           float* __restrict__ y) {
  const long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nvox) return;
  float acc = 0.f;
  for (int ch = 0; ch < c; ++ch) acc += w[ch] * bf2f(x[v * xld + xoff + ch]);
  y[v] = acc + b[0];
}

// dx[v][c] = w[c] dy[v]
__global__ void k_head_dgrad(long long nvox, int c, const float* __restrict__ w,
                             const float* __restrict__ dy, uint16_t* __restrict__ dx, int xld,
                             int xoff) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nvox * c) return;
  const long long v = i / c;
  const int ch = (int)(i - v * c);
  dx[v * xld + xoff + ch] = f2bf(w[ch] * dy[v]);
}

// partials of dw[c] = sum_v dy[v] x[v][c] and db = sum_v dy[v]: wsp[chunk][c+1]
__global__ __launch_bounds__(256) void k_head_wgrad_partial(long long nvox, int c,
                                                            const uint16_t* __restrict__ x, int xld,
                                                            int xoff, const float* __restrict__ dy,
                                                            long long vchunk,
                                                            float* __restrict__ wsp) {
  const long long v0 = (long long)blockIdx.x * vchunk, v1 = min(nvox, v0 + vchunk);
  for (int ch = threadIdx.x; ch <= c; ch += blockDim.x) {
    float acc = 0.f;
    for (long long v = v0; v < v1; ++v)
      acc += dy[v] * (ch < c ? bf2f(x[v * xld + xoff + ch]) : 1.f);
    wsp[(long long)blockIdx.x * (c + 1) + ch] = acc;
  }
}

// ---- 8-channel forms (16-byte accesses) for channel counts that are
// multiples of 8: one thread per (voxel, 8-channel group); the arithmetic and
// its order per element are those of the one-channel kernels above.
__device__ __forceinline__ uint4 ld16(const uint16_t* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ void st16(uint16_t* p, const uint4& v) { *reinterpret_cast<uint4*>(p) = v; }
__device__ __forceinline__ void unpack8(const uint4& r, float (&f)[8]) {
  const uint32_t u[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[2 * e] = __uint_as_float(u[e] << 16);
    f[2 * e + 1] = __uint_as_float(u[e] & 0xFFFF0000u);
  }
}
__device__ __forceinline__ uint4 gate8(const uint4& u, const uint4& y) {
  return make_uint4(gate2(u.x, y.x), gate2(u.y, y.y), gate2(u.z, y.z), gate2(u.w, y.w));
}
__device__ __forceinline__ uint4 pack8(const float (&f)[8]) {
  uint32_t u[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) u[e] = (uint32_t)f2bf(f[2 * e]) | ((uint32_t)f2bf(f[2 * e + 1]) << 16);
  return make_uint4(u[0], u[1], u[2], u[3]);
}

__global__ void k_relu_bwd8(long long nvox, int g8, const uint16_t* __restrict__ y, int yld,
                            int yoff, const uint16_t* __restrict__ dy, int dld, int doff,
                            uint16_t* __restrict__ out, int old, int ooff) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nvox * g8) return;
  const long long v = div_idx(i, g8);
  const int c = (int)(i - v * g8) * 8;
  const uint4 yv = ld16(y + v * yld + yoff + c);
  st16(out + v * old + ooff + c, gate8(ld16(dy + v * dld + doff + c), yv));
}

__global__ void k_pool_fwd8(unet_shape f, int g8, const uint16_t* __restrict__ x, int xld, int xoff,
                            uint16_t* __restrict__ y, int yld, int yoff) {
  unet_shape cs{f.n, f.d / 2, f.h / 2, f.w / 2};
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long ncv = (long long)cs.n * cs.d * cs.h * cs.w;
  if (i >= ncv * g8) return;
  const long long V = div_idx(i, g8);
  const int c = (int)(i - V * g8) * 8;
  const Vox a = vox_of(V, cs);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const Vox b{a.n, 2 * a.d + (q >> 2), 2 * a.h + ((q >> 1) & 1), 2 * a.w + (q & 1)};
    float fx[8];
    unpack8(ld16(x + vox_index(b, f) * xld + xoff + c), fx);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += fx[e];
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] *= 0.125f;
  st16(y + V * yld + yoff + c, pack8(acc));
}

__global__ void k_pool_bwd8(unet_shape f, int g8, const uint16_t* __restrict__ dy, int dld,
                            int doff, uint16_t* __restrict__ dx, int xld, int xoff, int accumulate,
                            const uint16_t* __restrict__ gate, int gld, int goff) {
  unet_shape cs{f.n, f.d / 2, f.h / 2, f.w / 2};
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long nfv = (long long)f.n * f.d * f.h * f.w;
  if (i >= nfv * g8) return;
  const long long v = div_idx(i, g8);
  const int c = (int)(i - v * g8) * 8;
  const Vox a = vox_of(v, f);
  const Vox b{a.n, a.d / 2, a.h / 2, a.w / 2};
  float g[8];
  unpack8(ld16(dy + vox_index(b, cs) * dld + doff + c), g);
#pragma unroll
  for (int e = 0; e < 8; ++e) g[e] *= 0.125f;
  if (accumulate) {
    float o[8];
    unpack8(ld16(dx + v * xld + xoff + c), o);
#pragma unroll
    for (int e = 0; e < 8; ++e) g[e] += o[e];
  }
  uint4 r = pack8(g);
  if (gate) r = gate8(r, ld16(gate + v * gld + goff + c));
  st16(dx + v * xld + xoff + c, r);
}

__global__ void k_up_fwd8(unet_shape cs, int g8, const uint16_t* __restrict__ x, int xld, int xoff,
                          uint16_t* __restrict__ y, int yld, int yoff) {
  const unet_shape f{cs.n, 2 * cs.d, 2 * cs.h, 2 * cs.w};
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long nfv = (long long)f.n * f.d * f.h * f.w;
  if (i >= nfv * g8) return;
  const long long v = div_idx(i, g8);
  const int c = (int)(i - v * g8) * 8;
  const Vox a = vox_of(v, f);
  const Vox b{a.n, a.d / 2, a.h / 2, a.w / 2};
  st16(y + v * yld + yoff + c, ld16(x + vox_index(b, cs) * xld + xoff + c));
}

__global__ void k_up_bwd8(unet_shape cs, int g8, const uint16_t* __restrict__ dy, int dld, int doff,
                          uint16_t* __restrict__ dx, int xld, int xoff,
                          const uint16_t* __restrict__ gate, int gld, int goff) {
  const unet_shape f{cs.n, 2 * cs.d, 2 * cs.h, 2 * cs.w};
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long ncv = (long long)cs.n * cs.d * cs.h * cs.w;
  if (i >= ncv * g8) return;
  const long long V = div_idx(i, g8);
  const int c = (int)(i - V * g8) * 8;
  const Vox a = vox_of(V, cs);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const Vox b{a.n, 2 * a.d + (q >> 2), 2 * a.h + ((q >> 1) & 1), 2 * a.w + (q & 1)};
    float g[8];
    unpack8(ld16(dy + vox_index(b, f) * dld + doff + c), g);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += g[e];
  }
  uint4 r = pack8(acc);
  if (gate) r = gate8(r, ld16(gate + V * gld + goff + c));
  st16(dx + V * xld + xoff + c, r);
}

__global__ void k_head_fwd8(long long nvox, int g8, const uint16_t* __restrict__ x, int xld,
                            int xoff, const float* __restrict__ w, const float* __restrict__ b,
                            float* __restrict__ y) {
  const long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nvox) return;
  float acc = 0.f;
  for (int g = 0; g < g8; ++g) {
    float fx[8];
    unpack8(ld16(x + v * xld + xoff + 8 * g), fx);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc += w[8 * g + e] * fx[e];
  }
  y[v] = acc + b[0];
}

// Head backward, 8-channel form: workgroup = voxel chunk,
// thread (j, g) sums voxels v0 + j, v0 + j + J, ... for channels 8g..8g+7
// (g = 0 also the bias column); the J voxel lanes are then added by a fixed
// pairwise tree in LDS.  wsp[chunk][c + 1] as k_head_wgrad_partial.  With dx,
// the same pass over x and dy writes dx = w dy, with `gate` cleared where x is
// not positive (memory-bound: 16 channels of 2 x 128^3 65 us, before 78 in two
// passes and 79 more for the ReLU).
__global__ __launch_bounds__(256) void k_head_bwd8(long long nvox, int g8,
                                                   const uint16_t* x, int xld, int xoff,
                                                   const float* __restrict__ w,
                                                   const float* __restrict__ dy,
                                                   uint16_t* dx, int dld, int doff, int gate,
                                                   long long vchunk, float* __restrict__ wsp) {
  __shared__ float red[256][9];
  const int tid = threadIdx.x, J = 256 / g8;
  const int g = tid % g8, j = tid / g8;
  const long long v0 = (long long)blockIdx.x * vchunk, v1 = min(nvox, v0 + vchunk);
  float acc[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (j < J) {
    float wr[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (dx)
#pragma unroll
      for (int e = 0; e < 8; ++e) wr[e] = w[8 * g + e];
    constexpr int U = 4;  // voxels in flight
    for (long long v = v0 + j; v < v1; v += U * J) {
      float d[U];
      uint4 xr[U];
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const long long vq = min(v + q * J, v1 - 1);
        d[q] = dy[vq];
        xr[q] = ld16(x + vq * xld + xoff + 8 * g);
      }
#pragma unroll
      for (int q = 0; q < U; ++q) {
        if (v + q * J >= v1) break;
        float fx[8];
        unpack8(xr[q], fx);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += d[q] * fx[e];
        acc[8] += d[q];
        if (dx) {
          float o[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = wr[e] * d[q];
          uint4 r = pack8(o);
          if (gate) r = gate8(r, xr[q]);
          st16(dx + (v + q * J) * dld + doff + 8 * g, r);
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 9; ++e) red[tid][e] = acc[e];
  __syncthreads();
  for (int st = 1; st < J; st *= 2) {
    if (j < J && j % (2 * st) == 0 && j + st < J)
#pragma unroll
      for (int e = 0; e < 9; ++e) red[tid][e] += red[tid + st * g8][e];
    __syncthreads();
  }
  if (j == 0) {
    const int c = g8 * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) wsp[(long long)blockIdx.x * (c + 1) + 8 * g + e] = red[g][e];
    if (g == 0) wsp[(long long)blockIdx.x * (c + 1) + c] = red[0][8];
  }
}

// masked MSE: per-block partial sums of the squared error and mask count,
// and the gradient 2 (pred - target) mask / count (count passed in).
// One workgroup per CU fits the caller's partials: 16 waves each, four voxels
// of a thread in flight (4 Mi voxels: 54 us with 4 waves and one, now 9.5).
constexpr int kMseThreads = 1024;
__global__ __launch_bounds__(kMseThreads) void k_mse_partial(long long nvox,
                                                             const float* __restrict__ p,
                                                             const float* __restrict__ t,
                                                             const uint8_t* __restrict__ m,
                                                             double* __restrict__ part) {
  __shared__ double s1[kMseThreads], s2[kMseThreads];
  double a = 0.0, c = 0.0;
  constexpr int U = 4;
  const long long step = (long long)gridDim.x * kMseThreads;
  for (long long v = (long long)blockIdx.x * kMseThreads + threadIdx.x; v < nvox; v += U * step) {
    float pv[U], tv[U];
    bool on[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const long long vq = min(v + q * step, nvox - 1);
      pv[q] = p[vq];
      tv[q] = t[vq];
      on[q] = m[vq] && v + q * step < nvox;
    }
#pragma unroll
    for (int q = 0; q < U; ++q)
      if (on[q]) {
        const double d = (double)pv[q] - (double)tv[q];
        a += d * d;
        c += 1.0;
      }
  }
  s1[threadIdx.x] = a;
  s2[threadIdx.x] = c;
  __syncthreads();
  for (int o = kMseThreads / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      s1[threadIdx.x] += s1[threadIdx.x + o];
      s2[threadIdx.x] += s2[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = s1[0];
    part[2 * blockIdx.x + 1] = s2[0];
  }
}

__global__ __launch_bounds__(256) void k_mse_finish(const double* __restrict__ part, int nb,
                                                    double* __restrict__ out) {
  __shared__ double s1[256], s2[256];
  double a = 0.0, c = 0.0;
  for (int i = threadIdx.x; i < nb; i += 256) {
    a += part[2 * i];
    c += part[2 * i + 1];
  }
  s1[threadIdx.x] = a;
  s2[threadIdx.x] = c;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      s1[threadIdx.x] += s1[threadIdx.x + o];
      s2[threadIdx.x] += s2[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double cnt = fmax(s2[0], 1.0);
    out[0] = s1[0] / cnt;
    out[1] = cnt;
  }
}

__global__ void k_mse_grad(long long nvox, const float* __restrict__ p, const float* __restrict__ t,
                           const uint8_t* __restrict__ m, const double* __restrict__ stats,
                           float* __restrict__ g) {
  const long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nvox) return;
  const double cnt = stats[1];
  g[v] = m[v] ? (float)(2.0 * ((double)p[v] - (double)t[v]) / cnt) : 0.f;
}

__global__ void k_adam(long long n, float* __restrict__ master, float* __restrict__ m,
                       float* __restrict__ v, const float* __restrict__ g,
                       uint16_t* __restrict__ out, float lr, float b1, float b2, float eps,
                       float c1, float c2) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float mh = mi / c1, vh = vi / c2;
  const float p = master[i] - lr * mh / (sqrtf(vh) + eps);
  master[i] = p;
  if (out) out[i] = f2bf(p);
}

__global__ void k_scale(long long n, const float* __restrict__ in, float a, float* __restrict__ out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = a * in[i];
}

__global__ void k_scale_f64(long long n, const float* __restrict__ in, double a,
                            double* __restrict__ out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = a * (double)in[i];
}

__global__ void k_to_bf16(long long n, const float* __restrict__ in, uint16_t* __restrict__ out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = f2bf(in[i]);
}
__global__ void k_from_bf16(long long n, const uint16_t* __restrict__ in, float* __restrict__ out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = bf2f(in[i]);
}

struct Scales {
  float s[64];
};
__global__ void k_pack_input(long long nvs, int ns, const float* __restrict__ sigma,
                             const float* __restrict__ L, Scales sc, uint16_t* __restrict__ x) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nvs * ns) return;
  const int k = (int)(i / nvs);
  const long long v = i - (long long)k * nvs;
  const float* Lk = L + (long long)k * 3 * nvs;
  uint16_t row[8];
  row[0] = f2bf(sigma[i] / sc.s[k]);
  row[1] = f2bf(Lk[v]);
  row[2] = f2bf(Lk[nvs + v]);
  row[3] = f2bf(Lk[2 * nvs + v]);
  row[4] = row[5] = row[6] = row[7] = 0;
  uint4 raw;
  __builtin_memcpy(&raw, row, 16);
  *reinterpret_cast<uint4*>(x + i * 8) = raw;
}

inline unsigned nblk(long long n, int b = 256) { return (unsigned)((n + b - 1) / b); }
inline long long nvox_of(const unet_shape& s) { return (long long)s.n * s.d * s.h * s.w; }

bool act_ok(const unet_act& a, int mult) {
  return a.p && a.ld > 0 && a.c > 0 && a.off >= 0 && a.off + a.c <= a.ld && a.ld % 8 == 0 &&
         a.off % 8 == 0 && a.c % mult == 0;
}
bool shape_ok(const unet_shape& s) { return s.n > 0 && s.d > 0 && s.h > 0 && s.w > 0; }

long long wgrad_chunk(long long nvox) {
  // about 512 chunks, each a multiple of 32 voxels, at least 1024 voxels
  long long c = (nvox + 511) / 512;
  c = std::max<long long>(1024, ((c + 31) / 32) * 32);
  return c;
}


// Size classes of a forward convolution (and of the data gradient, which is
// a forward convolution), as unet_conv_kernel reports them:
//   CONV_TILE:   3x3x3 taps, 8, 16, 32 or 64 input channels, 16-64 output
//                channels, w a multiple of 64 and h of 4, or w = 32 and h a
//                multiple of 8.
//   CONV_GATHER: everything else.
// Both with a blocking that splits the output channels while the grid would
// leave CUs without work.  The gathered kernel (1x1x1 taps; grids where
// conv_choice picks it) runs that blocking, in class CONV_TILE with 64 voxels per
// wave.
enum { CONV_GATHER = 0, CONV_TILE = 1 };
struct ConvPlan {
  int kind, mb, nb, tw;
  long long grid;  // workgroups per output-channel group
};

ConvPlan conv_plan(unet_shape s, int cin, int cout, int taps) {
  ConvPlan p{};
  const long long nv = (long long)s.n * s.d * s.h * s.w;
  const int ob = cout / 16;
  const bool t64 = s.w % 64 == 0 && s.h % 4 == 0, t32 = s.w == 32 && s.h % 8 == 0;
  if (taps == 27 && (t64 || t32) && ob <= 4 &&
      (cin == 8 || cin == 16 || cin == 32 || cin == 64)) {
    p.kind = CONV_TILE;
    p.tw = t64 ? 64 : 32;
    p.mb = 4;  // of the gathered kernel
    const int th = 256 / p.tw;
    const long long tiles = nv / 256;
    const long long lds = 3LL * (th + 2) * (p.tw + 2) * cin * 2;
    const long long target = 256 * std::min<long long>(4, (160 * 1024) / lds);
    p.nb = ob;
    while (p.nb > 1 && tiles * (ob / p.nb) < target) p.nb /= 2;
    p.grid = tiles;
  } else {
    // the widest output block per wave that still gives every CU a
    // workgroup, with 64 voxels per wave, else 16
    p.kind = CONV_GATHER;
    auto wgs = [&](int m, int b) { return ((nv + 64 * m - 1) / (64 * m)) * (ob / b); };
    p.mb = 4;
    p.nb = ob;
    while (p.nb > 1 && wgs(4, p.nb) < 256) p.nb /= 2;
    if (wgs(4, p.nb) < 256) {
      p.mb = 1;
      p.nb = std::min(ob, 2);
      while (p.nb > 1 && wgs(1, p.nb) < 256) p.nb /= 2;
    }
    p.grid = (nv + 64 * p.mb - 1) / (64 * p.mb);
  }
  return p;
}

// Launch plan of the brick kernel (3x3x3 taps): rows per wave, waves along d
// and along the output channels.
struct BrickShape {
  int mb, wd, wc;
};
constexpr BrickShape kBricks[] = {{8, 4, 1}, {8, 2, 2}, {8, 1, 4}, {4, 1, 2}, {4, 2, 1}};
constexpr int kNBricks = 5;

// Chunk size and chunks per pass: all channels at once for 64 and 128.
void brick_chunks(int cin, int* ck, int* nc) {
  *ck = cin % 32 == 0 ? 32 : (cin % 16 == 0 ? 16 : 8);
  *nc = cin == 128 ? 4 : (cin == 64 ? 2 : 1);
}

// Microseconds a CU spends on one work item (with one chunk per pass: on one
// pass), by shape and 8, 16, 32, 64 or 128 channels, with one output block per
// wave and with two; 0: no such instance.  Measured on the U-Net's layers of
// 128^3 and 48 x 56 x 104 inputs with every instance (also 4 x 4 waves along d,
// 4 rows x 4 waves along the channels, and two output blocks with 32 channels
// and more, none of which was the fastest anywhere by more than 4 %).
constexpr double kBrickUs[2][kNBricks][5] = {{{2.1, 2.8, 4.7, 0, 0},
                                              {0, 0, 4.4, 9.0, 20.0},
                                              {0, 0, 4.3, 8.3, 15.5},
                                              {0, 0, 2.2, 4.1, 7.8},
                                              {0.55, 0.93, 1.8, 4.7, 9.0}},
                                             {{3.3, 4.8, 0, 0, 0},
                                              {0, 0, 0, 0, 0},
                                              {0, 0, 0, 0, 0},
                                              {0, 0, 0, 0, 0},
                                              {0.9, 1.6, 0, 0, 0}}};
constexpr int brick_class(int ck, int nc) {
  return ck == 8 ? 0 : (ck == 16 ? 1 : (nc == 1 ? 2 : (nc == 2 ? 3 : 4)));
}
constexpr bool brick_exists(int shape, int ck, int nc, int nb) {
  return kBrickUs[nb - 1][shape][brick_class(ck, nc)] > 0;
}

struct BrickPlan {
  int ck, nc, shape, nb;  // shape < 0: no brick kernel for these sizes
  int nbw, nbh, nbd;
  double us;        // estimated time
  double us_march;  // the same as compared with the marching kernel's
};

// Whether the byte offsets of `planes` whole planes and `rows` rows of xld channels
// stay within a staging descriptor's 2^31.
bool offsets_fit(int planes, int rows, unet_shape s, int xld) {
  return ((double)planes * s.h + rows) * s.w * xld * 2 < (double)((1LL << 31) - 4096);
}

// The instance with the least estimated time (work items in rounds of 256 CUs,
// times kBrickUs): the fastest one on the grids measured, or within 8 % of it.
// Every instance gives bitwise the same result (8 to 128 channels in powers of
// two: all products in (tap, channel) order).  us_march is fitted to grids that
// either of the two kernels might take: there the last-level cache holds the
// operands, and a tall brick takes less than kBrickUs, measured on 2 x 128^3.
BrickPlan brick_plan(unet_shape s, int cin, int xld, int cout) {
  BrickPlan best{};
  best.shape = -1;
  int ck, nc;
  brick_chunks(cin, &ck, &nc);
  double tbest = 0.0;
  for (int sh = 0; sh < kNBricks; ++sh) {
    const BrickShape& b = kBricks[sh];
    for (int nb = 1; nb <= 2; ++nb) {
      if (!brick_exists(sh, ck, nc, nb) || (cout / 16) % (nb * b.wc)) continue;
      // staging offsets (and work items, below) are 32-bit
      if (!offsets_fit(nc > 1 ? b.wd : b.wd + 2, 0, s, xld)) continue;
      const int nbw = (s.w + 15) / 16, nbh = (s.h + b.mb - 1) / b.mb, nbd = (s.d + b.wd - 1) / b.wd;
      const double items = (double)s.n * nbw * nbh * nbd * (cout / 16 / nb / b.wc);
      const double t = std::ceil(items / 256.0) * kBrickUs[nb - 1][sh][brick_class(ck, nc)];
      if (items < 2e9 && (best.shape < 0 || t < tbest)) {
        tbest = t;
        // (passes after the first overlap)
        best = BrickPlan{ck, nc, sh, nb, nbw, nbh, nbd,
                         3 + (nc == 1 && cin > ck ? 0.85 * cin / ck * t : t), 0};
        const double cached = b.mb == 4 ? 1.0 : (b.wc == 4 ? 0.9 : (b.wc == 2 ? 0.87 : 0.85));
        const double used = (double)s.w * s.h * s.d / (16.0 * nbw * b.mb * nbh * b.wd * nbd);
        best.us_march = 4 + t * cached * (0.8 + 0.2 * used);
      }
    }
  }
  return best;
}

template <int CK, int NC, int NB, int SHAPE>
void launch_brick(const ConvArgs& a, hipStream_t st) {
  if constexpr (brick_exists(SHAPE, CK, NC, NB)) {
    constexpr BrickShape b = kBricks[SHAPE];
    using B = Brick<CK, NC, b.mb, NB, b.wd, b.wc>;
    // as many workgroups as run at once
    const dim3 grid((unsigned)std::min(a.total, 256 * std::max(1, B::PER_CU)));
    if constexpr (CK > 8)  // gates come with gradients, of 16 channels and more
      if (a.gate) {
        hipLaunchKernelGGL((k_conv_brick<CK, NC, b.mb, NB, b.wd, b.wc, true>), grid, dim3(B::NT), 0,
                           st, a);
        return;
      }
    hipLaunchKernelGGL((k_conv_brick<CK, NC, b.mb, NB, b.wd, b.wc, false>), grid, dim3(B::NT), 0, st,
                       a);
  }
}

template <int CK, int NC, int NB>
void launch_bricks(int shape, const ConvArgs& a, hipStream_t st) {
  switch (shape) {
    case 0: launch_brick<CK, NC, NB, 0>(a, st); break;
    case 1: launch_brick<CK, NC, NB, 1>(a, st); break;
    case 2: launch_brick<CK, NC, NB, 2>(a, st); break;
    case 3: launch_brick<CK, NC, NB, 3>(a, st); break;
    default: launch_brick<CK, NC, NB, 4>(a, st); break;
  }
}

void enq_brick(const BrickPlan& p, ConvArgs a, int cout, hipStream_t st) {
  a.nbw = p.nbw;
  a.nbh = p.nbh;
  a.nbd = p.nbd;
  a.groups = cout / 16 / p.nb / kBricks[p.shape].wc;
  a.total = (int)((long long)a.s.n * p.nbw * p.nbh * p.nbd * a.groups);
  if (p.ck == 32) {
    if (p.nc == 4)
      launch_bricks<32, 4, 1>(p.shape, a, st);
    else if (p.nc == 2)
      launch_bricks<32, 2, 1>(p.shape, a, st);
    else
      launch_bricks<32, 1, 1>(p.shape, a, st);
  } else if (p.ck == 16) {
    if (p.nb == 2)
      launch_bricks<16, 1, 2>(p.shape, a, st);
    else
      launch_bricks<16, 1, 1>(p.shape, a, st);
  } else {
    if (p.nb == 2)
      launch_bricks<8, 1, 2>(p.shape, a, st);
    else
      launch_bricks<8, 1, 1>(p.shape, a, st);
  }
}

// The marching kernel's instance for these channels, as f(March<...>{}); false if
// it has none.
template <typename F>
bool with_march(int cin, int cout, F&& f) {
  if (cin == 8) return f(unet::March<8, 1, 8, 2, 2>{});
  if (cin == 16)
    return cout % 32 ? f(unet::March<16, 1, 8, 2, 2>{}) : f(unet::March<16, 2, 4, 2, 2>{});
  return cin == 32 && f(unet::March<32, 1, 4, 2, 4>{});
}

struct MarchPlan {
  int nbw, nbh, groups;
  long long steps, nchunk;  // nchunk 0: no marching kernel for these sizes
  bool far;                 // planes past a descriptor's reach
  double us;                // estimated time
};

// The marching kernel's launch and estimated time: one step more than a
// workgroup's share, of 2.7 to 3.8 us each (less where the tile reaches past the
// grid).  The line between this kernel and the bricks follows from 200 ragged and
// regular grids timed with both, us (in brackets the estimates): 16 -> 16 on
// 100x90x120 27.7 / 28.7 (27.2 / 27.2), 48x56x104 15.5 / 11.5 (15.7 / 11.0); 16 -> 32
// on 2 x 64^3 22.8 / 22.7 (22.0 / 20.3), 109x127x135 57.4 / 64.5 (67.5 / 68.0); 32 ->
// 16 on 124x75x49 26.5 / 21.3 (24.8 / 22.8), 100x90x120 42.8 / 43.7 (42.6 / 43.0);
// 32 -> 64 on 2 x 64^3 64.5 / 68.3 (64.5 / 65.9), 83x120x13 42.8 / 23.4.  The kernel
// chosen was within 9 % of the faster one, 0.2 % in the mean (on 220 others 14 %,
// 2 us).  Beyond the cache both take longer: 2 x 128^3 8 -> 16 49 / 61 (51 / 61), 16
// -> 16 72 / 91 (70 / 80), 16 -> 32 135 / 166 (117 / 135), 32 -> 16 131 / 158 (121 /
// 132).  Flat grids, where a brick's other planes lie outside: 16 -> 16 on 512 x 512
// 9.9 / 15.3, 16 -> 32 on 8 x 256 x 256 22 / 43.  Narrow ones, where most of a tile
// does: 32 -> 32 on 4096 x 8 x 8 84 / 29, 16 -> 16 on 4096 x 16 x 16 34 / 24.
MarchPlan march_plan(unet_shape s, int cin, int xld, int cout) {
  MarchPlan p{};
  with_march(cin, cout, [&](auto kc) {
    using K = decltype(kc);
    if (cout / 16 % K::NB) return false;
    const int tw = 16 * K::WW, th = K::MB * K::WH;
    p.far = !offsets_fit(1, 0, s, xld);
    if (p.far && !offsets_fit(0, th + 2, s, xld)) return false;
    p.nbw = (s.w + tw - 1) / tw;
    p.nbh = (s.h + th - 1) / th;
    p.steps = (long long)s.n * p.nbw * p.nbh * s.d;
    p.groups = cout / 16 / K::NB;
    p.nchunk = std::min(p.steps, std::max(1LL, 256LL * K::PER_CU / p.groups));
    const double used = (double)s.w * s.h / ((double)p.nbw * tw * p.nbh * th);
    const double us = cin == 8 ? (p.groups > 1 ? 3.0 : 2.7)
                               : (cin == 16 ? (K::NB == 1 ? 3.8 : 3.4) : 3.5);
    p.us = 5 + (std::ceil((double)p.steps / p.nchunk) + 1) * us * (0.8 + 0.2 * used);
    return true;
  });
  return p;
}

void enq_march(const MarchPlan& p, ConvArgs a, int cout, hipStream_t st) {
  a.nbw = p.nbw;
  a.nbh = p.nbh;
  a.q = (int)(p.steps / p.nchunk);
  a.r = (int)(p.steps % p.nchunk);
  const dim3 grid((unsigned)p.nchunk, (unsigned)p.groups);
  with_march(a.cin, cout, [&](auto kc) {
    using K = decltype(kc);
    auto go = [&](auto gate, auto far) {
      hipLaunchKernelGGL((unet::k_conv_march<K::CK, K::NB, K::MB, K::WW, K::WH,
                                             decltype(gate)::value, decltype(far)::value>),
                         grid, dim3(K::NT), 0, st, a);
    };
    auto go_far = [&](auto gate) {
      if (p.far)
        go(gate, std::true_type{});
      else
        go(gate, std::false_type{});
    };
    if constexpr (K::CK > 8) {  // gates come with gradients, of 16 channels and more
      if (a.gate)
        go_far(std::true_type{});
      else
        go_far(std::false_type{});
    } else {
      go_far(std::false_type{});
    }
    return true;
  });
}

// Estimated time (us) of the gathered kernel: rounds of workgroups over its K
// steps, a latency each at least, and its 2-byte stores.  Measured on grids that
// waste a brick: 128 -> 128 channels on 256 x 256 x 1 170 (estimate 158), on
// 256 x 256 x 2 330 (309); 64 -> 64 80 (64) and 114 (121); 16 -> 16 17 and 20 (19).
double gather_us(unet_shape s, int cin, int cout) {
  const ConvPlan p = conv_plan(s, cin, cout, 27);
  const double steps = (27 * cin + 31) / 32;
  const double rounds = std::ceil((double)p.grid * (cout / 16 / p.nb) / 256);
  // per step and round, by output blocks; rows of 128 bytes and more fall out of the L1
  constexpr double kUs[2][4] = {{0.25, 0.33, 0.45, 0.7}, {0.5, 0.6, 0.85, 1.2}};
  double least = 0.6, us = kUs[cin >= 64][p.nb == 8 ? 3 : p.nb / 2];
  if (p.mb == 1) {  // (of a single column two taps of three load nothing new)
    least = 0.3;
    us = p.nb == 2 ? 0.28 : (s.w == 1 ? 0.07 : 0.2);
  }
  return 8 + steps * std::max(least, rounds * us) + (double)nvox_of(s) * cout * 2 / 0.8e6;
}

// The kernel of a convolution: the one of least estimated time, within margins
// for what the estimates miss.  Gathering is the faster one where a brick is
// mostly padding: 128 -> 128 channels on 256 x 256 x 1 170 us against 838 on
// bricks, on 128 x 128 x 4 172 / 212 (128 x 128 x 6: 337 / 214); 16 -> 16 on
// 256 x 256 x 2 19.7 / 21.4.  (The exceptions on random grids of 1 to 512 voxels a
// side are one or two voxels wide, or tens of microseconds short.)  March or bricks:
// march_plan.
enum { CONV_GATHERED = 0, CONV_BRICK = 1, CONV_MARCH = 2 };
struct ConvChoice {
  int kernel;
  BrickPlan brick;
  MarchPlan march;
};

ConvChoice conv_choice(unet_shape s, int cin, int xld, int cout, int taps) {
  ConvChoice c{};
  if (taps != 27) return c;
  c.brick = brick_plan(s, cin, xld, cout);
  c.march = march_plan(s, cin, xld, cout);
  double us = gather_us(s, cin, cout);
  if (c.brick.shape >= 0 && (s.w <= 2 ? 1.0 : 0.8) * c.brick.us <= us)
    c.kernel = CONV_BRICK, us = c.brick.us_march;
  else
    us *= 0.95;
  if (c.march.nchunk > 0 && c.march.us < us) c.kernel = CONV_MARCH;
  return c;
}

// Fixed-order sum of nchunk partial rows ws[c * rs + i] (i < rs): entries
// below nw go to dw, the rest to db.
void enq_sum_rows(float* ws, long long nchunk, long long rs, long long nw, float* dw, float* db,
                  hipStream_t st) {
  const dim3 grid((unsigned)((rs + 63) / 64));
  if (nchunk < 64)
    hipLaunchKernelGGL(k_sum_rows<4>, grid, dim3(256), 0, st, ws, rs, (int)nchunk, nw, dw, db);
  else
    hipLaunchKernelGGL(k_sum_rows<16>, grid, dim3(1024), 0, st, ws, rs, (int)nchunk, nw, dw, db);
}

// Partial rows and size class of the weight gradient, as unet_wgrad_kernel
// reports them.  Regular grids (rows:
// w a multiple of 32 or 16, h of 4, 8 or a multiple of 16 input channels, 3x3x3
// taps) split into 4-row blocks of 32-voxel rows (w a multiple of 32) or row
// pairs (w = 16).  Channel parts start at 32 x 32 and are halved while the
// grid would have fewer than 512 of them; d ranges of at least 4 planes
// then bring it to about 1024, while the partial rows stay within 8 Mi floats.
// All other grids split into chunks of voxels.  The workspace holds these rows
// (wgrad_rows: or a few more), the voxel-chunk kernel writes them and the tiled
// kernel at most as many.
struct WgradPlan {
  bool rows;
  int ct, ot, ws, dper;
  long long nchunk, rs, vchunk;
};

WgradPlan wgrad_plan(unet_shape s, int cin, int cout, int taps) {
  WgradPlan p{};
  const long long nv = (long long)s.n * s.d * s.h * s.w;
  p.rs = (long long)cout * taps * cin + cout;
  const int ws = s.w % 32 == 0 ? 32 : (s.w == 16 ? 16 : 0);
  p.rows = taps == 27 && ws > 0 && s.h % 4 == 0 && (cin == 8 || cin % 16 == 0) && cout % 16 == 0;
  if (p.rows) {
    auto blocks = [](int ot, int ct) { return (ot / 16) * (std::max(ct, 16) / 16); };
    const int pmin = ws == 16 ? 2 : 1;  // a 4-row block of w = 16 holds only 2 units
    int ot = cout % 32 == 0 ? 32 : 16;
    int ct = cin == 8 ? 8 : (cin % 32 == 0 ? 32 : 16);
    const long long cols = (long long)s.n * (s.w / ws) * (s.h / 4);
    const int maxnds = std::max(1, s.d / 4);
    for (;;) {
      const long long base = cols * (cin / ct) * (cout / ot);
      if (base * maxnds >= 512) break;
      if (ot == 32 && ot >= ct && blocks(16, ct) >= pmin)
        ot = 16;
      else if (ct == 32 && blocks(ot, 16) >= pmin)
        ct = 16;
      else
        break;
    }
    p.rows = blocks(ot, ct) >= pmin;
    if (p.rows) {
      p.ct = ct;
      p.ot = ot;
      p.ws = ws;
      const long long base = cols * (cin / ct) * (cout / ot);
      const long long want = (1024 + base - 1) / base;
      int nds = (int)std::min<long long>(maxnds, std::max<long long>(1, want));
      // partial rows beyond 8 Mi floats cost more to sum than the split gains
      while (nds > 1 && cols * nds * p.rs > (8LL << 20)) nds = (nds + 1) / 2;
      p.dper = (s.d + nds - 1) / nds;
      p.nchunk = cols * ((s.d + p.dper - 1) / p.dper);
    }
  }
  if (!p.rows) {
    p.vchunk = wgrad_chunk(nv);
    p.nchunk = (nv + p.vchunk - 1) / p.vchunk;
  }
  return p;
}

// Whether the tiled kernel (unet_wgrad.h) takes a weight gradient: 3x3x3 taps,
// 8 or a multiple of 16 input channels, voxels that an int counts and rows of a
// tile (34 at most) that a buffer descriptor spans.
bool wgrad_tiled(unet_shape s, int cin, int ld, int taps) {
  return taps == 27 && (cin == 8 || cin % 16 == 0) && nvox_of(s) < (1LL << 31) &&
         offsets_fit(0, 36, s, ld);
}

// Partial rows that the workspace holds: the plan's, and up to 64 where they take
// no more than 8 Mi floats, for grids whose voxels are few and whose tiles many
// (the plan counts chunks of 1024 voxels).
long long wgrad_rows(const WgradPlan& p) {
  return std::max(p.nchunk, std::min(64LL, (8LL << 20) / p.rs));
}

// Estimated time (us) of the tiled kernel on shares of few planes (a step's latency
// each, two short steps more at the start of a tile) and of writing and summing m
// rows.
double wgrad_us(unet_shape s, long long steps, int m, long long rs) {
  const long long share = (steps + m - 1) / m;
  return 7.5 + 2.0 * share + 1.4 * ((share + s.d - 1) / s.d) + m * (double)rs * 8 / 3e6;
}

// The tiled kernel's launch: instance, octets along w of a tile (2^ltwo), tiles
// along w and h, channel parts and shares.
struct WgradChoice {
  int ct, ot, ltwo, nbw, nbh, nparts, nchunk;
  long long steps;
  double cost;
  bool tiled;  // false: the voxel-chunk kernel is the faster one
};

// f(Wgrad<...>{}) of the instance for CT input and OT output channels
template <typename F>
auto with_wgrad(int ct, int ot, F&& f) {
  if (ct == 8) return f(unet::Wgrad<8, 16, 2, 512>{});
  if (ct == 16)
    return ot == 16 ? f(unet::Wgrad<16, 16, 2, 512>{}) : f(unet::Wgrad<16, 32, 2, 512>{});
  return ot == 16 ? f(unet::Wgrad<32, 16, 4, 256>{}) : f(unet::Wgrad<32, 32, 4, 256>{});
}

// Its workgroups fill every CU once (a CU holds PER_CU), split over
// the channel parts; the tile is the one that pads the grid least, then the
// one with the smallest halo (64 wide only where that saves a third of the tiles:
// grids of few rows; 48 -> 16 channels on 4 x 38x4x288 39 us, 56 at 32 wide).  More
// shares than the plan's rows where that takes a fifth off the estimate: 32 -> 32
// on 127x2x1 320 us with its one share, 16 with 64; 16 -> 16 on 1x1x4096 135 and 16.
// Channel parts of 32 unless parts of 16 leave a
// workgroup fewer steps, six counted for its start and end: the plan's rows
// bound the workgroups of a part (32 -> 32 channels on 24x28x52: 35 rows,
// parts of 32 31.5 us, of 16 18.2; 32 -> 16 on 2 x 128^3: 110 and 136).
WgradChoice wgrad_tiling(unet_shape s, int cin, int cout, const WgradPlan& p) {
  auto plan = [&](int ct, int ot, bool flat) {
    return with_wgrad(ct, ot, [&](auto kc) {
      using K = decltype(kc);
      WgradChoice c{};
      c.ct = K::CT;
      c.ot = K::OT;
      long long tiles = -1, halo = 0;
      for (int lg : {2, 1, 0, 3}) {
        const int two = 1 << lg, rows = K::NOC / two * K::RL;
        if (two < K::TWO_LO || two > (flat ? K::TWO_HI : 4)) continue;
        const int nbw = (s.w + 8 * two - 1) / (8 * two), nbh = (s.h + rows - 1) / rows;
        const long long nt = (long long)nbw * nbh * s.n, h = (rows + 2LL) * (8 * two + 2);
        if (tiles >= 0 && (nt > tiles || (nt == tiles && h >= halo))) continue;
        if (two == 8 && 3 * nt > 2 * tiles) continue;
        tiles = nt;
        halo = h;
        c.ltwo = lg;
        c.nbw = nbw;
        c.nbh = nbh;
      }
      c.steps = tiles * s.d;
      c.nparts = cin / K::CT * (cout / K::OT);
      const long long fill = std::min(c.steps, std::max(1LL, 256LL * K::PER_CU / c.nparts));
      c.nchunk = (int)std::min(p.nchunk, fill);
      // more rows than the plan's where a share would walk long alone
      const int most = (int)std::min({wgrad_rows(p), fill, std::max(1LL, 256LL / c.nparts)});
      int best = c.nchunk;
      for (int m = c.nchunk + 1; m <= most; ++m)
        if (wgrad_us(s, c.steps, m, p.rs) < wgrad_us(s, c.steps, best, p.rs)) best = m;
      if (wgrad_us(s, c.steps, best, p.rs) < 0.8 * wgrad_us(s, c.steps, c.nchunk, p.rs))
        c.nchunk = best;
      // a second workgroup on a CU takes half its time again (measured), more than
      // the CUs hold run in turns
      const double per_cu = (double)c.nchunk * c.nparts / 256;
      const double turns = per_cu <= 1 ? 1 : (per_cu <= 2 ? 0.5 + 0.5 * per_cu : per_cu * 0.75);
      c.cost = ((c.steps + c.nchunk - 1) / c.nchunk + 6) * turns;
      return c;
    });
  };
  if (cin == 8) return plan(8, 16, true);
  if (cin % 32 && cout % 32) return plan(16, 16, true);
  const WgradChoice base = plan(16, 16, false);
  const WgradChoice wide = plan(cin % 32 ? 16 : 32, cout % 32 ? 16 : 32, true);
  return wide.cost <= base.cost ? wide : base;
}

// Tiles or voxel chunks, by estimate: chunks (their bias sums walk up to 1024
// voxels one after another, 85 us) are the faster ones on irregular grids of a few
// voxels only: 128 -> 128 on 2x2x2 13.2 us and 14.0, on 1x1x4096 159 and 40; 16 ->
// 16 on 48x56x104 211 and 37, 64 -> 128 on 8x8x8 82 and 36.
WgradChoice wgrad_choice(unet_shape s, int cin, int cout, const WgradPlan& p) {
  WgradChoice c = wgrad_tiling(s, cin, cout, p);
  const int ob = cout / 16;
  if (p.rows || !(ob == 1 || ob == 2 || ob == 4 || ob == 8)) {
    c.tiled = true;
    return c;
  }
  const double nv = (double)nvox_of(s), vchunk = std::min(nv, (double)p.vchunk);
  const double wgs = std::ceil(27 * cin / 64.0) * p.nchunk;
  const double us = ob == 1 ? 12 : (ob == 2 ? 30 : (ob == 4 ? 43 : 50));
  const double chunks = 11.5 + vchunk / 1024 * (85 + wgs / 256 * us) + p.nchunk * p.rs * 8 / 3e6;
  c.tiled = wgrad_us(s, c.steps, c.nchunk, p.rs) <= chunks;
  return c;
}

void enq_wgrad(unet_shape s, unet_act x, unet_act dy, const WgradChoice& c, long long rs, float* ws,
               hipStream_t st) {
  const WgradArgs a{s, (const uint16_t*)x.p, x.ld, x.off, x.c, (const uint16_t*)dy.p, dy.ld, dy.off,
                    dy.c, c.ltwo, c.nbw, c.nbh, x.c / c.ct, (int)(c.steps / c.nchunk),
                    (int)(c.steps % c.nchunk), rs, ws};
  with_wgrad(c.ct, c.ot, [&](auto kc) {
    using K = decltype(kc);
    const dim3 grid(c.nchunk, c.nparts);
    if (offsets_fit(1, 0, s, std::max(x.ld, dy.ld)))
      hipLaunchKernelGGL((unet::k_wgrad<K::CT, K::OT, K::RL, K::NT, false>), grid, dim3(K::NT), 0,
                         st, a);
    else
      hipLaunchKernelGGL((unet::k_wgrad<K::CT, K::OT, K::RL, K::NT, true>), grid, dim3(K::NT), 0,
                         st, a);
  });
}

}  // namespace

extern "C" {

const char* unet_last_error(void) { return g_err.c_str(); }

unet_status unet_mfma_selfcheck(const void* a, const void* b, float* out, void* stream) {
  if (!a || !b || !out) return ufail(UNET_EINVAL, "NULL argument");
  hipLaunchKernelGGL(k_mfma_selfcheck, dim3(1), dim3(64), 0, (hipStream_t)stream,
                     (const uint16_t*)a, (const uint16_t*)b, out);
  UHIP(hipGetLastError());
  return UNET_OK;
}

static unet_status conv(unet_shape s, unet_act x, const void* w, const float* bias, int32_t taps,
                        unet_act y, float* out_f32, int32_t relu, const unet_act* gate,
                        void* stream) {
  if (!shape_ok(s) || !w || (taps != 27 && taps != 1)) return ufail(UNET_EINVAL, "bad conv args");
  if (!act_ok(x, 8) || x.c > 256)
    return ufail(UNET_EINVAL, "bad input view (ld/off/c multiples of 8, c <= 256)");
  if (nvox_of(s) >= (1LL << 31)) return ufail(UNET_EINVAL, "too many voxels (limit 2^31)");
  if (y.c % 16 || y.c > 128 || y.c <= 0 || y.ld % 8 || y.off % 8 || y.off + y.c > y.ld ||
      (!out_f32 && !y.p))
    return ufail(UNET_EINVAL, "bad output view (c multiple of 16, <= 128)");
  const int ob = y.c / 16;
  if (ob != 1 && ob != 2 && ob != 4 && ob != 8)
    return ufail(UNET_EINVAL, "output channels must be 16, 32, 64 or 128");
  hipStream_t st = (hipStream_t)stream;
  const ConvChoice ch = conv_choice(s, x.c, x.ld, y.c, taps);
  if (ch.kernel != CONV_GATHERED) {
    ConvArgs a{};
    a.s = s;
    a.x = (const uint16_t*)x.p;
    a.xld = x.ld;
    a.xoff = x.off;
    a.cin = x.c;
    a.w = (const uint16_t*)w;
    a.bias = bias;
    a.y = (uint16_t*)y.p;
    a.yld = y.ld;
    a.yoff = y.off;
    a.yf = out_f32;
    a.relu = relu;
    a.wide = (uintptr_t)(out_f32 ? (void*)out_f32 : y.p) % 16 == 0;
    if (gate) {
      a.gate = (const uint16_t*)gate->p;
      a.gld = gate->ld;
      a.goff = gate->off;
      a.wide = a.wide && (uintptr_t)gate->p % 16 == 0;
    }
    if (ch.kernel == CONV_MARCH)
      enq_march(ch.march, a, y.c, st);
    else
      enq_brick(ch.brick, a, y.c, st);
    UHIP(hipGetLastError());
    return UNET_OK;
  }
  const ConvPlan p = conv_plan(s, x.c, y.c, taps);
  const uint16_t* xp = (const uint16_t*)x.p;
  const uint16_t* wp = (const uint16_t*)w;
  uint16_t* yp = (uint16_t*)y.p;
  const dim3 grid((unsigned)p.grid, (unsigned)(ob / p.nb));
  auto nbs = [&](auto fn) {  // NB as a compile-time constant
    switch (p.nb) {
      case 1: fn(std::integral_constant<int, 1>{}); break;
      case 2: fn(std::integral_constant<int, 2>{}); break;
      case 4: fn(std::integral_constant<int, 4>{}); break;
      default: fn(std::integral_constant<int, 8>{}); break;
    }
  };
  nbs([&](auto nbc) {
    constexpr int NB = decltype(nbc)::value;
    if (p.mb == 4)
      hipLaunchKernelGGL((k_conv_fwd<4, NB>), grid, dim3(256), 0, st, s, xp, x.ld, x.off, x.c, wp,
                         bias, taps, yp, y.ld, y.off, out_f32, relu);
    else if constexpr (NB <= 2)
      hipLaunchKernelGGL((k_conv_fwd<1, NB>), grid, dim3(256), 0, st, s, xp, x.ld, x.off, x.c, wp,
                         bias, taps, yp, y.ld, y.off, out_f32, relu);
  });
  UHIP(hipGetLastError());
  return gate ? unet_relu_bwd(s, *gate, y, y, stream) : UNET_OK;
}

unet_status unet_conv_fwd(unet_shape s, unet_act x, const void* w, const float* bias, int32_t taps,
                          unet_act y, float* out_f32, int32_t relu, void* stream) {
  return conv(s, x, w, bias, taps, y, out_f32, relu, nullptr, stream);
}

unet_status unet_conv_kernel(unet_shape s, int32_t cin, int32_t cout, int32_t taps,
                             int32_t* info) {
  if (!info || !shape_ok(s) || cin <= 0 || cin % 8 || cin > 256 || (taps != 27 && taps != 1) ||
      (cout != 16 && cout != 32 && cout != 64 && cout != 128))
    return ufail(UNET_EINVAL, "bad conv_kernel args");
  const ConvPlan p = conv_plan(s, cin, cout, taps);
  info[0] = p.kind;
  info[1] = p.kind == CONV_GATHER ? p.mb : p.tw;
  info[2] = p.nb;
  info[3] = cout / 16 / p.nb;
  return UNET_OK;
}

unet_status unet_conv_launch(unet_shape s, int32_t cin, int32_t xld, int32_t cout, int32_t taps,
                             int32_t* info) {
  if (!info || !shape_ok(s) || cin <= 0 || cin % 8 || cin > 256 || xld < cin || xld % 8 ||
      (taps != 27 && taps != 1) || (cout != 16 && cout != 32 && cout != 64 && cout != 128) ||
      nvox_of(s) >= (1LL << 31))
    return ufail(UNET_EINVAL, "bad conv_launch args");
  const ConvChoice c = conv_choice(s, cin, xld, cout, taps);
  std::fill(info, info + 8, 0);
  info[0] = c.kernel;
  if (c.kernel == CONV_MARCH) {
    with_march(cin, cout, [&](auto kc) {
      using K = decltype(kc);
      info[1] = K::CK, info[2] = 1, info[3] = K::MB, info[4] = K::NB, info[5] = K::WW,
      info[6] = K::WH;
      return true;
    });
    info[7] = (int32_t)(c.march.nchunk * c.march.groups);
  } else if (c.kernel == CONV_BRICK) {
    const BrickShape& b = kBricks[c.brick.shape];
    info[1] = c.brick.ck, info[2] = c.brick.nc, info[3] = b.mb, info[4] = c.brick.nb,
    info[5] = b.wd, info[6] = b.wc;
    info[7] = (int32_t)((long long)s.n * c.brick.nbw * c.brick.nbh * c.brick.nbd *
                        (cout / 16 / c.brick.nb / b.wc));
  } else {
    const ConvPlan p = conv_plan(s, cin, cout, taps);
    info[3] = p.mb, info[4] = p.nb;
  }
  return UNET_OK;
}

static unet_status dgrad(unet_shape s, unet_act dy, const void* w, int32_t taps, unet_act dx,
                         const unet_act* gate, void* wflip, void* stream) {
  if (!shape_ok(s) || !w || !wflip || (taps != 27 && taps != 1))
    return ufail(UNET_EINVAL, "bad dgrad args");
  if (!act_ok(dy, 16) || !act_ok(dx, 16)) return ufail(UNET_EINVAL, "bad dgrad views");
  const long long n = (long long)dy.c * dx.c * taps;
  hipLaunchKernelGGL(k_flip_weights, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream,
                     (const uint16_t*)w, (uint16_t*)wflip, dy.c, dx.c, taps);
  UHIP(hipGetLastError());
  return conv(s, dy, wflip, nullptr, taps, dx, nullptr, 0, gate, stream);
}

unet_status unet_conv_dgrad(unet_shape s, unet_act dy, const void* w, int32_t taps, unet_act dx,
                            void* wflip, void* stream) {
  return dgrad(s, dy, w, taps, dx, nullptr, wflip, stream);
}

unet_status unet_conv_dgrad_relu(unet_shape s, unet_act dy, const void* w, int32_t taps, unet_act y,
                                 unet_act dx, void* wflip, void* stream) {
  if (!act_ok(y, 16) || y.c != dx.c) return ufail(UNET_EINVAL, "bad dgrad gate view");
  return dgrad(s, dy, w, taps, dx, &y, wflip, stream);
}

size_t unet_wgrad_workspace(unet_shape s, int32_t cin, int32_t cout, int32_t taps) {
  if (!shape_ok(s) || cin <= 0 || cout <= 0 || (taps != 27 && taps != 1)) return 0;
  const WgradPlan p = wgrad_plan(s, cin, cout, taps);
  return (size_t)(wgrad_rows(p) * p.rs) * sizeof(float);
}

unet_status unet_wgrad_kernel(unet_shape s, int32_t cin, int32_t cout, int32_t taps,
                              int32_t* info) {
  if (!info || !shape_ok(s) || cin <= 0 || cin % 8 || cout <= 0 || cout % 16 || cout > 128 ||
      (taps != 27 && taps != 1))
    return ufail(UNET_EINVAL, "bad wgrad_kernel args");
  const WgradPlan p = wgrad_plan(s, cin, cout, taps);
  info[0] = p.rows ? 1 : 0;
  info[1] = p.ct;
  info[2] = p.ot;
  info[3] = p.ws;
  info[4] = (int32_t)p.nchunk;
  info[5] = p.dper;
  return UNET_OK;
}

unet_status unet_wgrad_launch(unet_shape s, int32_t cin, int32_t xld, int32_t cout, int32_t dld,
                              int32_t taps, int32_t* info) {
  if (!info || !shape_ok(s) || cin <= 0 || cin % 8 || xld < cin || xld % 8 || cout <= 0 ||
      cout % 16 || cout > 128 || dld < cout || dld % 8 || (taps != 27 && taps != 1))
    return ufail(UNET_EINVAL, "bad wgrad_launch args");
  const WgradPlan p = wgrad_plan(s, cin, cout, taps);
  std::fill(info, info + 6, 0);
  if (!wgrad_tiled(s, cin, std::max(xld, dld), taps)) return UNET_OK;
  const WgradChoice c = wgrad_choice(s, cin, cout, p);
  if (!c.tiled) return UNET_OK;
  info[0] = 1, info[1] = c.ct, info[2] = c.ot, info[3] = 1 << c.ltwo, info[4] = c.nchunk,
  info[5] = c.nparts;
  return UNET_OK;
}

unet_status unet_conv_wgrad(unet_shape s, unet_act x, unet_act dy, int32_t taps, float* dw,
                            float* db, void* ws, void* stream) {
  if (!shape_ok(s) || !dw || !db || !ws || (taps != 27 && taps != 1))
    return ufail(UNET_EINVAL, "bad wgrad args");
  if (!act_ok(x, 8) || !act_ok(dy, 16) || dy.c > 128) return ufail(UNET_EINVAL, "bad wgrad views");
  hipStream_t st = (hipStream_t)stream;
  const WgradPlan p = wgrad_plan(s, x.c, dy.c, taps);
  const int K = taps * x.c;
  const long long nw = (long long)dy.c * K;
  float* wsp = (float*)ws;
  const uint16_t* xp = (const uint16_t*)x.p;
  const uint16_t* dp = (const uint16_t*)dy.p;
  const int obs = dy.c / 16;
  if (!p.rows && obs != 1 && obs != 2 && obs != 4 && obs != 8)
    return ufail(UNET_EINVAL, "output channels must be 16, 32, 64 or 128");
  long long nchunk = p.nchunk;
  WgradChoice c{};
  if (wgrad_tiled(s, x.c, std::max(x.ld, dy.ld), taps)) c = wgrad_choice(s, x.c, dy.c, p);
  if (c.tiled) {
    nchunk = c.nchunk;
    enq_wgrad(s, x, dy, c, p.rs, wsp, st);
  } else {
    const long long nv = nvox_of(s);
    const long long vchunk = p.rows ? ((nv + nchunk - 1) / nchunk + 31) / 32 * 32 : p.vchunk;
    nchunk = (nv + vchunk - 1) / vchunk;
    const dim3 grid((K + 63) / 64, (unsigned)nchunk);
    auto launch = [&](auto ob, int o) {  // output channels from block o on
      hipLaunchKernelGGL(k_conv_wgrad<decltype(ob)::value>, grid, dim3(256), 0, st, s, xp, x.ld,
                         x.off, x.c, dp, dy.ld, dy.off + 16 * o, taps, vchunk, p.rs,
                         wsp + 16LL * o * K);
    };
    switch (obs) {
      case 2: launch(std::integral_constant<int, 2>{}, 0); break;
      case 4: launch(std::integral_constant<int, 4>{}, 0); break;
      case 8: launch(std::integral_constant<int, 8>{}, 0); break;
      default:  // (of 3, 5, 6 and 7 blocks: regular grids past the tiled kernel's reach)
        for (int o = 0; o < obs; ++o) launch(std::integral_constant<int, 1>{}, o);
    }
    hipLaunchKernelGGL(k_bias_partial, dim3((unsigned)nchunk), dim3(128), 0, st, s, dp, dy.ld,
                       dy.off, dy.c, vchunk, p.rs, wsp + nw);
  }
  UHIP(hipGetLastError());
  enq_sum_rows(wsp, nchunk, p.rs, nw, dw, db, st);
  UHIP(hipGetLastError());
  return UNET_OK;
}

unet_status unet_relu_bwd(unet_shape s, unet_act y, unet_act dy, unet_act out, void* stream) {
  if (!shape_ok(s) || !act_ok(y, 1) || !act_ok(dy, 1) || !act_ok(out, 1) || y.c != dy.c ||
      y.c != out.c)
    return ufail(UNET_EINVAL, "bad relu_bwd views");
  const long long n = nvox_of(s) * y.c;
  if (y.c % 8 == 0)
    hipLaunchKernelGGL(k_relu_bwd8, dim3(nblk(n / 8)), dim3(256), 0, (hipStream_t)stream,
                       nvox_of(s), y.c / 8, (const uint16_t*)y.p, y.ld, y.off,
                       (const uint16_t*)dy.p, dy.ld, dy.off, (uint16_t*)out.p, out.ld, out.off);
  else
    hipLaunchKernelGGL(k_relu_bwd, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, nvox_of(s),
                       y.c, (const uint16_t*)y.p, y.ld, y.off, (const uint16_t*)dy.p, dy.ld,
                       dy.off, (uint16_t*)out.p, out.ld, out.off);
  UHIP(hipGetLastError());
  return UNET_OK;
}

unet_status unet_pool_fwd(unet_shape f, unet_act x, unet_act y, void* stream) {
  if (!shape_ok(f) || f.d % 2 || f.h % 2 || f.w % 2 || !act_ok(x, 1) || !act_ok(y, 1) || x.c != y.c)
    return ufail(UNET_EINVAL, "bad pool args");
  const long long n = nvox_of(f) / 8 * x.c;
  if (x.c % 8 == 0)
    hipLaunchKernelGGL(k_pool_fwd8, dim3(nblk(n / 8)), dim3(256), 0, (hipStream_t)stream, f,
                       x.c / 8, (const uint16_t*)x.p, x.ld, x.off, (uint16_t*)y.p, y.ld, y.off);
  else
    hipLaunchKernelGGL(k_pool_fwd, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, f, x.c,
                       (const uint16_t*)x.p, x.ld, x.off, (uint16_t*)y.p, y.ld, y.off);
  UHIP(hipGetLastError());
  return UNET_OK;
}

static unet_status pool_bwd(unet_shape f, unet_act dy, unet_act dx, int32_t accumulate,
                            const unet_act* gate, void* stream) {
  if (!shape_ok(f) || f.d % 2 || f.h % 2 || f.w % 2 || !act_ok(dy, 1) || !act_ok(dx, 1) ||
      dx.c != dy.c)
    return ufail(UNET_EINVAL, "bad pool_bwd args");
  const long long n = nvox_of(f) * dx.c;
  if (dx.c % 8 == 0)
    hipLaunchKernelGGL(k_pool_bwd8, dim3(nblk(n / 8)), dim3(256), 0, (hipStream_t)stream, f,
                       dx.c / 8, (const uint16_t*)dy.p, dy.ld, dy.off, (uint16_t*)dx.p, dx.ld,
                       dx.off, accumulate, gate ? (const uint16_t*)gate->p : nullptr,
                       gate ? gate->ld : 0, gate ? gate->off : 0);
  else
    hipLaunchKernelGGL(k_pool_bwd, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, f, dx.c,
                       (const uint16_t*)dy.p, dy.ld, dy.off, (uint16_t*)dx.p, dx.ld, dx.off,
                       accumulate);
  UHIP(hipGetLastError());
  return gate && dx.c % 8 ? unet_relu_bwd(f, *gate, dx, dx, stream) : UNET_OK;
}

unet_status unet_pool_bwd(unet_shape f, unet_act dy, unet_act dx, int32_t accumulate, void* stream) {
  return pool_bwd(f, dy, dx, accumulate, nullptr, stream);
}

unet_status unet_pool_bwd_relu(unet_shape f, unet_act dy, unet_act y, unet_act dx,
                               int32_t accumulate, void* stream) {
  if (!act_ok(y, 1) || y.c != dx.c) return ufail(UNET_EINVAL, "bad pool_bwd gate view");
  return pool_bwd(f, dy, dx, accumulate, &y, stream);
}

unet_status unet_up_fwd(unet_shape cs, unet_act x, unet_act y, void* stream) {
  if (!shape_ok(cs) || !act_ok(x, 1) || !act_ok(y, 1) || x.c != y.c)
    return ufail(UNET_EINVAL, "bad up args");
  const long long n = nvox_of(cs) * 8 * x.c;
  if (x.c % 8 == 0)
    hipLaunchKernelGGL(k_up_fwd8, dim3(nblk(n / 8)), dim3(256), 0, (hipStream_t)stream, cs,
                       x.c / 8, (const uint16_t*)x.p, x.ld, x.off, (uint16_t*)y.p, y.ld, y.off);
  else
    hipLaunchKernelGGL(k_up_fwd, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, cs, x.c,
                       (const uint16_t*)x.p, x.ld, x.off, (uint16_t*)y.p, y.ld, y.off);
  UHIP(hipGetLastError());
  return UNET_OK;
}

static unet_status up_bwd(unet_shape cs, unet_act dy, unet_act dx, const unet_act* gate,
                          void* stream) {
  if (!shape_ok(cs) || !act_ok(dy, 1) || !act_ok(dx, 1) || dx.c != dy.c)
    return ufail(UNET_EINVAL, "bad up_bwd args");
  const long long n = nvox_of(cs) * dx.c;
  if (dx.c % 8 == 0)
    hipLaunchKernelGGL(k_up_bwd8, dim3(nblk(n / 8)), dim3(256), 0, (hipStream_t)stream, cs,
                       dx.c / 8, (const uint16_t*)dy.p, dy.ld, dy.off, (uint16_t*)dx.p, dx.ld,
                       dx.off, gate ? (const uint16_t*)gate->p : nullptr, gate ? gate->ld : 0,
                       gate ? gate->off : 0);
  else
    hipLaunchKernelGGL(k_up_bwd, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, cs, dx.c,
                       (const uint16_t*)dy.p, dy.ld, dy.off, (uint16_t*)dx.p, dx.ld, dx.off);
  UHIP(hipGetLastError());
  return gate && dx.c % 8 ? unet_relu_bwd(cs, *gate, dx, dx, stream) : UNET_OK;
}

unet_status unet_up_bwd(unet_shape cs, unet_act dy, unet_act dx, void* stream) {
  return up_bwd(cs, dy, dx, nullptr, stream);
}

unet_status unet_up_bwd_relu(unet_shape cs, unet_act dy, unet_act y, unet_act dx, void* stream) {
  if (!act_ok(y, 1) || y.c != dx.c) return ufail(UNET_EINVAL, "bad up_bwd gate view");
  return up_bwd(cs, dy, dx, &y, stream);
}

unet_status unet_head_fwd(unet_shape s, unet_act x, const float* w, const float* b, float* y,
                          void* stream) {
  if (!shape_ok(s) || !act_ok(x, 1) || !w || !b || !y) return ufail(UNET_EINVAL, "bad head args");
  const long long nv = nvox_of(s);
  if (x.c % 8 == 0)
    hipLaunchKernelGGL(k_head_fwd8, dim3(nblk(nv)), dim3(256), 0, (hipStream_t)stream, nv,
                       x.c / 8, (const uint16_t*)x.p, x.ld, x.off, w, b, y);
  else
    hipLaunchKernelGGL(k_head_fwd, dim3(nblk(nv)), dim3(256), 0, (hipStream_t)stream, nv, x.c,
                       (const uint16_t*)x.p, x.ld, x.off, w, b, y);
  UHIP(hipGetLastError());
  return UNET_OK;
}

size_t unet_head_workspace(unet_shape s, int32_t cin) {
  if (!shape_ok(s) || cin <= 0) return 0;
  const long long nv = nvox_of(s);
  const long long ch = wgrad_chunk(nv);
  const long long nc = (nv + ch - 1) / ch;
  return (size_t)nc * (cin + 1) * sizeof(float);
}

static unet_status head_bwd(unet_shape s, unet_act x, const float* w, const float* dy, unet_act dx,
                            bool gate, float* dw, float* db, void* ws, void* stream) {
  if (!shape_ok(s) || !act_ok(x, 1) || !w || !dy || !dw || !db || !ws)
    return ufail(UNET_EINVAL, "bad head_bwd args");
  hipStream_t st = (hipStream_t)stream;
  const long long nv = nvox_of(s);
  const bool v8 = x.c % 8 == 0 && x.c <= 256;
  if (dx.p) {
    if (!act_ok(dx, 1) || dx.c != x.c) return ufail(UNET_EINVAL, "bad head dx view");
    if (!v8)
      hipLaunchKernelGGL(k_head_dgrad, dim3(nblk(nv * x.c)), dim3(256), 0, st, nv, x.c, w, dy,
                         (uint16_t*)dx.p, dx.ld, dx.off);
  }
  const long long ch = wgrad_chunk(nv);
  const int nc = (int)((nv + ch - 1) / ch);
  float* wsp = (float*)ws;
  if (v8)
    hipLaunchKernelGGL(k_head_bwd8, dim3(nc), dim3(256), 0, st, nv, x.c / 8,
                       (const uint16_t*)x.p, x.ld, x.off, w, dy, (uint16_t*)dx.p, dx.ld, dx.off,
                       gate ? 1 : 0, ch, wsp);
  else
    hipLaunchKernelGGL(k_head_wgrad_partial, dim3(nc), dim3(64), 0, st, nv, x.c,
                       (const uint16_t*)x.p, x.ld, x.off, dy, ch, wsp);
  // wsp[chunk][c + 1] -> dw[c] (the last column is the bias gradient)
  enq_sum_rows(wsp, nc, x.c + 1, x.c, dw, db, st);
  UHIP(hipGetLastError());
  return gate && dx.p && !v8 ? unet_relu_bwd(s, x, dx, dx, stream) : UNET_OK;
}

unet_status unet_head_bwd(unet_shape s, unet_act x, const float* w, const float* dy, unet_act dx,
                          float* dw, float* db, void* ws, void* stream) {
  return head_bwd(s, x, w, dy, dx, false, dw, db, ws, stream);
}

unet_status unet_head_bwd_relu(unet_shape s, unet_act x, const float* w, const float* dy,
                               unet_act dx, float* dw, float* db, void* ws, void* stream) {
  return head_bwd(s, x, w, dy, dx, true, dw, db, ws, stream);
}

unet_status unet_mse(unet_shape s, const float* pred, const float* target, const uint8_t* mask,
                     float* dpred, double* stats_dev, double* loss, void* stream) {
  if (!shape_ok(s) || !pred || !target || !mask || !dpred || !stats_dev)
    return ufail(UNET_EINVAL, "bad mse args");
  hipStream_t st = (hipStream_t)stream;
  const long long nv = nvox_of(s);
  const int nb = 256;
  double* part = stats_dev + 2;  // caller provides 2 + 2 * 256 doubles
  hipLaunchKernelGGL(k_mse_partial, dim3(nb), dim3(kMseThreads), 0, st, nv, pred, target, mask, part);
  hipLaunchKernelGGL(k_mse_finish, dim3(1), dim3(256), 0, st, part, nb, stats_dev);
  hipLaunchKernelGGL(k_mse_grad, dim3(nblk(nv)), dim3(256), 0, st, nv, pred, target, mask,
                     stats_dev, dpred);
  UHIP(hipGetLastError());
  if (loss) {
    UHIP(hipMemcpyAsync(loss, stats_dev, sizeof(double), hipMemcpyDeviceToHost, st));
    UHIP(hipStreamSynchronize(st));
  }
  return UNET_OK;
}

unet_status unet_adam(int64_t n, float* master, float* m, float* v, const float* g, void* bf16_out,
                      float lr, float beta1, float beta2, float eps, int32_t t, void* stream) {
  if (n <= 0 || !master || !m || !v || !g || t < 1) return ufail(UNET_EINVAL, "bad adam args");
  const float c1 = 1.f - std::pow(beta1, (float)t), c2 = 1.f - std::pow(beta2, (float)t);
  hipLaunchKernelGGL(k_adam, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, (long long)n, master,
                     m, v, g, (uint16_t*)bf16_out, lr, beta1, beta2, eps, c1, c2);
  UHIP(hipGetLastError());
  return UNET_OK;
}

unet_status unet_scale(int64_t n, const float* in, float a, float* out, void* stream) {
  if (n <= 0 || !in || !out) return ufail(UNET_EINVAL, "bad args");
  hipLaunchKernelGGL(k_scale, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, (long long)n, in, a,
                     out);
  UHIP(hipGetLastError());
  return UNET_OK;
}

unet_status unet_scale_f64(int64_t n, const float* in, double a, double* out, void* stream) {
  if (n <= 0 || !in || !out) return ufail(UNET_EINVAL, "bad args");
  hipLaunchKernelGGL(k_scale_f64, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, (long long)n,
                     in, a, out);
  UHIP(hipGetLastError());
  return UNET_OK;
}

unet_status unet_to_bf16(int64_t n, const float* in, void* out, void* stream) {
  if (n <= 0 || !in || !out) return ufail(UNET_EINVAL, "bad args");
  hipLaunchKernelGGL(k_to_bf16, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, (long long)n, in,
                     (uint16_t*)out);
  UHIP(hipGetLastError());
  return UNET_OK;
}

unet_status unet_from_bf16(int64_t n, const void* in, float* out, void* stream) {
  if (n <= 0 || !in || !out) return ufail(UNET_EINVAL, "bad args");
  hipLaunchKernelGGL(k_from_bf16, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, (long long)n,
                     (const uint16_t*)in, out);
  UHIP(hipGetLastError());
  return UNET_OK;
}

unet_status unet_pack_input(unet_shape s, const float* sigma, const float* L, const float* scale,
                            void* x, void* stream) {
  if (!shape_ok(s) || !sigma || !L || !scale || !x || s.n > 64)
    return ufail(UNET_EINVAL, "bad pack args (at most 64 samples)");
  Scales sc;
  for (int k = 0; k < s.n; ++k) sc.s[k] = scale[k] > 0.f ? scale[k] : 1.f;
  const long long nvs = (long long)s.d * s.h * s.w;
  hipLaunchKernelGGL(k_pack_input, dim3(nblk(nvs * s.n)), dim3(256), 0, (hipStream_t)stream, nvs,
                     s.n, sigma, L, sc, (uint16_t*)x);
  UHIP(hipGetLastError());
  return UNET_OK;
}

}  // extern "C"
