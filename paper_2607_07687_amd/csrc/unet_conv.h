// The 3x3x3 convolution (forward, and the data gradient on flipped weights):
// an implicit GEMM on bricks of voxels staged in LDS.
#pragma once

#include "unet_device.h"

namespace unet {

struct ConvArgs {
  unet_shape s;
  const uint16_t* x;
  int xld, xoff, cin;
  const uint16_t* w;  // [cout][27][cin]
  const float* bias;  // may be NULL
  uint16_t* y;
  int yld, yoff;
  float* yf;  // FP32 output instead of y when not NULL
  int relu;
  int nbw, nbh, nbd;  // bricks along w, h, d
  int groups;         // output-channel groups (workgroups that share a brick's input)
  int total;          // work items: bricks x groups
  int wide;           // y (or yf) takes 16-byte (NB = 1: 8-byte) stores
  const uint16_t* gate;  // y is cleared where this is not positive (GATE kernels)
  int gld, goff;
};

// Waves per SIMD that `regs` registers and about 50 more leave room for.
constexpr int brick_waves(int regs, int threads) {
  const int w = 512 / (regs + 50);
  const int most = w > 4 ? 4 : w, least = threads / 256;
  return most < least ? least : (most < 1 ? 1 : most);
}

// Compile-time shape of a brick kernel.  A workgroup computes bricks of
// 16 x MB x WD voxels (w, h, d) for WC x NB blocks of 16 output channels: per
// pass it stages the brick's input neighbourhood (one voxel more on every
// side, zeros outside the grid) of a chunk of CK channels in LDS and reads
// all 27 taps from there; with all NC chunks of 64 or 128 channels at once, a
// pass is one tap plane kd.  Wave (wd, wc) holds the MB rows of plane wd times
// NB output blocks.
//
// Every output sums K = (tap, channel) in that order in steps of 32 (with 8,
// 16, 32, 64 or 128 input channels; chunk by chunk otherwise) whatever the
// shape, as the gathered kernel does: the choice of a kernel does not change a
// bit of the result.  Orders that read LDS less (rows shared by the three kh,
// K split over waves) were no faster than this one once its reads were free of
// bank conflicts.
//
// What bounds it: with 16 and 32 channels neither memory (32 -> 16 channels at
// 2 x 128^3: 402 MB in 150 us, 2.7 TB/s) nor the matrix cores (116 GFLOP, 770
// TFLOP/s) but the latency of a brick's phases, two bricks of a CU overlapping
// each other; with 64 and 128 channels the matrix cores' issue (128 -> 64 on 2 x
// 32^3: 34 us, 855 TFLOP/s).  Before (a tile of one plane per workgroup, or
// operands gathered from global memory): 346 us and 143 us.
template <int CK_, int NC_, int MB_, int NB_, int WD_, int WC_>
struct Brick {
  static constexpr int CK = CK_, NC = NC_, MB = MB_, NB = NB_, WD = WD_, WC = WC_;
  static_assert(CK == 8 || CK == 16 || CK == 32, "channels per chunk");
  static_assert(NC == 1 || CK == 32, "several chunks of 32 channels");
  static constexpr int NT = 64 * WD * WC;
  // several chunks: a pass stages the WD input planes of one tap plane kd only
  // (with all three, two and four chunks leave room for one workgroup per CU)
  static constexpr bool KP = NC > 1;
  static constexpr int SW = 18, SH = MB + 2, SD = KP ? WD : WD + 2, SLOTS = SW * SH * SD;
  static constexpr int P8 = CK / 8, Q8 = NC * P8;  // 16-byte pieces per voxel: of a chunk, staged
  static constexpr int SPI = NT / Q8;              // slots staged per step of the workgroup
  static constexpr int NIT = (SLOTS + SPI - 1) / SPI;
  // K steps: one chunk of 32 channels of a tap, or two taps of 16 or four of 8
  // channels (a tap past the 27th counts as zero weights on zero inputs)
  static constexpr int STEPS = KP ? 9 * NC : (27 * CK + 31) / 32;  // per pass
  // steps of weights in flight: more where a step is short
  static constexpr int AHEAD = MB * NB <= 4 ? 8 : 3;
  static constexpr int REGS = 4 * (MB * NB + NIT + 2 * MB + (AHEAD + 1) * NB);
  static constexpr int LDS = NC * SLOTS * P8;
  static constexpr int WAVES = brick_waves(REGS, NT);
  // workgroups of a CU that run at once
  static constexpr int PER_CU = 160 * 1024 / (LDS * 16) < WAVES * 4 / (NT / 64)
                                    ? 160 * 1024 / (LDS * 16)
                                    : WAVES * 4 / (NT / 64);
};

// The workgroups are persistent: each takes every S-th work item of its
// XCD's contiguous range (S workgroups per XCD), so that neighbouring bricks
// run at the same time behind one L2, and loads the next item's (or pass's)
// neighbourhood into registers while it computes the current one.
//
// MFMA operands: A = weights (m = output channel), B = voxels (n).  The
// weight row of m is chosen so that a lane ends up with 4 NB consecutive
// channels of one voxel: 8- or 16-byte stores.
//
// LDS: the 16 lanes of a quarter wave read one 16-byte piece each of
// consecutive voxels.  The pieces of a voxel are permuted by its column (swz):
// a wave's read then takes 4.4 cycles (8.1 without, or permuted by col >> 2).
// GATE: the output is the gradient of a ReLU's output and is cleared where that
// (a.gate) is not positive; a variant of its own, since the test alone costs a
// forward convolution 4%.
template <int CK, int NC, int MB, int NB, int WD, int WC, bool GATE>
__global__ __launch_bounds__(64 * WD * WC)
    __attribute__((amdgpu_waves_per_eu(Brick<CK, NC, MB, NB, WD, WC>::WAVES))) void
    k_conv_brick(ConvArgs a) {
  using B = Brick<CK, NC, MB, NB, WD, WC>;
  constexpr int SW = B::SW, SH = B::SH, SD = B::SD, P8 = B::P8, Q8 = B::Q8, NIT = B::NIT;
  __shared__ uint4 tile[B::LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wd = wave % WD, wc = wave / WD;
  const int W = a.s.w, H = a.s.h, D = a.s.d;
  const int K = 27 * a.cin;
  const int l16 = lane & 15, g = lane >> 4;
  const long long plane = (long long)H * W;

  // position permutation of a voxel's pieces
  auto swz = [](int col) { return CK == 32 ? (col >> 1) & 3 : (CK == 16 ? (col >> 2) & 1 : 0); };

  // a work item: its brick's origin and the wave's first output channel
  struct Item {
    int w0, h0, d0, n0, co0;
  };
  auto item = [&](int b) {
    Item t;
    t.co0 = ((b % a.groups) * WC + wc) * (16 * NB);
    b /= a.groups;
    t.w0 = (b % a.nbw) * 16;
    b /= a.nbw;
    t.h0 = (b % a.nbh) * MB;
    b /= a.nbh;
    t.d0 = (b % a.nbd) * WD;
    t.n0 = b / a.nbd;
    return t;
  };

  // Staging: a thread keeps one piece of the slots it stages, SPI apart.  Raw
  // buffer loads from the plane below the brick: an offset at or past the
  // descriptor's size reads zero and touches no memory, which gives the zeros
  // outside the grid (the host keeps SD planes below 2^31 bytes).
  constexpr int kOut = 0x7FFFFFF0;
  constexpr int SPI = B::SPI;
  const int sp = tid % Q8, s0 = tid / Q8;
  const int rw = W * a.xld * 2, pl = H * rw, vx = a.xld * 2;
  uint4 v[NIT];
  const int passes = B::KP ? 3 : a.cin / CK;
  auto fetch = [&](const Item& t, int ps) {
    const int dlow = t.d0 - 1 + (B::KP ? ps : 0), c0 = B::KP ? 0 : ps * CK;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.x + (((long long)t.n0 * D + dlow) * plane) * a.xld + a.xoff), 0, kOut, 0x00020000);
    int col = s0 % SW, row = (s0 / SW) % SH, sd = s0 / (SW * SH);
    int off = sd * pl + (t.h0 - 1 + row) * rw + (t.w0 - 1 + col) * vx + sp * 16;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const bool in = (unsigned)(dlow + sd) < (unsigned)D &&
                      (unsigned)(t.h0 - 1 + row) < (unsigned)H &&
                      (unsigned)(t.w0 - 1 + col) < (unsigned)W &&
                      ((it + 1) * SPI <= B::SLOTS || sd < SD);
      v[it] = __builtin_bit_cast(
          uint4, __builtin_amdgcn_raw_buffer_load_b128(xr, in ? off : kOut, 2 * c0, 0));
      constexpr int DC = SPI % SW, DR = (SPI / SW) % SH, DD = SPI / (SW * SH);
      col += DC;
      row += DR;
      sd += DD;
      off += DC * vx + DR * rw + DD * pl;
      if (DC) {
        const bool up = col >= SW;
        col = up ? col - SW : col;
        row += up ? 1 : 0;
        off += up ? rw - SW * vx : 0;
      }
      const bool up = row >= SH;
      row = up ? row - SH : row;
      sd += up ? 1 : 0;
      off += up ? pl - SH * rw : 0;
    }
  };
  auto park = [&]() {
    const int ch = sp / P8, pc = sp % P8;
    int slot = s0, col = s0 % SW;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      if ((it + 1) * SPI <= B::SLOTS || slot < B::SLOTS)
        tile[(ch * B::SLOTS + slot) * P8 + (pc ^ swz(col))] = v[it];
      slot += SPI;
      col += SPI % SW;
      col = col >= SW ? col - SW : col;
    }
  };

  // the lane's tap of a step (two taps of 16 or four of 8 channels share a
  // step) and its piece of the chunk
  const int wtap = CK == 32 ? 0 : g / P8;
  const int wpc = CK == 32 ? g : g % P8;
  // byte offset of the lane's piece of weight row m of block 0
  const int wlane = (((l16 >> 2) * 4 * NB + (l16 & 3)) * K + wpc * 8) * 2;
  auto ldv = [&](int i) { return *reinterpret_cast<const bf16x8*>(&tile[i]); };
  constexpr int RS = SW * P8, PS = SH * SW * P8;  // row and plane strides
  // the lane's piece of its voxel of row 0 at each tap column (CK = 32) or step
  int ad[CK == 32 ? 3 : B::STEPS];
#pragma unroll
  for (int q = 0; q < (CK == 32 ? 3 : B::STEPS); ++q) {
    const int t = CK == 32 ? q : min(32 / CK * q + wtap, 26), kw = t % 3;
    ad[q] = (wd + t / 9) * PS + (t / 3 % 3) * RS + (l16 + kw) * P8 + (wpc ^ swz(l16 + kw));
  }

  f32x4 acc[MB][NB];
  auto clear = [&]() {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  };

  auto store = [&](const Item& t) {
    const int c = t.co0 + 4 * NB * g;  // the lane's first channel
    float bias[NB * 4];
#pragma unroll
    for (int r = 0; r < NB * 4; ++r) bias[r] = a.bias ? a.bias[c + r] : 0.f;
    const int wv = t.w0 + l16, dd = t.d0 + wd;
    if (dd >= D || wv >= W) return;
    const long long vx0 = ((long long)t.n0 * D + dd) * plane + (long long)t.h0 * W + wv;
    long long o = vx0 * a.yld + a.yoff + c;
    uint32_t gt[GATE ? MB : 1][NB * 2];
    if constexpr (GATE) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        if (t.h0 + mb >= H) continue;
        const uint16_t* gp = a.gate + (vx0 + (long long)mb * W) * a.gld + a.goff + c;
        if (a.wide) {
          if constexpr (NB == 1) {
            const uint2 q = *reinterpret_cast<const uint2*>(gp);
            gt[mb][0] = q.x, gt[mb][1] = q.y;
          } else {
            const uint4 q = *reinterpret_cast<const uint4*>(gp);
            gt[mb][0] = q.x, gt[mb][1] = q.y, gt[mb][2] = q.z, gt[mb][3] = q.w;
          }
        } else {
          for (int r = 0; r < NB * 2; ++r) gt[mb][r] = gp[2 * r] | (uint32_t)gp[2 * r + 1] << 16;
        }
      }
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb, o += (long long)W * a.yld) {
      if (t.h0 + mb >= H) continue;
      float u[NB * 4];
#pragma unroll
      for (int r = 0; r < NB * 4; ++r) {
        const float s = acc[mb][r / 4][r % 4] + bias[r];
        u[r] = a.relu ? fmaxf(s, 0.f) : s;
      }
      if (a.yf) {
        if (a.wide)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            *reinterpret_cast<float4*>(a.yf + o + nb * 4) =
                make_float4(u[nb * 4], u[nb * 4 + 1], u[nb * 4 + 2], u[nb * 4 + 3]);
        else
          for (int r = 0; r < 4 * NB; ++r) a.yf[o + r] = u[r];
        continue;
      }
      uint32_t h[NB * 2];
#pragma unroll
      for (int r = 0; r < NB * 2; ++r)
        h[r] = (uint32_t)f2bf(u[2 * r]) | ((uint32_t)f2bf(u[2 * r + 1]) << 16);
      if constexpr (GATE)
#pragma unroll
        for (int r = 0; r < NB * 2; ++r) h[r] = gate2(h[r], gt[mb][r]);
      if (a.wide) {
        if constexpr (NB == 1)
          *reinterpret_cast<uint2*>(a.y + o) = make_uint2(h[0], h[1]);
        else
          *reinterpret_cast<uint4*>(a.y + o) = make_uint4(h[0], h[1], h[2], h[3]);
      } else {
        for (int r = 0; r < NB * 2; ++r) {
          a.y[o + 2 * r] = (uint16_t)h[r];
          a.y[o + 2 * r + 1] = (uint16_t)(h[r] >> 16);
        }
      }
    }
  };

  // the workgroup's items: S apart in its XCD's range
  const int q8 = a.total / 8, r8 = a.total % 8, xcd = blockIdx.x % 8, S = (gridDim.x + 7 - xcd) / 8;
  const int end = (xcd + 1) * q8 + min(xcd + 1, r8);
  int b = xcd * q8 + min(xcd, r8) + blockIdx.x / 8;
  if (b >= end) return;
  Item cur = item(b);
  int ps = 0;
  fetch(cur, 0);
  clear();
  while (true) {
    // weights through buffer loads too: a lane offset fixed for the kernel and
    // a scalar one per step, so that no address arithmetic runs per load
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.w + (long long)cur.co0 * K + (B::KP ? ps * 9 * a.cin : ps * CK)), 0, kOut,
        0x00020000);
    constexpr int TPS = 32 / CK, STEPS = B::STEPS, AH = B::AHEAD;
    bf16x8 wq[AH + 1][NB], vq[2][MB];
    auto load_w = [&](int s, bf16x8 (&o)[NB]) {
      const int t0 = CK == 32 ? s / NC : TPS * s;  // the step's first tap
      const bool end_ = CK < 32 && t0 + TPS > 27;
      const int over = end_ ? max(t0 + wtap - 26, 0) : 0;
      const int off = wlane + 2 * (wtap - over) * a.cin;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const bf16x8 r = __builtin_bit_cast(
            bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                        wr, off, 2 * (t0 * a.cin + (s % NC) * 32 + nb * 4 * K), 0));
        o[nb] = end_ && over > 0 ? zero8() : r;
      }
    };
#pragma unroll
    for (int s = 0; s < AH; ++s) load_w(s, wq[s]);
    // park what was fetched, then fetch the next pass or item
    const bool last = ps + 1 == passes;
    const int bn = last ? b + S : b, pn = last ? 0 : ps + 1;
    const bool more = bn < end;
    Item nxt = cur;
    park();
    __syncthreads();
    if (last && more) nxt = item(bn);
    if (more) fetch(nxt, pn);
    auto load_v = [&](int s, bf16x8 (&o)[MB]) {
      int q;
      bool none = false;
      if constexpr (CK == 32) {
        const int t = s / NC;
        q = ad[t % 3] + ((s % NC) * SD + t / 9) * PS + (t / 3 % 3) * RS;
      } else {
        q = ad[s];
        none = TPS * (s + 1) > 27 && TPS * s + wtap > 26;
      }
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const bf16x8 r = ldv(q + mb * RS);
        o[mb] = none ? zero8() : r;
      }
    };
    load_v(0, vq[0]);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (s + AH < STEPS) load_w(s + AH, wq[(s + AH) % (AH + 1)]);
      if (s + 1 < STEPS) load_v(s + 1, vq[(s + 1) & 1]);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wq[s % (AH + 1)][nb], vq[s & 1][mb],
                                                                acc[mb][nb], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);  // later steps' loads stay where they are issued
    }
    if (last) {
      store(cur);
      clear();
    }
    if (!more) return;
    __syncthreads();
    b = bn;
    ps = pn;
    cur = nxt;
  }
}

}  // namespace unet
