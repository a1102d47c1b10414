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
  int q, r;           // output planes of a marching workgroup's share: q, one more for the first r
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
// What bounds it: with 16 and 32 channels the latency of a brick's phases, two
// bricks of a CU overlapping each other (grids with planes enough take the marching
// kernel below); with 64 and 128 channels the matrix cores' issue (128 -> 64 on 2 x
// 32^3: 34 us, 855 TFLOP/s).  Before (operands gathered from global memory): 143 us.
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

// What the store of a wave's output rows reads besides the sums.  Loaded
// before the next input's loads are issued: loads return in order, so that a
// load after those would wait for all of them.  (Data gradients, which come with
// the gates, have no bias.)
template <int MB, int NB, bool GATE>
struct StoreIn {
  float bias[NB * 4];
  uint32_t gate[GATE ? MB : 1][NB * 2];
};

// (of the lane's 4 NB channels from c)
template <int MB, int NB, bool GATE>
__device__ __forceinline__ void load_bias(const ConvArgs& a, int c, StoreIn<MB, NB, GATE>& in) {
#pragma unroll
  for (int r = 0; r < NB * 4; ++r) in.bias[r] = !GATE && a.bias ? a.bias[c + r] : 0.f;
}

// (of MB rows of 16 voxels from row h0 of plane d, the lane's voxel at w)
template <int MB, int NB, bool GATE>
__device__ __forceinline__ void load_gate(const ConvArgs& a, int n, int d, int h0, int w, int c,
                                          StoreIn<MB, NB, GATE>& in) {
  if constexpr (GATE) {
    const int W = a.s.w, H = a.s.h;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      if (d >= a.s.d || w >= W || h0 + mb >= H) continue;
      const uint16_t* gp =
          a.gate + ((((long long)n * a.s.d + d) * H + h0 + mb) * W + w) * a.gld + a.goff + c;
      if (a.wide) {
        if constexpr (NB == 1) {
          const uint2 q = *reinterpret_cast<const uint2*>(gp);
          in.gate[mb][0] = q.x, in.gate[mb][1] = q.y;
        } else {
          const uint4 q = *reinterpret_cast<const uint4*>(gp);
          in.gate[mb][0] = q.x, in.gate[mb][1] = q.y, in.gate[mb][2] = q.z, in.gate[mb][3] = q.w;
        }
      } else {
        for (int r = 0; r < NB * 2; ++r)
          in.gate[mb][r] = gp[2 * r] | (uint32_t)gp[2 * r + 1] << 16;
      }
    }
  }
}

// A wave's rows: bias, ReLU, gate, conversion, store.
template <int MB, int NB, bool GATE>
__device__ __forceinline__ void store_rows(const ConvArgs& a, const f32x4 (&acc)[MB][NB], int n,
                                           int d, int h0, int w, int c,
                                           const StoreIn<MB, NB, GATE>& in) {
  const int W = a.s.w, H = a.s.h;
  if (d >= a.s.d || w >= W) return;
  long long o = ((((long long)n * a.s.d + d) * H + h0) * W + w) * a.yld + a.yoff + c;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb, o += (long long)W * a.yld) {
    if (h0 + mb >= H) continue;
    float u[NB * 4];
#pragma unroll
    for (int r = 0; r < NB * 4; ++r) {
      const float s = acc[mb][r / 4][r % 4] + in.bias[r];
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
      for (int r = 0; r < NB * 2; ++r) h[r] = gate2(h[r], in.gate[mb][r]);
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
}

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
  // outside the grid (the host keeps SD planes below 2^31 bytes; unsigned, as the
  // offsets of slots outside the grid may wrap).
  constexpr int kOut = 0x7FFFFFF0;
  constexpr int SPI = B::SPI;
  const int sp = tid % Q8, s0 = tid / Q8;
  const unsigned rw = W * a.xld * 2, pl = H * rw, vx = a.xld * 2;
  uint4 v[NIT];
  const int passes = B::KP ? 3 : a.cin / CK;
  auto fetch = [&](const Item& t, int ps) {
    const int dlow = t.d0 - 1 + (B::KP ? ps : 0), c0 = B::KP ? 0 : ps * CK;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.x + (((long long)t.n0 * D + dlow) * plane) * a.xld + a.xoff), 0, kOut, 0x00020000);
    int col = s0 % SW, row = (s0 / SW) % SH, sd = s0 / (SW * SH);
    unsigned off = sd * pl + (t.h0 - 1 + row) * rw + (t.w0 - 1 + col) * vx + sp * 16;
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

  StoreIn<MB, NB, GATE> in;
  auto load_in = [&](const Item& t) {
    const int c = t.co0 + 4 * NB * g;  // the lane's first channel
    load_bias(a, c, in);
    load_gate(a, t.n0, t.d0 + wd, t.h0, t.w0 + l16, c, in);
  };
  auto store = [&](const Item& t) {
    store_rows(a, acc, t.n0, t.d0 + wd, t.h0, t.w0 + l16, t.co0 + 4 * NB * g, in);
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
    if (last) load_in(cur);
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

// Compile-time shape of a marching kernel, for the layers of few channels on
// large grids.  A workgroup walks down d on a tile of 16 WW x MB WH voxels: a
// step stages one input plane (fetched while the step before computes) in a ring
// of four and computes the output plane below it, each wave MB rows of 16 voxels
// for all of the workgroup's 16 NB output channels.  A brick stages 2.1 voxels
// for each of its own and every wave streams the weights from the caches; here
// it is 1.2 to 1.4, and a wave holds all its weights in registers.  The sums are
// the brick's, bitwise.
//
// What bounds it: with one block of outputs memory (16 -> 16 channels on 2 x 128^3:
// 268 MB in 72 us, 3.7 TB/s; 8 -> 16 201 MB in 49 us, 4.1), with 32 channels on
// either side the steps' phases (32 -> 16: 116 GFLOP in 131 us, 890 TFLOP/s; 16 ->
// 32 in 135).  Bricks: 91, 61, 158 and 166 us.
template <int CK_, int NB_, int MB_, int WW_, int WH_>
struct March {
  static constexpr int CK = CK_, NB = NB_, MB = MB_, WW = WW_, WH = WH_;
  static_assert(CK == 8 || CK == 16 || CK == 32, "input channels");
  static constexpr int NT = 64 * WW * WH, PER_CU = 512 / NT;
  static constexpr int SW = 16 * WW + 2, SH = MB * WH + 2, SLOTS = SW * SH;
  static constexpr int P8 = CK / 8, TPS = 32 / CK, STEPS = (27 + TPS - 1) / TPS;
  static constexpr int NIT = (SLOTS * P8 + NT - 1) / NT;
  static constexpr int PB = NIT * NT;  // 16-byte pieces of a plane's buffer
  static_assert(PER_CU * 4 * PB * 16 <= 160 * 1024, "four planes in LDS");
};

// FAR: planes of 2^31 bytes and more, whose offsets count from the row below the
// tile (a variant of its own: the plane's start as base is 0.5% faster).
template <int CK, int NB, int MB, int WW, int WH, bool GATE, bool FAR>
__global__ __launch_bounds__(64 * WW * WH, 2) void k_conv_march(ConvArgs a) {
  using B = March<CK, NB, MB, WW, WH>;
  constexpr int NT = B::NT, SW = B::SW, P8 = B::P8, TPS = B::TPS, STEPS = B::STEPS, NIT = B::NIT,
                PB = B::PB, RS = SW * P8;
  __shared__ uint4 ring[4 * PB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ww = wave % WW, wh = wave / WW;
  const int W = a.s.w, H = a.s.h, D = a.s.d;
  const int K = 27 * a.cin;
  const int l16 = lane & 15, g = lane >> 4;
  const int co0 = blockIdx.y * 16 * NB;
  auto swz = [](int col) { return CK == 32 ? (col >> 1) & 3 : (CK == 16 ? (col >> 2) & 1 : 0); };

  // the workgroup's share of all tiles' output planes
  const int nchunk = gridDim.x;
  int chunk = blockIdx.x;  // shares in order within an XCD (block b runs on XCD b % 8)
  if ((nchunk & 7) == 0) chunk = (blockIdx.x & 7) * (nchunk >> 3) + (blockIdx.x >> 3);
  const int t0 = a.q * chunk + min(chunk, a.r), t1 = t0 + a.q + (chunk < a.r ? 1 : 0);
  if (t0 >= t1) return;

  // weights as the brick kernel's A operands, for the whole launch
  const int wtap = CK == 32 ? 0 : g / P8, wpc = CK == 32 ? g : g % P8;
  bf16x8 wq[STEPS][NB];
  {
    const int row = co0 + (l16 >> 2) * 4 * NB + (l16 & 3);
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int t = TPS * s + wtap;
        wq[s][nb] = t < 27 ? ld8(a.w + (long long)(row + 4 * nb) * K + t * a.cin + wpc * 8) : zero8();
      }
  }
  // the lane's piece of its voxel of the wave's first row at each tap column
  // (CK = 32) or step, within a plane
  int ad[CK == 32 ? 3 : STEPS];
#pragma unroll
  for (int q = 0; q < (CK == 32 ? 3 : STEPS); ++q) {
    const int t = CK == 32 ? q : min(TPS * q + wtap, 26), kw = t % 3, col = 16 * ww + l16 + kw;
    ad[q] = (wh * MB + (CK == 32 ? 0 : t / 3 % 3)) * RS + col * P8 + (wpc ^ swz(col));
  }

  // staging: thread t takes pieces t, t + NT, ... of a plane's buffer
  constexpr int kOut = 0x7FFFFFF0;
  int xo[NIT];
  uint4 v[2][NIT];
  struct Step {
    int n, w0, h0, p;  // input plane p
    int of, ol;        // output planes of the segment
  };
  auto segment = [&](int t) {
    Step s;
    int tile = t / D;
    s.of = t - tile * D;
    s.ol = min(D, s.of + (t1 - t)) - 1;
    s.p = s.of - 1;
    s.w0 = tile % a.nbw * (16 * WW);
    tile /= a.nbw;
    s.h0 = tile % a.nbh * (MB * WH);
    s.n = tile / a.nbh;
#pragma unroll
    for (int i = 0; i < NIT; ++i) {
      const int e = tid + i * NT, slot = e / P8, row = slot / SW, col = slot % SW;
      const int h = s.h0 - 1 + row, w = s.w0 - 1 + col;
      xo[i] = slot < B::SLOTS && (unsigned)h < (unsigned)H && (unsigned)w < (unsigned)W
                  ? (((FAR ? row : h) * W + w) * a.xld + ((e % P8) ^ swz(col)) * 8) * 2
                  : kOut;
    }
    return s;
  };
  const long long plane = (long long)H * W;
  auto fetch = [&](const Step& s, uint4 (&v)[NIT]) {
    const long long below = FAR ? (s.h0 - 1LL) * W : 0;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.x + (((long long)s.n * D + s.p) * plane + below) * a.xld + a.xoff), 0,
        (unsigned)s.p < (unsigned)D ? kOut : 0, 0x00020000);
#pragma unroll
    for (int i = 0; i < NIT; ++i)
      v[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xr, xo[i], 0, 0));
  };
  auto park = [&](int k, const uint4 (&v)[NIT]) {
#pragma unroll
    for (int i = 0; i < NIT; ++i) ring[(k & 3) * PB + tid + i * NT] = v[i];
  };

  // the plane after f in the share (false: none left)
  int t = t0;
  auto advance = [&](Step& f) {
    if (f.p <= f.ol) {
      ++f.p;
      return true;
    }
    t += f.ol - f.of + 1;
    if (t >= t1) return false;
    f = segment(t);
    return true;
  };
  StoreIn<MB, NB, GATE> in;
  load_bias(a, co0 + 4 * NB * g, in);
  auto compute = [&](const Step& s, int k) {
    if (s.p > s.of) {  // planes p - 2, p - 1, p of the segment are staged
      int pb[3];
#pragma unroll
      for (int kd = 0; kd < 3; ++kd) pb[kd] = ((k - 2 + kd) & 3) * PB;
      f32x4 acc[MB][NB];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
      bf16x8 vq[2][MB];
      auto load_v = [&](int st, bf16x8 (&o)[MB]) {
        int q;
        bool none = false;
        if constexpr (CK == 32) {
          q = ad[st % 3] + pb[st / 9] + (st / 3 % 3) * RS;
        } else {
          const int first = TPS * st / 9, last = min(TPS * st + TPS - 1, 26) / 9;
          // a step's taps may lie on two planes
          q = ad[st] + (first == last || TPS * st + wtap < 9 * last ? pb[first] : pb[last]);
          none = TPS * (st + 1) > 27 && TPS * st + wtap > 26;
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          const bf16x8 r = *reinterpret_cast<const bf16x8*>(&ring[q + mb * RS]);
          o[mb] = none ? zero8() : r;
        }
      };
      load_v(0, vq[0]);
#pragma unroll
      for (int st = 0; st < STEPS; ++st) {
        if (st + 1 < STEPS) load_v(st + 1, vq[(st + 1) & 1]);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wq[st][nb], vq[st & 1][mb],
                                                                  acc[mb][nb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);  // the next step's reads stay where they are issued
      }
      store_rows(a, acc, s.n, s.p - 1, s.h0 + wh * MB, s.w0 + 16 * ww + l16, co0 + 4 * NB * g, in);
    }
  };

  // loads run two steps ahead: plane k + 2 is fetched while k computes
  Step s = segment(t), f = s;
  fetch(f, v[0]);
  Step nx = f;
  bool more = advance(f);
  if (more) {
    nx = f;
    fetch(f, v[1]);
  }
  park(0, v[0]);
  __syncthreads();
  bool ahead = more;  // f is the step after nx's
  auto turn = [&](int k, uint4 (&v0)[NIT], const uint4 (&v1)[NIT]) {
    if (ahead) ahead = advance(f);
    if (s.p > s.of)
      load_gate(a, s.n, s.p - 1, s.h0 + wh * MB, s.w0 + 16 * ww + l16, co0 + 4 * NB * g, in);
    if (ahead) fetch(f, v0);
    compute(s, k);
    if (!more) return false;
    park(k + 1, v1);
    __syncthreads();
    s = nx;
    nx = f;
    more = ahead;
    return true;
  };
  for (int k = 0; turn(k, v[0], v[1]) && turn(k + 1, v[1], v[0]); k += 2) {
  }
}

}  // namespace unet
