// Weight and bias gradients of the 3x3x3 convolution: a contraction over
// voxels of dy (output channels) with x shifted by every tap.
#pragma once

#include <type_traits>

#include "unet_device.h"

namespace unet {

struct WgradArgs {
  unet_shape s;
  const uint16_t* x;
  int xld, xoff, cin;
  const uint16_t* dy;
  int dld, doff, cout;
  int ltwo;            // tile: 2^ltwo octets of voxels along w
  int nbw, nbh;        // tiles along w, h
  int ncp;             // input-channel parts
  int q, r;            // dy planes (of all tiles) of a share: q, one more for the first r
  long long rs;        // ws row stride (floats)
  float* ws;
};

typedef short short4v __attribute__((ext_vector_type(4)));
using LdsBytes = __attribute__((address_space(3))) char*;

// Compile-time shape of a weight-gradient kernel: CT input and OT output
// channels per workgroup, in P blocks of 16 x 16; a wave holds one block's 27
// taps and takes four octets (8 voxels of a row) at a time, one per 16 lanes,
// down a chain of RL rows.  A tile is NOC octets: two of them along w (1 to 8), the
// chains along h.
//
// The MFMA's K runs over voxels, so that a lane wants 8 voxels of one channel
// where memory holds the channels of a voxel together: the tiles stay as they
// are in memory and LDS transposes while it reads (ds_read_b64_tr_b16).  Every
// fragment of x, of which a (plane, row) has three for the w taps, meets the
// dy fragments of three planes and three rows, kept in registers while the
// wave walks down its rows: six fragment reads for 27 MFMAs.
//
// What bounds it: with 16 input channels memory (16 -> 16 on 2 x 128^3: 268 MB
// in 64 us, 4.2 TB/s), with 32 and more the steps' starts and ends (32 -> 32 on 2
// x 64^3: 29 GFLOP in 36 us, 810 TFLOP/s, matrix cores busy 43% of it: 16 planes
// a share, the first and last two of them partial).  Before (4-row tiles
// transposed in registers on their way to LDS): 124 and 72 us; 32 -> 16 on 2 x
// 128^3 181 -> 110, 128 -> 64 on 2 x 32^3 72 -> 36.  Eight waves on one tile of
// 16 rows were better than twice four on 12 for 16 channels (64 and 78 us), twice
// four for 32 (36 and 44 us).
template <int CT_, int OT_, int RL_, int NT_>
struct Wgrad {
  static constexpr int CT = CT_, OT = OT_, RL = RL_, NT = NT_;
  static_assert(CT == 8 || CT == 16 || CT == 32, "input channels of a workgroup");
  static_assert(OT == 16 || OT == 32, "output channels of a workgroup");
  static constexpr int WAVES = NT / 64, PER_CU = 512 / NT;
  static constexpr int NCB = CT < 16 ? 1 : CT / 16, P = OT / 16 * NCB;
  static constexpr int KW = WAVES / P, NOC = 4 * KW;
  // x fragments of a row: one per w tap, or of 8 channels one per pair of taps
  static constexpr int NF = CT == 8 ? 2 : 3, NACC = 9 * NF;
  static constexpr int XQ = CT / 8, DQ = OT / 8;  // 16-byte pieces of a voxel
  // staged columns of a row: the octets and one voxel on either side; a single
  // octet's permuted slots (swizzle below) reach the 14th
  __host__ __device__ static constexpr int cols(int two) {
    return CT == 16 && two == 1 ? 14 : 8 * two + 2;
  }
  __host__ __device__ static constexpr int xslots(int two) {
    return (NOC / two * RL + 2) * cols(two);
  }
  static constexpr int most(int a, int b) { return a > b ? a : b; }
  // octets along w of a tile (a power of two): the widest and narrowest
  static constexpr int TWO_HI = NOC > 8 ? 8 : 4, TWO_LO = NOC > 8 ? 2 : 1;
  static constexpr int XS =
      most(most(xslots(TWO_HI), xslots(4)), most(xslots(2), xslots(TWO_LO))) + (CT == 8 ? 1 : 0);
  static constexpr int DS = NOC * 8 * RL;
  static constexpr int NIX = (XS * XQ + NT - 1) / NT, NID = DS * DQ / NT;
  static constexpr int XB = NIX * NT * 16, DB = DS * DQ * 16;  // bytes of one plane's buffer
  static constexpr int LDS = 2 * XB + 4 * DB;
  static_assert(PER_CU * LDS <= 160 * 1024, "two planes of x and four of dy");
  static_assert(WAVES * 9 * 4 * 64 * 4 <= LDS, "nine taps' sums of all waves fit in LDS");
};

// A workgroup walks plane by plane through its share of all tiles' planes
// (adjacent shares on one XCD).  Step k stages one plane of x and the dy plane
// above it, fetched while step k - 1 computes; dy planes stay for two more
// steps.  The shares' sums go to ws, one row per share; k_sum_* add the rows
// in order.
// FAR: planes of 2^31 bytes and more, whose offsets count from the tile's first
// rows.
template <int CT, int OT, int RL, int NT, bool FAR>
__global__ __launch_bounds__(NT, 2) void k_wgrad(WgradArgs a) {
  using K = Wgrad<CT, OT, RL, NT>;
  constexpr int XQ = K::XQ, DQ = K::DQ, NF = K::NF, P = K::P, KW = K::KW;
  __shared__ __align__(16) char lds[K::LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.s.d, H = a.s.h, W = a.s.w;
  const int two = 1 << a.ltwo, TW = 8 * two, cols = K::cols(two), rows = (K::NOC >> a.ltwo) * RL;
  const int c0 = (blockIdx.y % a.ncp) * CT, o0 = (blockIdx.y / a.ncp) * OT;
  const int nchunk = gridDim.x;
  int chunk = blockIdx.x;  // shares in order within an XCD (block b runs on XCD b % 8)
  if ((nchunk & 7) == 0) chunk = (blockIdx.x & 7) * (nchunk >> 3) + (blockIdx.x >> 3);
  const int t0 = a.q * chunk + min(chunk, a.r), t1 = t0 + a.q + (chunk < a.r ? 1 : 0);

  // Voxels of 32 bytes swap halves of an odd octet, those of 64 bytes swap
  // pieces there: four octets' rows then meet in all of the 64 banks.
  auto slot16 = [](int col) { return col ^ ((col >> 1) & 4); };
  auto swz32 = [](int col) { return (col >> 2) & 2; };

  // lane's addresses of the first row: transposing reads of 4 voxels x 16
  // channels by 16 lanes, lane l taking 8 bytes of voxel l / 4
  const int l16 = lane & 15, g = lane >> 4, lv = l16 >> 2, lb = (l16 & 3) * 8;
  const int cblk = wave % P, oc = wave / P * 4 + g;
  const int ob = cblk / K::NCB, cb = cblk % K::NCB;
  const int ow = oc & (two - 1), oh = oc >> a.ltwo;
  int xa[NF][2], da[2];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int col = 8 * ow + lv + 4 * h + (CT == 8 ? 2 * f : f), row = oh * RL;
      xa[f][h] = CT == 8    ? (row * cols + col) * 16 + lb
                 : CT == 16 ? (row * cols + slot16(col)) * 32 + lb
                            : (row * cols + col) * 64 + ((cb * 2) ^ swz32(col)) * 16 + lb;
    }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int col = 8 * ow + lv + 4 * h, row = oh * RL;
    da[h] = OT == 16 ? (row * TW + slot16(col)) * 32 + lb
                     : (row * TW + col) * 64 + ((ob * 2) ^ swz32(col)) * 16 + lb;
  }
  const int xrow = cols * CT * 2, drow = TW * OT * 2;  // bytes of a staged row

  // staging: thread t takes pieces t, t + NT, ... of the buffers; offsets
  // within a plane, or past every descriptor's size (reads zero) outside it
  constexpr int kOut = 0x7FFFFFF0;
  int xo[K::NIX], dof[K::NID];
  uint4 rx[K::NIX], rd[K::NID];
  const int rcols = (65535 + cols) / cols;  // v / cols = v rcols >> 16 for v < 2^11
  struct Step {
    int n, w0, h0, p;  // x plane p
    int df, dl;        // dy planes of the segment
  };
  auto segment = [&](int t) {  // the segment that starts with dy plane t
    Step s;
    int tile = t / D;
    s.df = t - tile * D;
    s.dl = min(D, s.df + (t1 - t)) - 1;
    s.p = s.df - 1;
    s.w0 = tile % a.nbw * TW;
    tile /= a.nbw;
    s.h0 = tile % a.nbh * rows;
    s.n = tile / a.nbh;
#pragma unroll
    for (int i = 0; i < K::NIX; ++i) {
      const int e = tid + i * NT, q0 = e % XQ, v = e / XQ, row = v * rcols >> 16,
                sl = v - row * cols;
      const int col = CT == 16 ? slot16(sl) : sl, q = CT == 32 ? q0 ^ swz32(col) : q0;
      const int h = s.h0 - 1 + row, w = s.w0 - 1 + col;
      xo[i] = row < rows + 2 && col < TW + 2 && (unsigned)h < (unsigned)H && (unsigned)w < (unsigned)W
                  ? (((FAR ? row : h) * W + w) * a.xld + q * 8) * 2
                  : kOut;
    }
#pragma unroll
    for (int i = 0; i < K::NID; ++i) {
      const int e = tid + i * NT, q0 = e % DQ, v = e / DQ, row = v >> (a.ltwo + 3), sl = v & (TW - 1);
      const int col = OT == 16 ? slot16(sl) : sl, q = OT == 32 ? q0 ^ swz32(col) : q0;
      const int h = s.h0 + row, w = s.w0 + col;
      dof[i] = row < rows && h < H && w < W ? (((FAR ? row : h) * W + w) * a.dld + q * 8) * 2
                                            : kOut;
    }
    return s;
  };
  const long long plane = (long long)H * W;
  auto fetch = [&](const Step& s) {
    const long long xb = FAR ? (s.h0 - 1LL) * W : 0, db = FAR ? (long long)s.h0 * W : 0;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.x + (((long long)s.n * D + s.p) * plane + xb) * a.xld + a.xoff + c0), 0,
        (unsigned)s.p < (unsigned)D ? kOut : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t dr = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.dy + (((long long)s.n * D + s.p + 1) * plane + db) * a.dld + a.doff + o0), 0,
        s.p < s.dl ? kOut : 0, 0x00020000);
#pragma unroll
    for (int i = 0; i < K::NIX; ++i)
      rx[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xr, xo[i], 0, 0));
#pragma unroll
    for (int i = 0; i < K::NID; ++i)
      rd[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(dr, dof[i], 0, 0));
  };
  auto park = [&](int k) {
    uint4* const xs = reinterpret_cast<uint4*>(lds + (k & 1) * K::XB);
    uint4* const ds = reinterpret_cast<uint4*>(lds + 2 * K::XB + (k & 3) * K::DB);
#pragma unroll
    for (int i = 0; i < K::NIX; ++i) xs[tid + i * NT] = rx[i];
#pragma unroll
    for (int i = 0; i < K::NID; ++i) ds[tid + i * NT] = rd[i];
  };

  const LdsBytes base = (LdsBytes)lds;
  auto frag = [&](int lo, int hi) {
    typedef __attribute__((address_space(3))) short4v* Ptr;
    const short4v u = __builtin_amdgcn_ds_read_tr16_b64_v4i16((Ptr)(base + lo));
    const short4v v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((Ptr)(base + hi));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(u, v, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  constexpr uint32_t one2 = 0x3F803F80u;
  const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(one2, one2, one2, one2));
  // every wave sums the bias (those of the first input block store it): an MFMA
  // more for 27, but no branch among the taps
  f32x4 acc[9][NF], bacc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 9; ++i)
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      acc[i][f] = f32x4{0.f, 0.f, 0.f, 0.f};
      // opaque: a constant here has the compiler keep the loop's accumulators
      // as single registers and copy them to and from MFMA's tuples
      asm volatile("" : "+v"(acc[i][f]));
    }

  // Taps kd of [KD0, KD1) of x plane s.p (buffer xb) against the dy planes in
  // buffers db[kd].  INSIDE: the tile lies inside the grid.
  auto taps_of = [&](const Step& s, int xb, const int (&db)[3], auto kd0, auto kd1, auto inside) {
    constexpr int KD0 = decltype(kd0)::value, KD1 = decltype(kd1)::value;
    constexpr bool INSIDE = decltype(inside)::value;
    const int past = W - (s.w0 + 8 * ow);  // the octet's first voxel past the grid
    // Fragments of x by w tap and of dy by row mod 3 and kd.  Each is reloaded
    // for the next row right after its last MFMA, 12 to 18 MFMAs ahead of its next.
    bf16x8 xv[NF], dv[3][3];
    // the pitches are opaque here, or every row's addresses would be computed
    // before the plane loop and held in some 40 registers
    int xp = xrow, dp = drow;
    asm volatile("" : "+s"(xp), "+s"(dp));
    auto load_x = [&](int r, int f) {
      xv[f] = frag(xa[f][0] + (xb + r * xp), xa[f][1] + (xb + r * xp));
    };
    auto load_dy = [&](int r, int kd) {
      dv[r % 3][kd] = frag(da[0] + (db[kd] + r * dp), da[1] + (db[kd] + r * dp));
    };
#pragma unroll
    for (int kd = KD0; kd < KD1; ++kd) load_dy(0, kd);
#pragma unroll
    for (int f = 0; f < NF; ++f) load_x(0, f);
#pragma unroll
    for (int r = 0; r < RL + 2; ++r) {
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        // A tile may reach past the grid.  There dy is zero, and so is x but for
        // the grid's last column and row, which meet dy one further at kw = 0
        // and kh = 0: they count as zero there, so that no zero multiplies an
        // infinity that the sum does not hold.
        if constexpr (!INSIDE) {
          if (f == 0 && s.w0 + TW > W) {
            uint4 m = __builtin_bit_cast(uint4, xv[0]);
            const int e = CT == 8 && l16 >= 8 ? -1 : past;  // of 8 channels: kw = 0 below
            m.x &= e == 0 ? 0xFFFF0000u : (e == 1 ? 0x0000FFFFu : 0xFFFFFFFFu);
            m.y &= e == 2 ? 0xFFFF0000u : (e == 3 ? 0x0000FFFFu : 0xFFFFFFFFu);
            m.z &= e == 4 ? 0xFFFF0000u : (e == 5 ? 0x0000FFFFu : 0xFFFFFFFFu);
            m.w &= e == 6 ? 0xFFFF0000u : (e == 7 ? 0x0000FFFFu : 0xFFFFFFFFu);
            xv[0] = __builtin_bit_cast(bf16x8, m);
          }
        }
#pragma unroll
        for (int kh = 2; kh >= 0; --kh) {
          const int j = r - kh;  // dy row
          if (j >= 0 && j < RL) {
            if constexpr (!INSIDE)
              if (kh == 0 && s.h0 + rows > H && s.h0 + oh * RL + r >= H) xv[f] = zero8();
#pragma unroll
            for (int kd = KD0; kd < KD1; ++kd) {
              acc[3 * kd + kh][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  dv[j % 3][kd], xv[f], acc[3 * kd + kh][f], 0, 0, 0);
              if (f == 0 && kd == 1 && kh == 1)
                bacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dv[j % 3][kd], ones, bacc, 0, 0, 0);
            }
          }
          if (f == NF - 1 && kh == 2 && r + 1 < RL)
#pragma unroll
            for (int kd = KD0; kd < KD1; ++kd) load_dy(r + 1, kd);
        }
        if (r + 1 < RL + 2) load_x(r + 1, f);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };

  if (t0 < t1) {
    int t = t0;  // the segment's first dy plane
    Step s = segment(t), nx = s;
    fetch(s);
    park(0);
    __syncthreads();
    int k = 0;
    bool more = true;
    // fetches the next step: the segment's next x plane or the next segment's first
    auto ahead = [&]() {
      nx = s;
      if (s.p <= s.dl) {
        nx.p = s.p + 1;
      } else {
        t += s.dl - s.df + 1;
        more = t < t1;
        if (more) nx = segment(t);
      }
      if (more) fetch(nx);
    };
    auto turn = [&]() {
      if (more) {
        park(k + 1);
        __syncthreads();
      }
      s = nx;
      ++k;
    };
    auto inner = [&]() {
      return s.p > s.df && s.p < s.dl && s.w0 + TW <= W && s.h0 + rows <= H;
    };
    int db[3];
    auto bufs = [&]() {
#pragma unroll
      for (int kd = 0; kd < 3; ++kd) db[kd] = 2 * K::XB + ((k - kd) & 3) * K::DB;
      return (k & 1) * K::XB;
    };
    constexpr std::integral_constant<int, 0> i0{};
    constexpr std::integral_constant<int, 1> i1{};
    constexpr std::integral_constant<int, 2> i2{};
    constexpr std::integral_constant<int, 3> i3{};
    while (more) {
      do {
        ahead();
        const int xb = bufs();
        if (s.p < s.dl) taps_of(s, xb, db, i0, i1, std::false_type{});
        if (s.p >= s.df && s.p <= s.dl) taps_of(s, xb, db, i1, i2, std::false_type{});
        if (s.p > s.df) taps_of(s, xb, db, i2, i3, std::false_type{});
        turn();
      } while (more && !inner());
      while (more && inner()) {
        ahead();
        const int xb = bufs();
        taps_of(s, xb, db, i0, i3, std::true_type{});
        turn();
      }
    }
  }

  // Final sums into the share's row.  A lane holds output channels 4 g + e and
  // column l16 of its block.  With several waves per block they park nine
  // accumulators at a time in LDS and a thread adds one (e, lane) of each.
  const int KR = 27 * a.cin;
  float* const out = a.ws + (long long)chunk * a.rs;
  auto put = [&](int bk, int ln, int e, int i, int f, float v) {
    const int col = ln & 15, o = o0 + (bk / K::NCB) * 16 + 4 * (ln >> 4) + e;
    const int kw = CT == 8 ? 2 * f + (col >> 3) : f;
    const int c = CT == 8 ? (col & 7) : (bk % K::NCB) * 16 + col;
    if (CT > 8 || kw < 3) out[(long long)o * KR + (3 * i + kw) * a.cin + c0 + c] = v;
  };
  float* const bias = out + (long long)a.cout * KR + o0;
  if constexpr (KW == 1) {
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int i = 0; i < 9; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) put(cblk, lane, e, i, f, acc[i][f][e]);
    if (c0 == 0 && cb == 0 && l16 == 0)
#pragma unroll
      for (int e = 0; e < 4; ++e) bias[ob * 16 + 4 * g + e] = bacc[e];
  } else {
    float* const red = reinterpret_cast<float*>(lds);
    const int e = wave & 3;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 9; ++i)
        *reinterpret_cast<f32x4*>(red + ((wave * 9 + i) * 64 + lane) * 4) = acc[i][f];
      __syncthreads();
#pragma unroll
      for (int bi = 0; bi < P * 9; ++bi) {
        const int bk = bi / 9, i = bi % 9;
        if (NT > 256 && (bi & 1) != wave >> 2) continue;  // the waves' halves take turns
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < KW; ++q) v += red[(((bk + P * q) * 9 + i) * 64 + lane) * 4 + e];
        put(bk, lane, e, i, f, v);
      }
    }
    if (c0 == 0) {
      __syncthreads();
      *reinterpret_cast<f32x4*>(red + (wave * 64 + lane) * 4) = bacc;
      __syncthreads();
      if (tid < OT) {
        const int bk = (tid >> 4) * K::NCB, gg = (tid >> 2) & 3, be = tid & 3;
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < KW; ++q) v += red[((bk + P * q) * 64 + 16 * gg) * 4 + be];
        bias[tid] = v;
      }
    }
  }
}

}  // namespace unet
