// Application of an explicit convolution kernel with circular padding, and
// of its transpose (Section 3: AOC layers run as one convolution, natively
// strided, dilated, grouped, and transposed for learnable upsampling).
//
// Forward (cross-correlation, NCHW, kernel cout x c x k x k, c = cin / g):
//   y[b, o, u, v] = sum_{i,a,e} K[o, i, a, e] x[b, g(o) c + i, (s u + d a - pl) mod H, (s v + d e - pl) mod W]
// Transposed (the adjoint, from the cout x H/s x W/s grid to cin x H x W):
//   z[b, g c + i, p, q] = sum_{o,a,e} K[g og + o, i, a, e] y[b, g og + o, u, v]
//   with u = ((p + pl - d a) mod H) / s when that is a multiple of s (else
//   the term is absent), v likewise; pl = floor((d (k - 1) + 1 - s) / 2).
//
// Both run as an implicit GEMM: rows are output channels (the kernel is the
// first operand), columns are output pixels, the reduction runs over (input
// channel, tap).  Every output element is written once by one lane:
// deterministic, no atomics.  Kernels up to 3 x 3 run on the staged form
// (below, 16-bit matrix cores), others and grids too wide for its staged
// rows on the direct form: fp32 MFMA (v_mfma_f32_32x32x2f32), the second
// operand gathered from the input on the fly, 64 x 64 tiles, four waves, K
// steps of 32 through two LDS stages.
#include "internal.h"

namespace orth {

typedef float f32x16 __attribute__((ext_vector_type(16)));

namespace {

struct ApplyGeom {
  int cin, cout, k, s, d, g, c, og;
  int H, W, Ho, Wo;      // the forward conv's input and output grids
  int pl;
  int batch;
  int rows, red;         // per group: output channels, reduction length
  int64_t pix;           // output pixels (batch x output grid)
  int kdtype;
};

__device__ inline int pmod(int a, int m) {
  int r = a % m;
  return r < 0 ? r + m : r;
}
__device__ inline int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }
// a mod m for a in [-m, 2m)
__device__ inline int wrap1(int a, int m) { return a < 0 ? a + m : (a >= m ? a - m : a); }

// WRAP1: every circular index lies within one period of the grid (the host
// checks d (k - 1) and the padding against H and W), so a conditional add
// or subtract replaces the integer modulo in the gather.
// BM x BN tiles (64 or 128 each): four waves of (BM / 2) x (BN / 2), that
// is (BM / 64) x (BN / 64) accumulators of 32 x 32 each.
template <bool TR, bool WRAP1, int BM, int BN>
__global__ __launch_bounds__(256) void conv_apply_kernel(ApplyGeom G, const void* __restrict__ kern,
                                                         const float* __restrict__ x, float* __restrict__ y) {
  constexpr int BK = 32, PITCH = BK + 4;
  static_assert((BM == 64 || BM == 128) && (BN == 64 || BN == 128), "tiles of 64 or 128");
  constexpr int EA = BM * BK / 256, EB = BN * BK / 256;   // elements per thread and k-step
  constexpr int MI = BM / 64, NI = BN / 64;
  __shared__ __attribute__((aligned(16))) float As[2][BM * PITCH];
  __shared__ __attribute__((aligned(16))) float Bs[2][BN * PITCH];
  const int grp = blockIdx.z;
  const int row0 = blockIdx.y * BM;
  const int64_t pix0 = (int64_t)blockIdx.x * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int kk2 = G.k * G.k;

  // first operand: the kernel, thread -> (row, EA consecutive k)
  const int ar = tid / (BK / EA), ak = (tid % (BK / EA)) * EA;
  // second operand: gathered pixels, thread -> (pixel, EB consecutive k)
  const int bp = tid % BN, bk = (tid / BN) * EB;
  const int64_t pix = pix0 + bp;
  const bool pix_ok = pix < G.pix;
  // decompose this thread's pixel once
  int pb = 0, pu = 0, pv = 0;   // batch, row, column of the output pixel
  if (pix_ok) {
    const int ow = TR ? G.W : G.Wo, oh = TR ? G.H : G.Ho;
    pv = (int)(pix % ow);
    pu = (int)((pix / ow) % oh);
    pb = (int)(pix / ((int64_t)ow * oh));
  }
  const int64_t xplane = TR ? (int64_t)G.Ho * G.Wo : (int64_t)G.H * G.W;
  const int xch = TR ? G.cout : G.cin;
  const float* xb = x + (int64_t)pb * xch * xplane;

  uint32_t ra[EA];
  float rb[EB];
  auto gload = [&](int k0) {
    // kernel values
    {
      const int row = row0 + ar;
      int kk = k0 + ak;
      int ch = kk / kk2, tap = kk - ch * kk2;   // (input channel, tap) or (output channel, tap)
      // raw bits, widened at the LDS store (a conversion inside the guarded
      // load would make every load wait for its data)
#pragma unroll
      for (int j = 0; j < EA; ++j) {
        uint32_t v = 0;
        if (row < G.rows && kk < G.red) {
          const int64_t idx = TR ? ((int64_t)(grp * G.og + ch) * G.c + row) * kk2 + tap
                                 : (int64_t)(grp * G.og + row) * G.red + kk;
          v = G.kdtype == ORTH_BF16 ? (uint32_t) static_cast<const uint16_t*>(kern)[idx]
                                    : static_cast<const uint32_t*>(kern)[idx];
        }
        ra[j] = v;
        ++kk;
        if (++tap == kk2) {
          tap = 0;
          ++ch;
        }
      }
    }

    // gathered input values
    {
      int kk = k0 + bk;
      int ch = kk / kk2, tap = kk - ch * kk2;
      int a = tap / G.k, e = tap - a * G.k;
      // window origin of this pixel; the tap moves it by +-(d a, d e)
      const int r0 = TR ? pu + G.pl : G.s * pu - G.pl, q0 = TR ? pv + G.pl : G.s * pv - G.pl;
      int da = G.d * a, de = G.d * e;
      const float* xg = xb + (int64_t)(grp * (TR ? G.og : G.c) + ch) * xplane;
#pragma unroll
      for (int j = 0; j < EB; ++j) {
        float v = 0.f;
        if (pix_ok && kk < G.red) {
          const int rr = TR ? r0 - da : r0 + da, qq = TR ? q0 - de : q0 + de;
          const int r = WRAP1 ? wrap1(rr, G.H) : pmod(rr, G.H);
          const int q = WRAP1 ? wrap1(qq, G.W) : pmod(qq, G.W);
          if (!TR) {
            v = xg[(int64_t)r * G.W + q];
          } else if (G.s == 1) {
            v = xg[(int64_t)r * G.Wo + q];
          } else if (r % G.s == 0 && q % G.s == 0) {
            v = xg[(int64_t)(r / G.s) * G.Wo + q / G.s];
          }
        }
        rb[j] = v;
        ++kk;
        de += G.d;
        if (++e == G.k) {
          e = 0;
          de = 0;
          da += G.d;
          if (++a == G.k) {
            a = 0;
            da = 0;
            ++ch;
            xg += xplane;
          }
        }
      }
    }
  };
  auto sstore = [&](int buf) {
    // the raw values materialize here, after the MFMAs that the loads
    // overlap (otherwise the widening shift is moved into each guarded
    // load's block, where it waits for the data)
#pragma unroll
    for (int j = 0; j < EA; ++j) asm volatile("" : "+v"(ra[j]));
    float4* pa = reinterpret_cast<float4*>(&As[buf][ar * PITCH + ak]);
    const int sh = G.kdtype == ORTH_BF16 ? 16 : 0;
#pragma unroll
    for (int q = 0; q < EA / 4; ++q)
      pa[q] = make_float4(__uint_as_float(ra[4 * q] << sh), __uint_as_float(ra[4 * q + 1] << sh),
                          __uint_as_float(ra[4 * q + 2] << sh), __uint_as_float(ra[4 * q + 3] << sh));
    float4* pbv = reinterpret_cast<float4*>(&Bs[buf][bp * PITCH + bk]);
#pragma unroll
    for (int q = 0; q < EB / 4; ++q) pbv[q] = make_float4(rb[4 * q], rb[4 * q + 1], rb[4 * q + 2], rb[4 * q + 3]);
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = f32x16{};
  const int nk = (G.red + BK - 1) / BK;
  gload(0);
  sstore(0);
  __syncthreads();
  const int aoff = (wm * (BM / 2) + (lane & 31)) * PITCH + (lane >> 5) * 4;
  const int boff = (wn * (BN / 2) + (lane & 31)) * PITCH + (lane >> 5) * 4;
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) gload((kt + 1) * BK);
#pragma unroll
    for (int gq = 0; gq < BK / 8; ++gq) {
      float4 a4[MI], b4[NI];
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
        a4[mi] = *reinterpret_cast<const float4*>(&As[buf][aoff + mi * 32 * PITCH + gq * 8]);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
        b4[ni] = *reinterpret_cast<const float4*>(&Bs[buf][boff + ni * 32 * PITCH + gq * 8]);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
          f32x16& c = acc[mi][ni];
          c = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[mi].x, b4[ni].x, c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[mi].y, b4[ni].y, c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[mi].z, b4[ni].z, c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[mi].w, b4[ni].w, c, 0, 0, 0);
        }
    }
    if (kt + 1 < nk) sstore(buf ^ 1);
    __syncthreads();
  }

  // columns are pixels: consecutive lanes store consecutive pixels
  const int ow = TR ? G.W : G.Wo, oh = TR ? G.H : G.Ho;
  const int ych = TR ? G.cin : G.cout;
  const int chbase = grp * (TR ? G.c : G.og);
  const int64_t plane = (int64_t)oh * ow;
#pragma unroll
  for (int ni = 0; ni < NI; ++ni) {
    const int64_t p = pix0 + wn * (BN / 2) + ni * 32 + (lane & 31);
    if (p >= G.pix) continue;
    const int ov = (int)(p % ow);
    const int ou = (int)((p / ow) % oh);
    const int ob = (int)(p / ((int64_t)ow * oh));
    float* yp = y + ((int64_t)ob * ych + chbase) * plane + (int64_t)ou * ow + ov;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int ch = row0 + wm * (BM / 2) + mi * 32 + acc_row(r, lane);
        if (ch < G.rows) yp[(int64_t)ch * plane] = acc[mi][ni][r];
      }
  }
}


// ---------------------------------------------------------------------------
// Staged variant for k <= 3, on the 16-bit matrix cores: the fp32 values are
// split into three bfloat16 pieces x = h + m + l on their way into LDS (8 +
// 8 + 8 bits, exact), and hh + hm + mh + hl + lh + mm run on bf16 MFMA with
// fp32 accumulation, the leading product and the corrections in an
// accumulator each (a kernel stored in bf16 is its own leading piece: three
// products).  The relative error against 64 bits is about a third of fp32
// MFMA's.  A block with a result that the split cannot give (split_failed) is
// computed again with fp32 MFMA.
//
// Work: a tile is 64 output channels x 128 pixels of a grid (4 waves of 32 x
// 64); the reduction runs in chunks of CB = 8 G8 channels.  Per chunk, every
// source row that the tile's pixels need is staged once, circularly extended
// by the taps' reach, as 16-byte groups of 8 channels per position, and the
// kernel tile as such groups per (tap, row).  One MFMA covers 16 k: two
// (tap, 8-channel group) entries, lanes 0-31 reading the first and lanes
// 32-63 the second, each with its own offset from the pixel's position; so a
// staged value is split once and read by up to k^2 taps.  The next chunk's
// loads are in flight during the MFMAs (no branch around them: channels past
// the end re-read the last one, and the source's are zeroed).
//
// The grid a tile's pixels lie on, and the source position that tap (a, e)
// of pixel (u, v) reads, are the same in all forms up to constants:
//   row (ss u + rt[a]) mod Hs, column (ss v + ct[e]) mod Ws
//   forward             the output grid, ss = s, rt[a] = d a - pl
//   transposed, s = 1   the output grid, ss = 1, rt[a] = pl - d a
//   transposed, s = 2   the source's own grid (PH = 4): position (u, v) has
//                       the four outputs (2u + fh, 2v + fw); tap row a only
//                       meets outputs of one parity, fh = (d a - pl) mod 2,
//                       and reads row u + (fh + pl - d a) / 2: a quarter of
//                       the products of the zero-stuffed form.  A wave holds
//                       32 channels x 32 positions x 4 outputs.
//   transposed, k = s   one tap per output phase: a 1 x 1 kernel with its
//                       own tap, the phases in the block index
// Staged rows: consecutive source rows of each image that the tile touches,
// or (large dilation) k rows per grid row, whichever is fewer.
//
// What bounds it: six products per fp32 product; 256 channels at 28 x 28 keep
// the matrix pipes busy 58% of the cycles, at a clock of 1.98 GHz, beside VALU
// instructions in 34% of the issue cycles; the waves wait 20% of their time
// for loads and barriers (the transposed form with stride 2: 34%, 31% and
// 26%, at 2.15 GHz).  Measured with fp32 MFMA and
// staged rows (the zero-stuffed transposed form) and now: 256 -> 256 channels,
// 28 x 28, batch 64: 969 -> 387 us (61 -> 153 TFLOP/s; bf16 kernel 1032 ->
// 243), transposed 998 -> 376 (1158 -> 243); 128 -> 256, stride 2, 32 x 32,
// batch 128: 389 -> 155 (380 -> 100), transposed 1183 -> 165 (1376 -> 134).
// With one infinity per sample 984 us and transposed 814, 343 and 722; NaN
// throughout 458, 396, 225 and 203.
struct StageGeom {
  int Hg, Wg;            // the grid of the tile's pixels
  int Hs, Ws;            // the source grid
  int ss;                // source step per grid step
  int64_t pix;           // batch x Hg x Wg
  int rt[3], ct[3];      // tap row / column shifts
  int rmin, cmin;        // their minima
  int rows_sep;          // 1: k staged rows per grid row, 0: consecutive rows
  int seg;               // consecutive rows: staged rows of a whole image
  int WX;                // staged columns
  int npos;              // staged positions (rows x WX), at most PU 256
  int nch;               // reduction channels per group
  int os, nph;           // output step; phases in the block index (k = s > 2: os^2)
  int kk2;               // taps of the stored kernel
  int par;               // s = 2: parity of pl (the output parity of tap row a is (a + par) mod 2)
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
// 16- and 8-byte global loads at element alignment (gfx950 needs no more)
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x2_a2 __attribute__((ext_vector_type(2), aligned(2)));

// A wave's 32 x 32 block with fp32 MFMA: this lane's channel `row` of the
// group (as MFMA row) and output pixel (as column), by the formula.  16
// channels of one tap at a time straight from memory (the lower lanes hold
// the first eight, the upper ones the others; all taps of 16 channels before
// the next 16, so that the kernel's lines are read whole); loads past an end
// re-read the last value and count as zero (byte offsets fit 32 bits, see
// stage_geom).  Done early where every value is NaN already.
template <bool TR>
__device__ __forceinline__ f32x16 conv_block_f32(const ApplyGeom& G, const void* kern, const float* x, int grp,
                                                 int row, bool pix_ok, int b, int p, int q) {
  constexpr int CN = 8;   // (a lane half's channels)
  f32x16 acc = {};
  const int kk2 = G.k * G.k, nch = TR ? G.og : G.c, chh = CN * ((threadIdx.x >> 5) & 1);
  const uint32_t cplane = TR ? G.Ho * G.Wo : G.H * G.W, kch = TR ? G.c * kk2 : kk2;   // between channels
  const uint32_t rc = row < G.rows ? row : G.rows - 1;
  const uint32_t k0 = TR ? (grp * G.og * G.c + rc) * kk2 : (grp * G.og + rc) * G.red;
  const uint32_t x0 = (b * (TR ? G.cout : G.cin) + grp * nch) * cplane;
  const bool row_ok = row < G.rows, narrow = G.kdtype == ORTH_BF16;
#pragma unroll 1
  for (int ch0 = 0; ch0 < nch; ch0 += 2 * CN) {
    const int ch = ch0 + chh;
#pragma unroll 1
    for (int tap = 0; tap < kk2; ++tap) {
      const int a = tap / G.k, e = tap - a * G.k;
      int r = pmod(TR ? p + G.pl - G.d * a : G.s * p + G.d * a - G.pl, G.H);
      int c = pmod(TR ? q + G.pl - G.d * e : G.s * q + G.d * e - G.pl, G.W);
      const bool hit = pix_ok && (!TR || (r % G.s == 0 && c % G.s == 0));
      if (!__any(hit)) continue;
      if (TR) {
        r /= G.s;
        c /= G.s;
      }
      const uint32_t xt = x0 + r * (TR ? G.Wo : G.W) + c, kt = k0 + tap;
      uint32_t av[CN], bv[CN];
#pragma unroll
      for (int i = 0; i < CN; ++i) {
        const uint32_t cc = ch + i < nch ? ch + i : nch - 1;
        const uint32_t ko = kt + cc * kch, xo = (xt + cc * cplane) * 4;
        const char* kp = static_cast<const char*>(kern);
        av[i] = narrow ? (uint32_t)gld_u16(kp + ko * 2u, 0) << 16 : gld_u32(kp + ko * 4u, 0);
        bv[i] = gld_u32(reinterpret_cast<const char*>(x) + xo, 0);
      }
#pragma unroll
      for (int i = 0; i < CN; ++i) {
        const bool in = ch + i < nch;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(in && row_ok ? __uint_as_float(av[i]) : 0.f,
                                                   in && hit ? __uint_as_float(bv[i]) : 0.f, acc, 0, 0, 0);
      }
    }
    if (__all(all_nan(acc) || !pix_ok)) break;
  }
  return acc;
}

template <bool TR, int KS, int PH, bool KBF16, int PU>
__global__ __launch_bounds__(256, 2) void conv_apply_staged_kernel(ApplyGeom G, StageGeom T,
                                                                   const void* __restrict__ kern,
                                                                   const float* __restrict__ x,
                                                                   float* __restrict__ y) {
  static_assert(PH == 1 || (TR && KS >= 2), "output phases of the transposed form with stride 2");
  constexpr int KK = KS * KS, G8 = KS == 3 ? 1 : 2, CB = 8 * G8, NE = KK * G8, NS = (NE + 1) / 2;
  constexpr int NB = PH == 4 ? 4 : 2;                // 32 x 32 blocks of a wave
  constexpr int BN = PH == 4 ? 64 : 128;             // positions of a tile
  constexpr int PA = KBF16 ? 1 : 3;                  // pieces of the kernel
  extern __shared__ __attribute__((aligned(16))) uint4 smem4[];
  uint4* const As = smem4;                           // [piece][entry 0 .. 2 NS)[64 rows]
  uint4* const Xs = smem4 + PA * 2 * NS * 64;        // [piece][group][position]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
  const int wm = wave >> 1, wn = wave & 1;
  const int grp = blockIdx.z, row0 = blockIdx.y * 64;
  const int phase = T.nph > 1 ? (int)(blockIdx.x % T.nph) : 0;
  const int64_t p0 = (int64_t)(T.nph > 1 ? blockIdx.x / T.nph : blockIdx.x) * BN;
  const int pfh = phase / T.os, pfw = phase - pfh * T.os;   // (only read with T.nph > 1)

  int tap0 = 0, rt0 = 0, ct0 = 0;
  if (T.nph > 1) {
    // the tap (a, e) whose outputs have this phase: (d a - pl) mod s = pfh
    for (int a = 0; a < G.k; ++a)
      for (int e = 0; e < G.k; ++e)
        if (pmod(G.d * a - G.pl, G.s) == pfh && pmod(G.d * e - G.pl, G.s) == pfw) {
          tap0 = a * G.k + e;
          rt0 = (pfh + G.pl - G.d * a) / G.s;
          ct0 = (pfw + G.pl - G.d * e) / G.s;
        }
  }

  // entry of (tap, group): (tap, group) in order; four output phases: the
  // taps of one phase side by side
  auto entry = [&](int tap, int g) {
    if (PH == 4 && KS == 3) return (int)((0x352786140ull >> (4 * tap)) & 15);   // see tap_of
    return tap * G8 + g;
  };
  // its inverse: tap of entry i (the last entry of an odd count repeats its
  // neighbour's position, with zero kernel values)
  auto tap_of = [&](int i) {
    if (PH == 4 && KS == 3) {
      constexpr int t[10] = {0, 2, 6, 8, 1, 7, 3, 5, 4, 4};
      return t[i];
    }
    return (i < NE ? i : NE - 1) / G8;
  };
  // block of slot q (two entries): always both with one phase, else that of
  // the tap's parities
  auto phase_of = [&](int q) {
    if (PH == 1) return 0;
    if (KS == 3) return q < 2 ? 0 : q - 1;
    return q;   // KS == 2: slot = tap
  };

  // staged position of grid row `orow`: first staged row for tap offset 0
  const int64_t first_row = p0 / T.Wg;
  const int b0 = (int)(first_row / T.Hg), u0 = (int)(first_row - (int64_t)b0 * T.Hg);
  const int seg0 = T.ss * (T.Hg - 1 - u0) + (T.seg - T.ss * (T.Hg - 1));   // staged rows of the first image
  int poff[NB];   // this lane's pixel (PH == 4: the same for every block)
#pragma unroll
  for (int i = 0; i < (PH == 4 ? 1 : NB); ++i) {
    const int64_t pn = p0 + wn * (BN / 2) + i * 32 + (lane & 31);
    poff[i] = 0;
    if (pn < T.pix) {
      const int64_t orow = pn / T.Wg;
      const int v = (int)(pn - orow * T.Wg), j = (int)(orow - first_row);
      const int b = (int)(orow / T.Hg), u = (int)(orow - (int64_t)b * T.Hg);
      const int slot = T.rows_sep ? j * KS : b == b0 ? T.ss * (u - u0) : seg0 + (b - b0 - 1) * T.seg + T.ss * u;
      poff[i] = slot * T.WX + T.ss * v;
    }
  }
  int koff[NS];   // this lane half's entry of each slot, relative to the pixel
#pragma unroll
  for (int q = 0; q < NS; ++q) {
    const int t0 = tap_of(2 * q), t1 = tap_of(2 * q + 1);
    const int g0 = (KS == 3) ? 0 : (2 * q) % G8, g1 = (KS == 3) ? 0 : (2 * q + 1) % G8;
    auto off = [&](int t, int g) {
      const int a = t / KS, e = t % KS;
      return g * T.npos + (T.rows_sep ? a : T.rt[a] - T.rmin) * T.WX + (T.ct[e] - T.cmin);
    };
    const int o0 = KS == 1 ? 0 : off(t0, g0), o1 = KS == 1 ? T.npos : off(t1, g1);
    koff[q] = half ? o1 : o0;
  }

  // this thread's staged positions: byte offset of the first channel group
  const int64_t cplane = (int64_t)T.Hs * T.Ws;
  const int src_ch = TR ? G.cout : G.cin;
  uint32_t xoff[PU];
#pragma unroll
  for (int i = 0; i < PU; ++i) {
    const int pos = tid + i * 256;
    xoff[i] = 0;
    if (pos < T.npos) {
      const int slot = pos / T.WX, col = pos - slot * T.WX;
      int b, r;
      if (T.rows_sep) {
        const int64_t orow = first_row + slot / KS;
        const int a = slot % KS;
        b = (int)(orow / T.Hg);
        r = T.ss * (int)(orow - (int64_t)b * T.Hg) + (T.nph > 1 ? rt0 : T.rt[a]);
      } else if (slot < seg0) {
        b = b0;
        r = T.ss * u0 + slot + (T.nph > 1 ? rt0 : T.rmin);
      } else {
        const int g = (slot - seg0) / T.seg;
        b = b0 + 1 + g;
        r = slot - seg0 - g * T.seg + (T.nph > 1 ? rt0 : T.rmin);
      }
      const int sr = pmod(r, T.Hs), sc = pmod(col + (T.nph > 1 ? ct0 : T.cmin), T.Ws);
      if (b < G.batch)
        xoff[i] = (uint32_t)((((int64_t)b * src_ch + (int64_t)grp * T.nch) * cplane + (int64_t)sr * T.Ws + sc) * 4);
    }
  }
  // this thread's kernel values: row `krow`, channels 2 kc2 and 2 kc2 + 1 of
  // each group, all taps (a contiguous run per channel).  Lanes of a wave
  // hold 16 rows x 4 channel pairs, so the stores of a tap are conflict free
  const int krow = tid >> 2, kc2 = tid & 3;
  const int64_t ch_stride = TR ? (int64_t)G.c * T.kk2 : T.kk2;   // elements between reduction channels
  const int krc = row0 + krow < G.rows ? row0 + krow : G.rows - 1;
  const int64_t kbase = (TR ? ((int64_t)grp * G.og * G.c + krc) * T.kk2 : (int64_t)(grp * G.og + krc) * G.red) +
                        (KS == 1 ? tap0 : 0);
  // the zero entry of an odd count
  if (NE & 1)
    for (int i = tid; i < PA * 64; i += 256) As[(i / 64 * 2 * NS + NE) * 64 + i % 64] = make_uint4(0, 0, 0, 0);

  constexpr int KW = KBF16 ? (KK + 1) / 2 : KK;   // words of a run
  uint32_t ra[G8][2][KW];
  float rx[PU][G8][8];
  auto load = [&](int ch0) {
#pragma unroll
    for (int g = 0; g < G8; ++g)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int ch = ch0 + 8 * g + 2 * kc2 + c;
        const int64_t e = kbase + (ch < T.nch ? ch : T.nch - 1) * ch_stride;
        uint32_t* w = ra[g][c];
        if constexpr (KBF16) {
          const uint16_t* q = static_cast<const uint16_t*>(kern) + e;
          if constexpr (KK >= 8) {
            const u32x4_a2 v = *(const ORTH_GLOBAL u32x4_a2*)q;
            w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
            w[4] = gld_u16(q, 8);
          } else if constexpr (KK == 4) {
            const u32x2_a2 v = *(const ORTH_GLOBAL u32x2_a2*)q;
            w[0] = v.x; w[1] = v.y;
          } else {
            w[0] = gld_u16(q, 0);
          }
        } else {
          const float* q = static_cast<const float*>(kern) + e;
#pragma unroll
          for (int k = 0; k + 4 <= KK; k += 4) {
            const u32x4_a4 v = *(const ORTH_GLOBAL u32x4_a4*)(q + k);
            w[k] = v.x; w[k + 1] = v.y; w[k + 2] = v.z; w[k + 3] = v.w;
          }
          if constexpr (KK % 4) w[KK - 1] = gld_u32(q, KK - 1);
        }
      }
#pragma unroll
    for (int g = 0; g < G8; ++g)
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int ch = ch0 + 8 * g + c < T.nch ? ch0 + 8 * g + c : T.nch - 1;
        const char* xq = reinterpret_cast<const char*>(x + ch * cplane);
#pragma unroll
        for (int i = 0; i < PU; ++i) rx[i][g][c] = gld_f32(xq + xoff[i], 0);
      }
  };
  auto stage = [&](int ch0) {
    uint32_t* aw = reinterpret_cast<uint32_t*>(As);
#pragma unroll
    for (int g = 0; g < G8; ++g)
#pragma unroll
      for (int t = 0; t < KK; ++t) {
        const int dst = (entry(t, g) * 64 + krow) * 4 + kc2;
        if constexpr (KBF16) {
          const uint32_t a = ra[g][0][t / 2], b = ra[g][1][t / 2];
          aw[dst] = t & 1 ? (a >> 16) | (b & 0xffff0000u) : (a & 0xffffu) | (b << 16);
        } else {
          uint32_t h, m, l;
          split2_bf16(__uint_as_float(ra[g][0][t]), __uint_as_float(ra[g][1][t]), h, m, l);
          aw[dst] = h;
          aw[dst + 2 * NS * 256] = m;
          aw[dst + 4 * NS * 256] = l;
        }
      }
    const int nv = T.nch - ch0;
    if (nv < CB) {
#pragma unroll
      for (int g = 0; g < G8; ++g)
#pragma unroll
        for (int c = 0; c < 8; ++c)
          if (8 * g + c >= nv) {
#pragma unroll
            for (int i = 0; i < PU; ++i) rx[i][g][c] = 0.f;
          }
    }
#pragma unroll
    for (int i = 0; i < PU; ++i) {
      const int pos = tid + i * 256;
      if (pos < T.npos) {
#pragma unroll
        for (int g = 0; g < G8; ++g) {
          uint32_t w[3][4];
#pragma unroll
          for (int q = 0; q < 4; ++q) split2_bf16(rx[i][g][2 * q], rx[i][g][2 * q + 1], w[0][q], w[1][q], w[2][q]);
#pragma unroll
          for (int q = 0; q < 3; ++q) Xs[(q * G8 + g) * T.npos + pos] = make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
        }
      }
    }
  };

  f32x16 acc[2][NB];   // the leading products, the corrections
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int i = 0; i < NB; ++i) acc[q][i] = f32x16{};
  auto mma = [&](uint4 a, uint4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
  };
  const int arow = wm * 32 + (lane & 31);
  load(0);
  for (int ch0 = 0; ch0 < T.nch; ch0 += CB) {
    __syncthreads();
    stage(ch0);
    __syncthreads();
    load(ch0 + CB < T.nch ? ch0 + CB : ch0);
#pragma unroll
    for (int q = 0; q < NS; ++q) {
      uint4 fa[PA];
#pragma unroll
      for (int p = 0; p < PA; ++p) fa[p] = As[(p * 2 * NS + 2 * q + half) * 64 + arow];
#pragma unroll
      for (int i = 0; i < (PH == 4 ? 1 : NB); ++i) {
        uint4 fb[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) fb[p] = Xs[p * G8 * T.npos + poff[i] + koff[q]];
        f32x16& lead = acc[0][PH == 4 ? phase_of(q) : i];
        f32x16& corr = acc[1][PH == 4 ? phase_of(q) : i];
        if constexpr (KBF16) {
          corr = mma(fa[0], fb[2], corr);
          corr = mma(fa[0], fb[1], corr);
        } else {
          corr = mma(fa[2], fb[0], corr);
          corr = mma(fa[0], fb[2], corr);
          corr = mma(fa[1], fb[1], corr);
          corr = mma(fa[1], fb[0], corr);
          corr = mma(fa[0], fb[1], corr);
        }
        lead = mma(fa[0], fb[0], lead);
      }
    }
  }

  // this lane's output of block i: sample and position; false past the end
  auto output = [&](int i, int& b, int& u, int& v) -> bool {
    const int64_t pn = p0 + wn * (BN / 2) + (PH == 4 ? 0 : i * 32) + (lane & 31);
    const int64_t orow = pn / T.Wg;
    b = (int)(orow / T.Hg);
    u = (int)(orow - (int64_t)b * T.Hg);
    v = (int)(pn - orow * T.Wg);
    if (PH == 4) {   // block i holds the taps of row parity i / 2, column parity i % 2
      u = 2 * u + ((i >> 1) ^ T.par);
      v = 2 * v + ((i & 1) ^ T.par);
    } else if (T.nph > 1) {
      u = T.os * u + pfh;
      v = T.os * v + pfw;
    }
    return pn < T.pix;
  };
  uint32_t failed = 0;   // this wave's blocks that the split cannot give
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    acc[0][i] += acc[1][i];
    failed |= __any(split_failed(acc[0][i], kSplitLo)) ? 1u << i : 0u;
  }
  if (__builtin_expect(failed != 0, 0)) {
#pragma unroll 1
    for (int n = 0; n < NB; ++n) {
      if (!(failed >> n & 1)) continue;
      int b, u, v;
      const bool ok = output(n, b, u, v);
      const f32x16 t = conv_block_f32<TR>(G, kern, x, grp, row0 + wm * 32 + (lane & 31), ok, ok ? b : 0, u, v);
#pragma unroll
      for (int i = 0; i < NB; ++i)
        if (i == n) acc[0][i] = t;
    }
  }
  // columns are pixels: consecutive lanes store consecutive pixels
  const int oh = TR ? G.H : G.Ho, ow = TR ? G.W : G.Wo;
  const int ych = TR ? G.cin : G.cout, chb = grp * (TR ? G.c : G.og);
  const int64_t plane = (int64_t)oh * ow;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    int b, u, v;
    if (!output(i, b, u, v)) continue;
    float* yp = y + ((int64_t)b * ych + chb) * plane + (int64_t)u * ow + v;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int ch = row0 + wm * 32 + acc_row(r, lane);
      if (ch < G.rows) gst_f32(yp, (int64_t)ch * plane, acc[0][i][r]);
    }
  }
}

template <bool TR, int KS, int PH, bool KBF16, int PU>
hipError_t launch_staged_one(const ApplyGeom& G, const StageGeom& T, const orth_conv_apply_args* a, hipStream_t s) {
  constexpr int KK = KS * KS, G8 = KS == 3 ? 1 : 2, NS = (KK * G8 + 1) / 2, BN = PH == 4 ? 64 : 128;
  const size_t lds = ((size_t)(KBF16 ? 1 : 3) * 2 * NS * 64 + (size_t)3 * G8 * T.npos) * 16;
  auto kp = &conv_apply_staged_kernel<TR, KS, PH, KBF16, PU>;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kp),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const dim3 grid((unsigned)((T.pix + BN - 1) / BN * T.nph), (unsigned)((G.rows + 63) / 64), (unsigned)G.g);
  hipLaunchKernelGGL((conv_apply_staged_kernel<TR, KS, PH, KBF16, PU>), grid, dim3(256), lds, s, G, T, a->kernel, a->x,
                     a->y);
  return hipGetLastError();
}
// Staged positions a workgroup holds at most (k = 3: 6 a thread, which takes
// in the forward form with stride 3 on any grid: 96 channels, 27 x 27, batch
// 16, 42.7 us staged, 69.9 direct).
constexpr int max_positions(int ks) { return ks == 3 ? 6 * 256 : 5 * 256; }
template <bool TR, int KS, int PH>
hipError_t launch_staged(const ApplyGeom& G, const StageGeom& T, const orth_conv_apply_args* a, hipStream_t s) {
  constexpr int PW = max_positions(KS) / 256;
  const bool narrow = G.kdtype == ORTH_BF16, wide = T.npos > 2 * 256;
  if (narrow) return wide ? launch_staged_one<TR, KS, PH, true, PW>(G, T, a, s)
                          : launch_staged_one<TR, KS, PH, true, 2>(G, T, a, s);
  return wide ? launch_staged_one<TR, KS, PH, false, PW>(G, T, a, s)
              : launch_staged_one<TR, KS, PH, false, 2>(G, T, a, s);
}

// The staged form's geometry; false where it does not apply (k > 3, other
// strides of the transposed form, more staged positions than a workgroup
// holds, tensors past 32-bit byte offsets).
bool stage_geom(const ApplyGeom& G, bool tr, StageGeom& T, int& ks, int& ph) {
  if (G.k > 3) return false;
  if (tr && G.s > 2 && G.k != G.s) return false;
  const int64_t src = (int64_t)G.batch * (tr ? (int64_t)G.cout * G.Ho * G.Wo : (int64_t)G.cin * G.H * G.W);
  if (src >= ((int64_t)1 << 30) || (int64_t)G.cout * G.c * G.k * G.k >= ((int64_t)1 << 30)) return false;
  const bool one_tap = tr && G.s > 2;            // k = s: one tap per output phase
  ks = one_tap ? 1 : G.k;
  ph = tr && G.s == 2 ? 4 : 1;
  T.Hs = tr ? G.Ho : G.H;
  T.Ws = tr ? G.Wo : G.W;
  T.Hg = tr && G.s > 1 ? G.Ho : tr ? G.H : G.Ho;
  T.Wg = tr && G.s > 1 ? G.Wo : tr ? G.W : G.Wo;
  T.ss = tr ? 1 : G.s;
  T.pix = (int64_t)G.batch * T.Hg * T.Wg;
  T.nch = tr ? G.og : G.c;
  T.os = one_tap ? G.s : 1;
  T.nph = T.os * T.os;
  T.kk2 = G.k * G.k;
  T.par = G.pl & 1;
  for (int a = 0; a < 3; ++a) {
    int t = 0;
    if (a < ks && !one_tap) {
      if (!tr)
        t = G.d * a - G.pl;
      else if (G.s == 1)
        t = G.pl - G.d * a;
      else   // s = 2, d odd: the parity of d a - pl, then an exact half
        t = (((a + T.par) & 1) + G.pl - G.d * a) / 2;
    }
    T.rt[a] = T.ct[a] = t;
  }
  T.rmin = T.rt[0];
  int rmax = T.rt[0];
  for (int a = 1; a < ks; ++a) {
    T.rmin = std::min(T.rmin, T.rt[a]);
    rmax = std::max(rmax, T.rt[a]);
  }
  T.cmin = T.rmin;
  const int span = rmax - T.rmin, bn = ph == 4 ? 64 : 128;
  T.WX = T.ss * (T.Wg - 1) + span + 1;
  T.seg = T.ss * (T.Hg - 1) + span + 1;
  const int64_t J = (T.Wg - 1 + bn - 1) / T.Wg + 1;             // grid rows a tile touches, at most
  const int64_t nimg = (T.Hg - 1 + J - 1) / T.Hg + 1;           // images, at most
  const int64_t cons = std::max((J - 1) * T.ss + span + 1, (J - nimg) * T.ss + nimg * (span + 1));
  T.rows_sep = J * ks < cons;
  const int64_t npos = (T.rows_sep ? J * ks : cons) * T.WX;
  if (npos > max_positions(ks)) return false;
  T.npos = (int)npos;
  return T.nch > 0;
}

}  // namespace

hipError_t launch_conv_apply(const orth_conv_apply_args* a, hipStream_t s) {
  const orth_conv_geom& g = a->geom;
  ApplyGeom G{};
  G.cin = g.cin;
  G.cout = g.cout;
  G.k = g.k;
  G.s = g.stride;
  G.d = g.dilation;
  G.g = g.groups;
  G.c = g.cin / g.groups;
  G.og = g.cout / g.groups;
  G.H = a->height;
  G.W = a->width;
  G.Ho = a->height / g.stride;
  G.Wo = a->width / g.stride;
  G.pl = (g.dilation * (g.k - 1) + 1 - g.stride) / 2;
  G.batch = a->batch;
  G.rows = a->transposed ? G.c : G.og;
  G.red = (a->transposed ? G.og : G.c) * g.k * g.k;
  G.pix = (int64_t)a->batch * (a->transposed ? (int64_t)G.H * G.W : (int64_t)G.Ho * G.Wo);
  G.kdtype = a->kernel_dtype;
  // staged kernel where it applies
  {
    StageGeom T{};
    int ks = 1, ph = 1;
    const bool tr = a->transposed != 0;
    if (stage_geom(G, tr, T, ks, ph)) {
      const char* name = tr ? "conv_apply_transposed" : "conv_apply";
      timing_begin(name, s);
      hipError_t e;
      if (!tr)
        e = ks == 1   ? launch_staged<false, 1, 1>(G, T, a, s)
            : ks == 2 ? launch_staged<false, 2, 1>(G, T, a, s)
                      : launch_staged<false, 3, 1>(G, T, a, s);
      else if (ph == 4)
        e = ks == 2 ? launch_staged<true, 2, 4>(G, T, a, s) : launch_staged<true, 3, 4>(G, T, a, s);
      else
        e = ks == 1   ? launch_staged<true, 1, 1>(G, T, a, s)
            : ks == 2 ? launch_staged<true, 2, 1>(G, T, a, s)
                      : launch_staged<true, 3, 1>(G, T, a, s);
      timing_end(name, s);
      return e;
    }
  }
  // 64 x 64 tiles: measured on the CIFAR- and ImageNet-like stacks, 128 x
  // 128 tiles (four times the MFMA work per gathered element) were no
  // faster on wide layers and up to 2x slower where the small late grids
  // leave few tiles, and 16-deep k-steps won on neither
  constexpr int TB = 64;
  const dim3 grid((unsigned)((G.pix + TB - 1) / TB), (unsigned)((G.rows + TB - 1) / TB), (unsigned)g.groups);
  const char* name = a->transposed ? "conv_apply_transposed" : "conv_apply";
  // circular indices within one period: forward s u + d a - pl over
  // [-pl, H - s + d (k - 1) - pl], transposed p + pl - d a over
  // [pl - d (k - 1), H - 1 + pl] (likewise for W)
  const int span = G.d * (G.k - 1);
  const int lo = a->transposed ? G.pl - span : -G.pl;
  const int hi_h = a->transposed ? G.H - 1 + G.pl : G.H - G.s + span - G.pl;
  const int hi_w = a->transposed ? G.W - 1 + G.pl : G.W - G.s + span - G.pl;
  const bool w1 = lo >= -std::min(G.H, G.W) && hi_h < 2 * G.H && hi_w < 2 * G.W;
  timing_begin(name, s);
#define ORTH_APPLY(TR_, W1_, T_)                                                                              \
  hipLaunchKernelGGL((conv_apply_kernel<TR_, W1_, T_, T_>), grid, dim3(256), 0, s, G, a->kernel, a->x, a->y)
  if (a->transposed && w1) ORTH_APPLY(true, true, TB);
  else if (a->transposed) ORTH_APPLY(true, false, TB);
  else if (w1) ORTH_APPLY(false, true, TB);
  else ORTH_APPLY(false, false, TB);
#undef ORTH_APPLY
  hipError_t e = hipGetLastError();
  timing_end(name, s);
  return e;
}

}  // namespace orth
