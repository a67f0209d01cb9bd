// Table-driven fp32 "NT" GEMM on gfx950: every work item is one product
// C = A B^T (+ A2 B2^T and any further pairs from a table, accumulated into
// the same tile) with its own operands, shapes and epilogue, and every block
// one square tile of such an item (from a tile list), so a single launch
// covers a whole ragged batch (all matrices of a Björck step, all tap
// products of a composition step, all Gram checks).  A launch's step
// argument moves each operand by its item's per-step offset, so one table
// serves every step of a recurrence whose buffers are laid out step after
// step.
//
// fp32 operands stay fp32 in memory; on the way into LDS each value is split
// into 16-bit pieces whose sum carries its 24 bits, and the products of the
// pieces run on the 16-bit matrix cores (16 times the fp32 MFMA rate) with
// fp32 accumulation:
//   GEMM_BF16X3  x = h + m + l in bfloat16 (8 + 8 + 8 bits, any exponent);
//                hh + hm + mh + hl + lh + mm, the dropped products are below
//                2^-25 of hh
//   GEMM_F16X2   2^e x = h + 2^-11 l in half (11 + 11 bits and a sign);
//                hh + 2^-11 (hl + lh).  For operands whose range is known:
//                the item's exponents e put values up to 4 below half's
//                largest, and values down to 2^-27 of that keep 22 bits or
//                more.
// The leading product and the corrections have an accumulator each: a
// correction's rounding then no longer happens at the size of the whole sum.
// Relative error against 64 bits, normal operands, K = 64 / 512 / 4096:
// fp32 MFMA 1.4e-7 / 4.1e-7 / 1.2e-6, three bf16 pieces 5.0e-8 / 1.3e-7 /
// 4.0e-7, two half pieces 9.8e-8 / 1.7e-7 / 4.1e-7 (one accumulator for
// all: 1.1e-7 / 3.4e-7 / 1.0e-6).
// A tile whose result is not finite (an infinity splits into inf - inf; a
// value past half's range) is computed again with fp32 MFMA, so infinities,
// NaN and overflow come out as fp32 arithmetic has them.
//
// Operands that only products read (transposed iterates, E, S', the powers
// of an exponential) are stored as half pieces by the launch that makes them
// (GEMM_PRE_*; store_pieces8 has the layout, in the space of the fp32
// values) and go to LDS as they are.
//
// What bounds it where operands are split on the way: the splitting.  VALU
// and MFMA instructions of a SIMD's waves share its issue slots (8 full-rate
// VALU instructions beside each 32 x 32 x 16 MFMA take 100 cycles per two of
// them, 64 without), and per 32-deep step a 64 x 64 tile spends about 270
// cycles of VALU per wave beside 192 of MFMA (two pieces, both operands);
// 128 x 128 tiles halve the splitting per product.  So lists with a
// 128-tile for every compute unit use those, others 64.  With stored pieces
// it is the wait for loads issued a step ahead (0.62 us per 32-deep step of
// 256 128-tiles, 0.49 without loads; the L2 gives 17 TB/s and more to a
// plain reader, 13.5 here).  Measured with fp32 MFMA, splitting on the way,
// and stored pieces: exponential map of 4 x 2048^2, 676, 287, 251 us per
// power (102, 239, 274 TFLOP/s); update of a 2048 x 1024 iterate 58, 31,
// 28.8 us, of eight 512^2 ones 36, 21, 20.4 us; Gram matrix of 2048 x 1024
// 34 -> 26.7, of eight 512^2 18 -> 15.4 us (the last two columns).  Three
// pieces, split on the way: conv exponential of 512 channels, 776 -> 456 us
// per power (86 -> 147 TFLOP/s).
//
// K advances in steps of 32 through two LDS stages (see the pipeline below).
#include "internal.h"

namespace orth {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

namespace {

__device__ inline int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// 16 bytes from any 4-byte aligned global address (gfx950 needs no more for
// multi-dword accesses)
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ uint4 gld_u32x4_a4(const float* p) {
  const u32x4u v = *(const ORTH_GLOBAL u32x4u*)p;
  return make_uint4(v.x, v.y, v.z, v.w);
}

template <int SC>
struct Split;
template <>
struct Split<GEMM_BF16X3> {
  static constexpr int P = 3, NP = 6;   // pieces, products (smallest first, the leading one last)
  static __device__ constexpr int pa(int q) { return q == 0 ? 2 : q == 2 || q == 3 ? 1 : 0; }
  static __device__ constexpr int pb(int q) { return q == 1 ? 2 : q == 2 || q == 4 ? 1 : 0; }
  static constexpr float CORR = 1.f;
  static __device__ __forceinline__ uint32_t cvt2(float a, float b) {
    const f32x2v v{a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2v));
  }
  static __device__ __forceinline__ void split2(float a, float b, float, uint32_t (&o)[P]) {
    o[0] = cvt2(a, b);
    const float ra = a - __uint_as_float(o[0] << 16), rb = b - __uint_as_float(o[0] & 0xffff0000u);
    o[1] = cvt2(ra, rb);
    o[2] = cvt2(ra - __uint_as_float(o[1] << 16), rb - __uint_as_float(o[1] & 0xffff0000u));
  }
  static __device__ __forceinline__ float scale(int) { return 1.f; }
  static __device__ __forceinline__ f32x16 mma(uint4 a, uint4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
  }
};
template <>
struct Split<GEMM_F16X2> {
  static constexpr int P = 2, NP = 3;
  static __device__ constexpr int pa(int q) { return q == 0 ? 1 : 0; }
  static __device__ constexpr int pb(int q) { return q == 1 ? 1 : 0; }
  static constexpr float CORR = 1.f / 2048.f;
  static __device__ __forceinline__ void split2(float a, float b, float s, uint32_t (&o)[P]) {
    split2_f16(a, b, s, o[0], o[1]);
  }
  static __device__ __forceinline__ float scale(int e) { return pow2f(e); }
  static __device__ __forceinline__ f32x16 mma(uint4 a, uint4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
  }
};

// One operand pair of an item at the launch's step.
struct PairView {
  const char *A, *B;
  int64_t lda, ldb;
  int K, atr, btr;
};
// `g` may be a copy in registers: both pairs' values are taken, then chosen
// (a choice between their addresses would keep the copy in scratch memory)
__device__ __forceinline__ PairView pair_view(const GemmItem& g, const GemmPair* extra, int pair, int64_t st) {
  PairView v;
  if (pair < 2) {
    const int64_t sa = g.a_dtype == ORTH_BF16 ? 2 : 4, sb = g.b_dtype == ORTH_BF16 ? 2 : 4;
    const int tr = g.trans >> (2 * pair);
    const char* a1 = static_cast<const char*>(g.A) + g.a_step * st * sa;
    const char* a2 = static_cast<const char*>(g.A2) + g.a2_step * st * sa;
    const char* b1 = static_cast<const char*>(g.B) + g.b_step * st * sb;
    const char* b2 = static_cast<const char*>(g.B2) + g.b2_step * st * sb;
    const int64_t la1 = g.lda, la2 = g.lda2, lb1 = g.ldb, lb2 = g.ldb2;
    const int k1 = g.K, k2 = g.K2;
    v.A = pair ? a2 : a1;
    v.B = pair ? b2 : b1;
    v.lda = pair ? la2 : la1;
    v.ldb = pair ? lb2 : lb1;
    v.K = pair ? k2 : k1;
    v.atr = tr & GEMM_A_TRANS;
    v.btr = tr & GEMM_B_TRANS;
  } else {
    const GemmPair* x = extra + g.pair_base + (pair - 2);
    v.A = static_cast<const char*>(x->A);
    v.B = static_cast<const char*>(x->B);
    v.lda = x->lda;
    v.ldb = x->ldb;
    v.K = x->K;
    v.atr = x->a_trans;
    v.btr = x->b_trans;
  }
  return v;
}
__device__ __forceinline__ int exp_of(int exps, int i) { return (int)((uint32_t)exps << (24 - 8 * i)) >> 24; }

// The wave's 32 x 32 block at (i0, j0) with fp32 MFMA and guarded loads: the
// tiles whose split result is not finite.
__device__ __forceinline__ f32x16 block_f32(const GemmItem& g, const GemmPair* extra, int64_t st, int i0,
                                            int j0) {
  const int lane = threadIdx.x & 63;
  const int i = i0 + (lane & 31), j = j0 + (lane & 31);
  f32x16 acc = {};
  const int npairs = 2 + g.pair_count;
  for (int pair = 0; pair < npairs; ++pair) {
    const PairView v = pair_view(g, extra, pair, st);
    for (int k0 = 0; k0 < v.K; k0 += 2) {
      const int k = k0 + (lane >> 5);
      float a = 0.f, b = 0.f;
      const int e0 = pair == 1 ? 2 : 0;
      if (i < g.M && k < v.K)
        a = g.trans & GEMM_PRE_A ? load_piece(v.A + i * v.lda * 4, k, pow2f(-exp_of(g.exps, e0)))
                                 : load_as_f32(v.A, v.atr ? k * v.lda + i : i * v.lda + k, g.a_dtype);
      if (j < g.N && k < v.K)
        b = g.trans & GEMM_PRE_B ? load_piece(v.B + j * v.ldb * 4, k, pow2f(-exp_of(g.exps, e0 + 1)))
                                 : load_as_f32(v.B, v.btr ? k * v.ldb + j : j * v.ldb + k, g.b_dtype);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
    }
  }
  return acc;
}

// MODE: the operands of every tile of the launch are GEMM_ROWS all fp32 and
// row-major ([M][K]), GEMM_KMAJOR all fp32, stored [K][M] and with M and N
// multiples of four, GEMM_ANY fp32 or bf16 in either order.  A thread loads
// 8 values of each operand per step: 8 consecutive k of one row, or (stored
// k-major) 4 consecutive rows of 2 k.  In the first two modes the whole
// steps of all pairs run through the pipeline without a branch around their
// loads (rows past the end re-read the last ones: their results are not
// stored), and what is left of each pair's K follows, value by value;
// GEMM_ANY loads every step that way, as vectors where it can.
// PRE: operands stored as half pieces (whole steps only: K a multiple of 32)
// go to LDS as they are; the epilogue is then that of the lists which use
// them (GEMM_PRE_RIGHT: updates, GEMM_PRE_BOTH: Gram, S' and series items).
template <int SC, int BM, int MODE, int PRE = GEMM_PRE_NONE>
__global__ __launch_bounds__(BM == 64 ? 256 : 512, 2) void gemm_f32_kernel(const GemmItem* __restrict__ items,
                                                                           const GemmTile* __restrict__ tiles,
                                                                           int step,
                                                                           const GemmPair* __restrict__ extra) {
  using S = Split<SC>;
  constexpr int P = S::P, BK = 32, CH = BK / 8;
  constexpr int WM = 2, WN = BM == 64 ? 2 : 4;          // waves
  constexpr int MI = BM / WM / 32, NI = BM / WN / 32;   // 32 x 32 blocks per wave
  static_assert(64 * WM * WN * 8 == BM * BK, "eight values of each operand per thread and step");
  extern __shared__ __attribute__((aligned(16))) uint4 smem[];   // [stage][operand][piece][BM rows][CH chunks]
  const GemmTile tl = tiles[blockIdx.x];
  const GemmItem item = items[tl.item];   // (whole: its fields arrive together)
  const int M = item.M, N = item.N;
  const int row0 = tl.ti * BM, col0 = tl.tj * BM;
  const bool mirror = item.mirror != 0 && tl.ti != tl.tj;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int64_t st = step;
  const int adt = MODE == GEMM_ANY ? item.a_dtype : ORTH_F32, bdt = MODE == GEMM_ANY ? item.b_dtype : ORTH_F32;

  // chunk c (8 values of k) of row r lives at c ^ swz(r): the fragment reads
  // (one row per lane) and the row-major stores are conflict free
  auto swz = [](int r) { return ((r >> 1) & 3) ^ ((r >> 3) & 1); };
  auto plane = [&](int s, int o, int p) { return smem + ((s * 2 + o) * P + p) * (BM * CH); };
  // this thread's values: row-major (row rr, k 8 rc ..; whole cache lines per
  // load, 4 k of two rows, were no faster), k-major (rows tr .. tr + 3, k tk
  // and tk + 1)
  const int rr = tid / CH, rc = tid % CH;
  const int tr = (tid % (BM / 4)) * 4, tk = (tid / (BM / 4)) * 2;
  const int exps = SC == GEMM_F16X2 ? item.exps : 0;

  uint4 raw[2][2][2];      // [register set][operand][half]
  float scl[2][2];
  PairView pv;
  uint32_t voff[2];        // this thread's byte offset from the step's first value (row strides up to 2^23)
  const char* at[2];       // the step's first value of the tile's rows
  int64_t astep[2];
  int pair = -1, left = 0; // whole steps of the pair that are not loaded yet
  float psc[2] = {1.f, 1.f};
  const int npairs = 2 + item.pair_count;
  // moves to the next whole step, pair after pair; false past the last
  auto next = [&]() -> bool {
    if (--left > 0) {
      at[0] += astep[0];
      at[1] += astep[1];
      return true;
    }
    int k = 0;
    while (k < BK) {
      if (++pair >= npairs) return false;
      k = pair == 0 ? item.K : pair == 1 ? item.K2 : extra[item.pair_base + (pair - 2)].K;
    }
    left = k / BK;
    pv = pair_view(item, extra, pair, st);
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int64_t ld = o ? pv.ldb : pv.lda;
      const int base = o ? col0 : row0, last = (o ? N : M) - base;   // rows of this tile that exist
      if (MODE == GEMM_KMAJOR) {
        at[o] = (o ? pv.B : pv.A) + (int64_t)base * 4;
        voff[o] = (uint32_t)((tk * ld + (tr + 4 <= last ? tr : last - 4)) * 4);
        astep[o] = ld * BK * 4;
      } else {
        at[o] = (o ? pv.B : pv.A) + base * ld * 4;
        voff[o] = (uint32_t)(((rr < last ? rr : last - 1) * ld + rc * 8) * 4);
        astep[o] = BK * 4;
      }
      psc[o] = S::scale(exp_of(exps, (pair == 1 ? 2 : 0) + o));
    }
    return true;
  };
  auto load = [&](int set) {
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const char* p = at[o] + voff[o];
      raw[set][o][0] = gld_u32x4_a4(reinterpret_cast<const float*>(p));
      raw[set][o][1] = gld_u32x4_a4(
          reinterpret_cast<const float*>(MODE == GEMM_KMAJOR ? p + (o ? pv.ldb : pv.lda) * 4 : p + 16));
      scl[set][o] = psc[o];
    }
  };
  // a thread's values of operand o -> the pieces in LDS stage s
  auto split_store = [&](const float (&x)[8], float sc, bool tro, int s, int o) {
    uint32_t w[4][P];
    if (tro) {
      // k pairs (tk, tk + 1) of the four rows
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        S::split2(x[j], x[j + 4], sc, w[j]);
        const int r = tr + j;
        const int dst = (r * CH + ((tk >> 3) ^ swz(r))) * 4 + ((tk & 7) >> 1);
#pragma unroll
        for (int i = 0; i < P; ++i) reinterpret_cast<uint32_t*>(plane(s, o, i))[dst] = w[j][i];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) S::split2(x[2 * j], x[2 * j + 1], sc, w[j]);
      const int dst = rr * CH + (rc ^ swz(rr));
#pragma unroll
      for (int i = 0; i < P; ++i) plane(s, o, i)[dst] = make_uint4(w[0][i], w[1][i], w[2][i], w[3][i]);
    }
  };
  auto stage = [&](int set, int s, int o) {
    const uint4 a = raw[set][o][0], b = raw[set][o][1];
    if (PRE == GEMM_PRE_BOTH || (PRE == GEMM_PRE_RIGHT && o == 1)) {
      // (8 h, then 8 l)
      const int dst = rr * CH + (rc ^ swz(rr));
      plane(s, o, 0)[dst] = a;
      plane(s, o, 1)[dst] = b;
      return;
    }
    const float x[8] = {__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(a.z), __uint_as_float(a.w),
                        __uint_as_float(b.x), __uint_as_float(b.y), __uint_as_float(b.z), __uint_as_float(b.w)};
    split_store(x, scl[set][o], MODE == GEMM_KMAJOR, s, o);
  };
  // the step at k0 of pair v, whole or not, into stage s: guarded loads
  auto stage_guarded = [&](const PairView& v, int pr, int k0, int s) {
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const char* ptr = o ? v.B : v.A;
      const int64_t ld = o ? v.ldb : v.lda;
      const bool tro = MODE == GEMM_KMAJOR || (MODE == GEMM_ANY && (o ? v.btr : v.atr) != 0);
      const int dt = o ? bdt : adt, base = o ? col0 : row0, lim = o ? N : M;
      float x[8];
      if (MODE == GEMM_ANY && k0 + BK <= v.K && dt == ORTH_F32 && (!tro || base + BM <= lim || lim % 4 == 0)) {
        const int r = tro ? (base + tr + 4 <= lim ? base + tr : lim - 4) : (base + rr < lim ? base + rr : lim - 1);
        const float* p = reinterpret_cast<const float*>(ptr) +
                         (tro ? (int64_t)(k0 + tk) * ld + r : (int64_t)r * ld + k0 + rc * 8);
        const uint4 a = gld_u32x4_a4(p), b = gld_u32x4_a4(tro ? p + ld : p + 4);
        x[0] = __uint_as_float(a.x); x[1] = __uint_as_float(a.y); x[2] = __uint_as_float(a.z);
        x[3] = __uint_as_float(a.w); x[4] = __uint_as_float(b.x); x[5] = __uint_as_float(b.y);
        x[6] = __uint_as_float(b.z); x[7] = __uint_as_float(b.w);
      } else if (MODE == GEMM_ANY && k0 + BK <= v.K && dt == ORTH_BF16 && !tro && vec8_ok(ptr, ld, ORTH_BF16)) {
        load8_f32(ptr, (int64_t)(base + rr < lim ? base + rr : lim - 1) * ld + k0 + rc * 8, ORTH_BF16, x);
      } else {
        // (raw bits first: a conversion inside the guarded load would make
        // every load wait for its data)
        uint32_t w[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int r = base + (tro ? tr + (q & 3) : rr), k = k0 + (tro ? tk + (q >> 2) : rc * 8 + q);
          w[q] = 0;
          if (r < lim && k < v.K) {
            const int64_t e = tro ? (int64_t)k * ld + r : (int64_t)r * ld + k;
            w[q] = dt == ORTH_BF16 ? (uint32_t)gld_u16(ptr, e) : gld_u32(ptr, e);
          }
        }
        const int sh = dt == ORTH_BF16 ? 16 : 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          asm volatile("" : "+v"(w[q]));
          x[q] = __uint_as_float(w[q] << sh);
        }
      }
      split_store(x, S::scale(exp_of(exps, (pr == 1 ? 2 : 0) + o)), tro, s, o);
    }
  };

  f32x16 acc[2][MI][NI];   // the leading products, the corrections
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[q][i][j] = f32x16{};
  struct Frags {
    uint4 a[MI][P], b[NI][P];
  };
  // the fragments of half kk (16 k) of the step in LDS stage buf
  auto read_frags = [&](int buf, int kk, Frags& f) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int r = wm * (BM / WM) + i * 32 + (lane & 31);
        f.a[i][p] = plane(buf, 0, p)[r * CH + ((2 * kk + (lane >> 5)) ^ swz(r))];
      }
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int r = wn * (BM / WN) + j * 32 + (lane & 31);
        f.b[j][p] = plane(buf, 1, p)[r * CH + ((2 * kk + (lane >> 5)) ^ swz(r))];
      }
    }
  };
  auto mfmas = [&](const Frags& f) {
#pragma unroll
    for (int q = 0; q < S::NP; ++q)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          f32x16& t = acc[q < S::NP - 1][i][j];
          t = S::mma(f.a[i][S::pa(q)], f.b[j][S::pb(q)], t);
        }
  };
  // The pipeline.  Step t's halves lie in LDS stage t & 1.  First half: the
  // second half's fragments are read, operand B of step t + 1 is split into
  // the other stage.  Then a barrier: step t + 1 is complete and nobody
  // reads step t's stage any more.  Second half: step t + 1's first
  // fragments are read, operand A of step t + 2 is split into step t's
  // stage.  So the MFMAs of each half have LDS reads and VALU work beside
  // them, and the loads of step t + 3, issued at the barrier, a whole step
  // to land.  Past the last step the same work runs on stale values that
  // nothing uses.
  Frags f0, f1;
  int loaded = 0;   // steps whose loads have been issued
  // (past the last step the loads re-read it: a branch around them would
  // make every later wait count as if they had not been issued)
  auto fetch = [&](int set) {
    loaded += next();
    load(set);
  };
  auto body = [&](int buf) {
    read_frags(buf, 1, f1);
    stage(buf ^ 1, buf ^ 1, 1);
    mfmas(f0);
    __syncthreads();
    fetch(buf ^ 1);
    read_frags(buf ^ 1, 0, f0);
    stage(buf, buf, 0);
    mfmas(f1);
  };
  // an update's old values, on their way during the products
  float src_v[MI][NI][PRE == GEMM_PRE_RIGHT ? 16 : 1];
  if constexpr (PRE == GEMM_PRE_RIGHT) {
    const float* src = item.src + item.src_step * st;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int a = row0 + wm * (BM / WM) + i * 32 + acc_row(r, lane);
          const int b = col0 + wn * (BM / WN) + j * 32 + (lane & 31);
          src_v[i][j][r] = gld_f32(src, (int64_t)(a < M ? a : M - 1) * item.ld_src + (b < N ? b : N - 1));
        }
  }
  if constexpr (MODE != GEMM_ANY) {
    if (next()) {
      loaded = 1;
      load(0);
      fetch(1);
      stage(0, 0, 0);
      stage(0, 0, 1);
      fetch(0);
      stage(1, 1, 0);
      __syncthreads();
      read_frags(0, 0, f0);
      for (int t = 0; t < loaded; t += 2) {
        body(0);
        if (t + 1 >= loaded) break;
        body(1);
      }
      __syncthreads();
    }
  }
  // what the pipeline left (every wave is past the pipeline)
  if constexpr (PRE == GEMM_PRE_NONE) {
    int s = 0;
    for (int p = 0; p < npairs; ++p) {
      const PairView v = pair_view(item, extra, p, st);
      for (int k0 = MODE == GEMM_ANY ? 0 : v.K / BK * BK; k0 < v.K; k0 += BK, s ^= 1) {
        stage_guarded(v, p, k0, s);
        __syncthreads();
        for (int kk = 0; kk < BK / 16; ++kk) {
          read_frags(s, kk, f0);
          mfmas(f0);
        }
      }
    }
    __syncthreads();   // the epilogue reuses LDS
  }

  // ------------------------------------------------------------ epilogue --
  const float out_s = SC == GEMM_F16X2 ? S::scale(-(exp_of(exps, 0) + exp_of(exps, 1))) : 1.f;
  bool bad = false;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float v = (acc[0][i][j][r] + S::CORR * acc[1][i][j][r]) * out_s;
        acc[0][i][j][r] = v;
        bad |= !isfinite(v);
      }
  if (__builtin_expect(__any(bad), 0)) {
    // every row of the wave's part of A starts with a NaN: so does the
    // fp32 result (a matrix that is NaN throughout)
    bool all_nan = true;
    for (int i = 0; i < MI; ++i) {
      const int r = row0 + wm * (BM / WM) + i * 32 + (lane & 31);
      if (r < M && item.K > 0) {
        const PairView v = pair_view(item, extra, 0, st);
        const float a = PRE == GEMM_PRE_BOTH ? load_piece(v.A + r * v.lda * 4, 0, 1.f)
                                             : load_as_f32(v.A, v.atr ? r : r * v.lda, item.a_dtype);
        all_nan &= isnan(a);
      } else if (r < M) {
        all_nan = false;
      }
    }
    if (!__all(all_nan)) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
          acc[0][i][j] = block_f32(item, extra, st, row0 + wm * (BM / WM) + i * 32, col0 + wn * (BM / WN) + j * 32);
    }
  }

  if constexpr (PRE != GEMM_PRE_NONE) {
    // Results that later products read as pieces are written 8 values (32
    // bytes) at a time from a 32 x 33 region of LDS per wave, which holds a
    // block's rows in one orientation and then the other.
    float* Tt = reinterpret_cast<float*>(smem) + wave * (32 * 33);
    const float po = pow2f((int)((uint32_t)item.trans << 16) >> 24);
    auto wave_sync = [&]() {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    // the block's values, `t` of this lane's column, to rows [r0, r0 + 32)
    // x columns [c0, c0 + 32) of dst (limits rl, cl; zero past czero)
    auto put_pieces = [&](const float (&t)[16], bool flip, float* dst, int64_t ld, int r0, int c0, int rl, int cl,
                          int czero) {
      wave_sync();
#pragma unroll
      for (int r = 0; r < 16; ++r)
        Tt[flip ? (lane & 31) * 33 + acc_row(r, lane) : acc_row(r, lane) * 33 + (lane & 31)] = t[r];
      wave_sync();
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int e = q * 64 + lane, r = e >> 2, c = (e & 3) * 8;
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = c0 + c + k < czero ? Tt[r * 33 + c + k] : 0.f;
        if (r0 + r < rl && c0 + c < cl) store_pieces8(dst + (int64_t)(r0 + r) * ld + c0 + c, v, po);
      }
    };
#pragma unroll
    for (int bi = 0; bi < MI; ++bi)
#pragma unroll
      for (int bj = 0; bj < NI; ++bj) {
        const f32x16& v = acc[0][bi][bj];
        const int ibase = row0 + wm * (BM / WM) + bi * 32, jbase = col0 + wn * (BM / WN) + bj * 32;
        const int j = jbase + (lane & 31);
        float* C = static_cast<float*>(item.C) + item.c_step * st;
        const int64_t ldc = item.ldc;
        float t[16];
        if constexpr (PRE == GEMM_PRE_RIGHT) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int i = ibase + acc_row(r, lane);
            t[r] = src_v[bi][bj][r] + item.beta * v[r];
            if (i < M && j < N) gst_f32(C, (int64_t)i * ldc + j, t[r]);
          }
          if (item.dst2) put_pieces(t, true, item.dst2 + item.d2_step * st, item.ld2, jbase, ibase, N, M, M);
        } else if (item.epi == EPI_SERIES) {
          const float g = pow2f(item.src ? series_exp(gld_f32(item.src, 0)) : 0);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int i = ibase + acc_row(r, lane);
            t[r] = item.beta * g * v[r];
            // each element belongs to one item of the launch
            if (i < M && j < N)
              gst_f32(item.dst2, (int64_t)i * item.ld2 + j, gld_f32(item.dst2, (int64_t)i * item.ld2 + j) + t[r] * g);
          }
          if (C) put_pieces(t, false, C, ldc, ibase, jbase, M, (int)ldc, N);
        } else {   // EPI_GRAM_E, EPI_NEG
          const float one = item.epi == EPI_GRAM_E ? 1.f : 0.f;
#pragma unroll
          for (int r = 0; r < 16; ++r) t[r] = (ibase + acc_row(r, lane) == j ? one : 0.f) - v[r];
          put_pieces(t, false, C, ldc, ibase, jbase, M, N, N);
          if (mirror) put_pieces(t, true, C, ldc, jbase, ibase, N, M, M);
        }
      }
    return;
  }
  const int epi = item.epi;
  float dev = 0.f;
#pragma unroll
  for (int bi = 0; bi < MI; ++bi)
#pragma unroll
    for (int bj = 0; bj < NI; ++bj) {
      const f32x16& v = acc[0][bi][bj];
      const int ibase = row0 + wm * (BM / WM) + bi * 32, jbase = col0 + wn * (BM / WN) + bj * 32;
      const int j = jbase + (lane & 31);
      float* C = static_cast<float*>(item.C) + item.c_step * st;
      const int64_t ldc = item.ldc;
      if (epi == EPI_MAXDEV) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = ibase + acc_row(r, lane);
          if (i < M && j < N) {
            const float d = fabsf((i == j ? 1.f : 0.f) - v[r]);
            dev = (d > dev || isnan(d)) ? d : dev;
          }
        }
      } else if (epi == EPI_STORE) {
        const int cdt = item.c_dtype;
        void* Cv = static_cast<char*>(item.C) + item.c_step * st * (cdt == ORTH_BF16 ? 2 : 4);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = ibase + acc_row(r, lane);
          if (i < M && j < N) store_from_f32(Cv, (int64_t)i * ldc + j, cdt, v[r]);
        }
      } else if (epi == EPI_GRAM_E || epi == EPI_NEG) {
        // 1 or 0 on the diagonal; the mirrored tile in runs of four (a
        // lane's rows come in fours)
        const float one = epi == EPI_GRAM_E ? 1.f : 0.f;
        float e[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = ibase + acc_row(r, lane);
          e[r] = (i == j ? one : 0.f) - v[r];
          if (i < M && j < N) gst_f32(C, (int64_t)i * ldc + j, e[r]);
        }
        if (mirror && j < N) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int i = ibase + acc_row(4 * q, lane);
            float* d = C + (int64_t)j * ldc + i;
            if (i + 4 <= M && (reinterpret_cast<uintptr_t>(d) & 15) == 0) {
              gst_f32x4(d, make_float4(e[4 * q], e[4 * q + 1], e[4 * q + 2], e[4 * q + 3]));
            } else {
#pragma unroll
              for (int k = 0; k < 4; ++k)
                if (i + k < M) gst_f32(d, k, e[4 * q + k]);
            }
          }
        }
      } else {  // EPI_UPDATE
        const float* src = item.src + item.src_step * st;
        float* dst2 = item.dst2 ? item.dst2 + item.d2_step * st : nullptr;
        const int64_t lds_ = item.ld_src, ld2 = item.ld2;
        const float beta = item.beta;
        float u[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = ibase + acc_row(r, lane);
          u[r] = i < M && j < N ? gld_f32(src, (int64_t)i * lds_ + j) : 0.f;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = ibase + acc_row(r, lane);
          if (i < M && j < N) {
            u[r] += beta * v[r];
            gst_f32(C, (int64_t)i * ldc + j, u[r]);
          }
        }
        if (dst2) {
          // the wave's 32 x 32 block transposed through LDS (a 32 x 33
          // region of its own; the stages are free after the last k-step's
          // barrier), so that every row of the copy is written as 16-byte
          // pieces
          float* Tt = reinterpret_cast<float*>(smem) + wave * (32 * 33);
#pragma unroll
          for (int r = 0; r < 16; ++r) Tt[(lane & 31) * 33 + acc_row(r, lane)] = u[r];
          __syncthreads();
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int e = q * 64 + lane;
            const int jj = e >> 3, c4 = (e & 7) * 4;
            const int gj = jbase + jj, gi = ibase + c4;
            if (gj >= N) continue;
            const float* t = Tt + jj * 33 + c4;
            float* d = dst2 + (int64_t)gj * ld2 + gi;
            if (gi + 4 <= M && (reinterpret_cast<uintptr_t>(d) & 15) == 0) {
              gst_f32x4(d, make_float4(t[0], t[1], t[2], t[3]));
            } else {
#pragma unroll
              for (int k = 0; k < 4; ++k)
                if (gi + k < M) gst_f32(d, k, t[k]);
            }
          }
          __syncthreads();
        }
      }
    }
  if (epi == EPI_MAXDEV) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const float o = __shfl_xor(dev, off, 64);
      dev = (o > dev || isnan(o)) ? o : dev;
    }
    if (lane == 0) atomicMax(reinterpret_cast<unsigned int*>(item.red), __float_as_uint(dev));
  }
}

template <int SC, int BM, int MODE, int PRE = GEMM_PRE_NONE>
hipError_t launch_one(const GemmItem* items, const GemmTile* tiles, int n, int step, const GemmPair* pairs,
                      hipStream_t s) {
  if (n <= 0) return hipSuccess;
  // two stages of two operands (the update epilogue needs less); above the
  // default limit with three pieces and 128-tiles
  constexpr int lds = 2 * 2 * Split<SC>::P * BM * 32 * 2;
  if constexpr (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_f32_kernel<SC, BM, MODE, PRE>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((gemm_f32_kernel<SC, BM, MODE, PRE>), dim3(n), dim3(BM == 64 ? 256 : 512), lds, s, items, tiles, step,
                     pairs);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_f32(const GemmItem* items, const GemmTile* tiles, const GemmRun& run, const char* name,
                           hipStream_t s, int step, const GemmPair* pairs) {
  const int n = run.n[GEMM_ROWS] + run.n[GEMM_KMAJOR] + run.n[GEMM_ANY];
  if (n <= 0) return hipSuccess;
  timing_begin(name, s);
  hipError_t e = hipSuccess;
  const GemmTile* t = tiles;
  if (run.split == GEMM_F16X2) {
    // only row-major products are planned with two pieces
    const bool big = run.tile == 128;
    if (run.n[GEMM_ROWS] != n)
      e = hipErrorInvalidValue;
    else if (run.pre == GEMM_PRE_RIGHT)
      e = big ? launch_one<GEMM_F16X2, 128, GEMM_ROWS, GEMM_PRE_RIGHT>(items, t, n, step, pairs, s)
              : launch_one<GEMM_F16X2, 64, GEMM_ROWS, GEMM_PRE_RIGHT>(items, t, n, step, pairs, s);
    else
      e = big ? launch_one<GEMM_F16X2, 128, GEMM_ROWS, GEMM_PRE_BOTH>(items, t, n, step, pairs, s)
              : launch_one<GEMM_F16X2, 64, GEMM_ROWS, GEMM_PRE_BOTH>(items, t, n, step, pairs, s);
  } else {
    const bool big = run.tile == 128;
    e = big ? launch_one<GEMM_BF16X3, 128, GEMM_ROWS>(items, t, run.n[GEMM_ROWS], step, pairs, s)
            : launch_one<GEMM_BF16X3, 64, GEMM_ROWS>(items, t, run.n[GEMM_ROWS], step, pairs, s);
    t += run.n[GEMM_ROWS];
    if (e == hipSuccess)
      e = big ? launch_one<GEMM_BF16X3, 128, GEMM_KMAJOR>(items, t, run.n[GEMM_KMAJOR], step, pairs, s)
              : launch_one<GEMM_BF16X3, 64, GEMM_KMAJOR>(items, t, run.n[GEMM_KMAJOR], step, pairs, s);
    t += run.n[GEMM_KMAJOR];
    if (e == hipSuccess)
      e = big ? launch_one<GEMM_BF16X3, 128, GEMM_ANY>(items, t, run.n[GEMM_ANY], step, pairs, s)
              : launch_one<GEMM_BF16X3, 64, GEMM_ANY>(items, t, run.n[GEMM_ANY], step, pairs, s);
  }
  timing_end(name, s);
  return e;
}

}  // namespace orth
