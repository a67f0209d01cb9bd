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
// into three bfloat16 pieces x = h + m + l (split2_bf16: all 24 bits, fp32's
// exponents), and hh + hm + mh + hl + lh + mm run on the 16-bit matrix cores
// (16 times the fp32 MFMA rate) with fp32 accumulation; the products left
// out are below 2^-25 of hh.  The leading product and the corrections have
// an accumulator each: a correction's rounding then no longer happens at the
// size of the whole sum.  Relative error against 64 bits, normal operands, K
// = 64 / 512 / 4096: fp32 MFMA 1.4e-7 / 4.1e-7 / 1.2e-6, this 5.0e-8 /
// 1.3e-7 / 4.0e-7 (one accumulator for all: 1.1e-7 / 3.4e-7 / 1.0e-6).  Two
// half pieces take half the products, but 22 bits and half's range: light
// rows and columns beside heavy ones lost theirs.
//
// A wave's block with a result that the split cannot give (split_failed:
// infinities, NaN, overflow, values near the low end of fp32) is computed
// again with fp32 MFMA by the wave that meets it, straight from memory.
// Conv exponentials of 256 channels: 0.89 ms, 1.36 with one NaN in the kernel
// (1.23 when every tile ran on fp32 MFMA; a vote of the workgroup and LDS
// staging took 1.80, and 0.2 us more of every launch).
//
// Lists with a 128-tile for every compute unit use those (half the splitting
// and LDS writes per product), others 64.
//
// What bounds it: with 128-tiles (exponential map of 4 x 2048^2) the matrix
// pipes are busy 53% of the cycles, at a clock of 1.83 GHz, beside VALU
// instructions (the splitting) in 37% of the issue cycles; the two waves of a
// SIMD wait 32% of their time for loads and barriers.
// 64-tile lists have one or two waves a SIMD and pipes that are busy 20 to
// 26%: one tile's first loads, K loop and epilogue.  Measured with fp32 MFMA
// and now: exponential map of 4 x 2048^2, 674 -> 410 us per power (102 -> 168
// TFLOP/s); conv exponential of 512 channels, 1379 -> 849 us per power (100 ->
// 162); Gram matrix and update of a 2048 x 1024 iterate 65 -> 42 and 59 -> 42
// us, of eight 512^2 ones 32 -> 22.5 and 36 -> 26.7.
//
// K advances in steps of 32 through two LDS stages (see the pipeline below).
#include "internal.h"

namespace orth {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

namespace {

__device__ inline int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// 16 bytes from any 4-byte aligned global address (gfx950 needs no more for
// multi-dword accesses)
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2u __attribute__((ext_vector_type(2), aligned(2)));   // (or 2-byte aligned)
__device__ __forceinline__ uint4 gld_u32x4_a4(const float* p) {
  const u32x4u v = *(const ORTH_GLOBAL u32x4u*)p;
  return make_uint4(v.x, v.y, v.z, v.w);
}

constexpr int P = 3, NP = 6;   // pieces, products (smallest first, the leading one last)
__device__ constexpr int prod_a(int q) { return q == 0 ? 2 : q == 2 || q == 3 ? 1 : 0; }
__device__ constexpr int prod_b(int q) { return q == 1 ? 2 : q == 2 || q == 4 ? 1 : 0; }
__device__ __forceinline__ f32x16 mma(uint4 a, uint4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

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

// The wave's 32 x 32 block at (i0, j0) with fp32 MFMA: the blocks whose split
// result fails.  16 k at a time straight from memory (the lower lanes hold
// the first eight, the upper ones the others), the next 16 on their way;
// done early where every value is NaN already.
__device__ __forceinline__ f32x16 block_f32(const GemmItem& g, const GemmPair* extra, int64_t st, int i0,
                                            int j0) {
  const int lane = threadIdx.x & 63, kh = 8 * (lane >> 5);
  f32x16 acc = {};
  const int npairs = 2 + g.pair_count;
#pragma unroll 1
  for (int pair = 0; pair < npairs; ++pair) {
    const PairView v = pair_view(g, extra, pair, st);
    const char* at[2];       // the next of this lane's values
    int64_t ks[2];           // bytes between them
    bool in[2], narrow[2];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int row = (o ? j0 : i0) + (lane & 31);
      const int64_t ld = o ? v.ldb : v.lda;
      const bool tr = (o ? v.btr : v.atr) != 0;
      narrow[o] = (o ? g.b_dtype : g.a_dtype) == ORTH_BF16;
      in[o] = row < (o ? g.N : g.M);
      const int64_t vb = narrow[o] ? 2 : 4;
      ks[o] = (tr ? ld : 1) * vb;
      at[o] = (o ? v.B : v.A) + (in[o] ? tr ? row * vb : row * ld * vb : 0) + kh * ks[o];
    }
    uint32_t w[2][8];
    // the values of the step at k, as they are stored; zeros past the end
    // (rows past it re-read the first one: their results are not stored)
    auto load = [&](int k) {
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        if (k + 16 <= v.K && ks[o] == 4 && !narrow[o]) {
          const uint4 a = gld_u32x4_a4(reinterpret_cast<const float*>(at[o]));
          const uint4 b = gld_u32x4_a4(reinterpret_cast<const float*>(at[o]) + 4);
          w[o][0] = a.x; w[o][1] = a.y; w[o][2] = a.z; w[o][3] = a.w;
          w[o][4] = b.x; w[o][5] = b.y; w[o][6] = b.z; w[o][7] = b.w;
        } else {
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            w[o][q] = 0;
            if (in[o] && k + kh + q < v.K)
              w[o][q] = narrow[o] ? (uint32_t)gld_u16(at[o] + q * ks[o], 0) : gld_u32(at[o] + q * ks[o], 0);
          }
        }
        at[o] += 16 * ks[o];
      }
    };
    load(0);
#pragma unroll 1
    for (int k0 = 0; k0 < v.K; k0 += 16) {
      float x[2][8];
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int q = 0; q < 8; ++q) x[o][q] = __uint_as_float(w[o][q] << (narrow[o] ? 16 : 0));
      load(k0 + 16);
#pragma unroll
      for (int q = 0; q < 8; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[0][q], x[1][q], acc, 0, 0, 0);
      if (k0 % 128 == 0 && __all(all_nan(acc))) return acc;
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
template <int BM, int MODE>
__global__ __launch_bounds__(BM == 64 ? 256 : 512, 2) void gemm_f32_kernel(const GemmItem* __restrict__ items,
                                                                           const GemmTile* __restrict__ tiles,
                                                                           int step,
                                                                           const GemmPair* __restrict__ extra) {
  constexpr int BK = 32, CH = BK / 8;
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

  uint4 raw[2][2][2];      // [register set][operand][half]
  PairView pv;
  uint32_t voff[2];        // this thread's byte offset from the step's first value (row strides up to 2^23)
  const char* at[2];       // the step's first value of the tile's rows
  int64_t astep[2];
  int pair = -1, left = 0; // whole steps of the pair that are not loaded yet
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
    }
  };
  // a thread's values of operand o -> the pieces in LDS stage s
  auto split_store = [&](const float (&x)[8], bool tro, int s, int o) {
    uint32_t w[4][P];
    if (tro) {
      // k pairs (tk, tk + 1) of the four rows
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        split2_bf16(x[j], x[j + 4], w[j][0], w[j][1], w[j][2]);
        const int r = tr + j;
        const int dst = (r * CH + ((tk >> 3) ^ swz(r))) * 4 + ((tk & 7) >> 1);
#pragma unroll
        for (int i = 0; i < P; ++i) reinterpret_cast<uint32_t*>(plane(s, o, i))[dst] = w[j][i];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) split2_bf16(x[2 * j], x[2 * j + 1], w[j][0], w[j][1], w[j][2]);
      const int dst = rr * CH + (rc ^ swz(rr));
#pragma unroll
      for (int i = 0; i < P; ++i) plane(s, o, i)[dst] = make_uint4(w[0][i], w[1][i], w[2][i], w[3][i]);
    }
  };
  auto stage = [&](int set, int s, int o) {
    const uint4 a = raw[set][o][0], b = raw[set][o][1];
    const float x[8] = {__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(a.z), __uint_as_float(a.w),
                        __uint_as_float(b.x), __uint_as_float(b.y), __uint_as_float(b.z), __uint_as_float(b.w)};
    split_store(x, MODE == GEMM_KMAJOR, s, o);
  };
  // What the pipeline leaves: this thread's values of operand o at k0 of pair
  // v, a whole step or not (zeros past the end), as they are stored: words of
  // fp32, of one bfloat16 each, or (four words) of two.
  enum { WORDS_F32, WORDS_BF16, WORDS_2BF16 };
  auto k_major = [&](const PairView& v, int o) {
    return MODE == GEMM_KMAJOR || (MODE == GEMM_ANY && (o ? v.btr : v.atr) != 0);
  };
  auto load_guarded = [&](const PairView& v, int k0, int o, uint32_t (&w)[8]) -> int {
    const char* ptr = o ? v.B : v.A;
    const int64_t ld = o ? v.ldb : v.lda;
    const bool tro = k_major(v, o);
    const int dt = o ? bdt : adt, base = o ? col0 : row0, lim = o ? N : M;
    if (MODE == GEMM_ANY && k0 + BK <= v.K && (!tro || base + BM <= lim || lim % 4 == 0)) {
      const int r = tro ? (base + tr + 4 <= lim ? base + tr : lim - 4) : (base + rr < lim ? base + rr : lim - 1);
      const int64_t e = tro ? (int64_t)(k0 + tk) * ld + r : (int64_t)r * ld + k0 + rc * 8;
      if (dt == ORTH_F32) {
        const float* p = reinterpret_cast<const float*>(ptr) + e;
        const uint4 a = gld_u32x4_a4(p), b = gld_u32x4_a4(tro ? p + ld : p + 4);
        w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w;
        w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
        return WORDS_F32;
      }
      const uint16_t* p = reinterpret_cast<const uint16_t*>(ptr) + e;
      const u32x2u a = *(const ORTH_GLOBAL u32x2u*)p, b = *(const ORTH_GLOBAL u32x2u*)(tro ? p + ld : p + 4);
      w[0] = a.x; w[1] = a.y; w[2] = b.x; w[3] = b.y;
      return WORDS_2BF16;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int r = base + (tro ? tr + (q & 3) : rr), k = k0 + (tro ? tk + (q >> 2) : rc * 8 + q);
      w[q] = 0;
      if (r < lim && k < v.K) {
        const int64_t e = tro ? (int64_t)k * ld + r : (int64_t)r * ld + k;
        w[q] = dt == ORTH_BF16 ? (uint32_t)gld_u16(ptr, e) : gld_u32(ptr, e);
      }
    }
    return dt == ORTH_BF16 ? WORDS_BF16 : WORDS_F32;
  };
  // those words -> LDS stage s (of two bfloat16 the leading piece alone: the
  // products of the others are left out)
  auto store_guarded = [&](const uint32_t (&w)[8], int form, bool tro, int s, int o) {
    if (MODE == GEMM_ANY && form == WORDS_2BF16) {
      if (!tro) {
        plane(s, o, 0)[rr * CH + (rc ^ swz(rr))] = make_uint4(w[0], w[1], w[2], w[3]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = tr + j, dst = (r * CH + ((tk >> 3) ^ swz(r))) * 4 + ((tk & 7) >> 1);
          const uint32_t a = w[j >> 1], b = w[2 + (j >> 1)];
          reinterpret_cast<uint32_t*>(plane(s, o, 0))[dst] =
              j & 1 ? (a >> 16) | (b & 0xffff0000u) : (a & 0xffffu) | (b << 16);
        }
      }
      return;
    }
    const int sh = form == WORDS_BF16 ? 16 : 0;
    float x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      uint32_t u = w[q];
      asm volatile("" : "+v"(u));   // (no conversion inside the guarded load: it would wait for each)
      x[q] = __uint_as_float(u << sh);
    }
    split_store(x, tro, s, o);
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
  // (bfloat16 operands are their own leading piece)
  const bool a_one = MODE == GEMM_ANY && adt == ORTH_BF16, b_one = MODE == GEMM_ANY && bdt == ORTH_BF16;
  auto mfmas = [&](const Frags& f) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      if ((a_one && prod_a(q) > 0) || (b_one && prod_b(q) > 0)) continue;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          f32x16& t = acc[q < NP - 1][i][j];
          t = mma(f.a[i][prod_a(q)], f.b[j][prod_b(q)], t);
        }
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
  {
    int s = 0;
    for (int p = 0; p < npairs; ++p) {
      const PairView v = pair_view(item, extra, p, st);
      for (int k0 = MODE == GEMM_ANY ? 0 : v.K / BK * BK; k0 < v.K; k0 += BK, s ^= 1) {
#pragma unroll
        for (int o = 0; o < 2; ++o) {
          uint32_t w[8];
          const int form = load_guarded(v, k0, o, w);
          store_guarded(w, form, k_major(v, o), s, o);
        }
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
  // (Series are not asked: a small power comes from operands in range, and one
  // below 2^-110 loses 2^-134 at most.  Conv exponentials of 256 channels,
  // entries of 1e-8: 1.90 ms asked, 0.80 not.)
  const float lo = item.epi == EPI_SERIES ? 0.f : kSplitLo;
  bool bad = false;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      acc[0][i][j] += acc[1][i][j];
      bad |= split_failed(acc[0][i][j], lo);
    }
  if (__builtin_expect(__any(bad), 0)) {
#pragma unroll 1
    for (int n = 0; n < MI * NI; ++n) {
      const f32x16 t = block_f32(item, extra, st, row0 + wm * (BM / WM) + n / NI * 32,
                                 col0 + wn * (BM / WN) + n % NI * 32);
#pragma unroll
      for (int i = 0; i < MI * NI; ++i)
        if (i == n) acc[0][i / NI][i % NI] = t;
    }
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
      } else if (epi == EPI_SERIES) {
        float* dst2 = item.dst2;
        const int64_t ld2 = item.ld2;
        const float beta = item.beta;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = ibase + acc_row(r, lane);
          const float p = beta * v[r];
          // each element belongs to one item of the launch
          if (i < M && j < N) gst_f32(dst2, (int64_t)i * ld2 + j, gld_f32(dst2, (int64_t)i * ld2 + j) + p);
          if (C && i < M && j < ldc) gst_f32(C, (int64_t)i * ldc + j, j < N ? p : 0.f);
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

template <int BM, int MODE>
hipError_t launch_one(const GemmItem* items, const GemmTile* tiles, int n, int step, const GemmPair* pairs,
                      hipStream_t s) {
  if (n <= 0) return hipSuccess;
  // two stages of two operands (the epilogues need less); above the default
  // limit with 128-tiles
  constexpr int lds = 2 * 2 * P * BM * 32 * 2;
  if constexpr (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_f32_kernel<BM, MODE>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((gemm_f32_kernel<BM, MODE>), dim3(n), dim3(BM == 64 ? 256 : 512), lds, s, items, tiles, step,
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
  const bool big = run.tile == 128;
  e = big ? launch_one<128, GEMM_ROWS>(items, t, run.n[GEMM_ROWS], step, pairs, s)
          : launch_one<64, GEMM_ROWS>(items, t, run.n[GEMM_ROWS], step, pairs, s);
  t += run.n[GEMM_ROWS];
  if (e == hipSuccess)
    e = big ? launch_one<128, GEMM_KMAJOR>(items, t, run.n[GEMM_KMAJOR], step, pairs, s)
            : launch_one<64, GEMM_KMAJOR>(items, t, run.n[GEMM_KMAJOR], step, pairs, s);
  t += run.n[GEMM_KMAJOR];
  if (e == hipSuccess)
    e = big ? launch_one<128, GEMM_ANY>(items, t, run.n[GEMM_ANY], step, pairs, s)
            : launch_one<64, GEMM_ANY>(items, t, run.n[GEMM_ANY], step, pairs, s);
  timing_end(name, s);
  return e;
}

}  // namespace orth
