// intq.hpp -- integer operands of the low-bit inverse paths on gfx950's
// int8 MFMA (v_mfma_i32_16x16x64_i8): int8 "quad" fragments of lower
// block-triangular C x C matrices (C = 16, 32, 64), their exact int32
// products, the identity, band masks, a wave-wide maximum, the scale rule
// of the quantiser, exact sums in fp64, and the integer inverse of one tile
// (int_engine) that both code widths run.
//
// A quad holds 16 int8 per lane, four 16 x 16 blocks of 4 bytes: row quad
// R[I] = blocks (I, 0..3) in row form, column quad Cq[J] = blocks (0..3, J)
// in column form (the fragment forms of tile16.hpp); one MFMA contracts all
// four k-blocks (zero blocks where K > I or K < J).  C = 16, 32 use the
// leading one or two blocks.  Values are held as int32 blocks AccI between
// products (index bidx(I, J) of the lower blocks).
#pragma once

#include "tile16.hpp"

#include <stdint.h>

#include <type_traits>

// wave reductions of the ROCm device library
extern "C" __device__ __attribute__((const)) int __ockl_wfred_max_i32(int);
extern "C" __device__ __attribute__((const)) float __ockl_wfred_max_f32(float);

namespace gdn {
namespace iq {

typedef double f64x4 __attribute__((ext_vector_type(4)));

struct Quad {
  i32x4 v;  // dword K = 4 bytes of block K
};

template <int NB> struct RowQ { Quad r[NB]; };
template <int NB> struct ColQ { Quad c[NB]; };
template <int NB> struct AccI { i32x4 a[nlower(NB)]; };

__device__ __forceinline__ i32x4 zero_i4() { return i32x4{0, 0, 0, 0}; }

// byte B of four dwords, one after another (two byte permutes and an or)
template <int B>
__device__ __forceinline__ int gather_bytes(int x0, int x1, int x2, int x3) {
  constexpr uint32_t b = B;
  const uint32_t lo = __builtin_amdgcn_perm((uint32_t)x1, (uint32_t)x0, 0x0c0c0400u + b * 0x101u);
  const uint32_t hi = __builtin_amdgcn_perm((uint32_t)x3, (uint32_t)x2, 0x04000c0cu + b * 0x1010000u);
  return (int)(lo | hi);
}
// 4 int32 in [-128, 127] <-> 4 bytes (value v in byte v)
__device__ __forceinline__ int pack4(i32x4 x) { return gather_bytes<0>(x[0], x[1], x[2], x[3]); }
__device__ __forceinline__ i32x4 unpack4(int w) {
  i32x4 r;
#pragma unroll
  for (int v = 0; v < 4; ++v) r[v] = (int)(int8_t)(w >> (8 * v));
  return r;
}

// Quads from blocks; blocks that cannot meet the band [lo, hi] (structurally
// zero) are packed as constant zeros.
template <int NB>
__device__ __forceinline__ void to_rowq(RowQ<NB>& X, const AccI<NB>& D, int lo = 0,
                                        int hi = 16 * NB) {
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int K = 0; K < 4; ++K)
      X.r[I].v[K] = (K <= I && I < NB && blk_nz(I - K, lo, hi)) ? pack4(D.a[bidx(I, K)]) : 0;
}
template <int NB>
__device__ __forceinline__ void to_colq(ColQ<NB>& Y, const AccI<NB>& D, int lo = 0,
                                        int hi = 16 * NB) {
#pragma unroll
  for (int J = 0; J < NB; ++J)
#pragma unroll
    for (int K = 0; K < 4; ++K)
      Y.c[J].v[K] = (K >= J && K < NB && blk_nz(K - J, lo, hi)) ? pack4(D.a[bidx(K, J)]) : 0;
}

// D = X Y (lower), blocks outside [olo, ohi] set to 0; OUTQ: row-form result.
template <int NB, bool OUTQ>
__device__ __forceinline__ void mmi(AccI<NB>& D, const RowQ<NB>& X, const ColQ<NB>& Y, int olo,
                                    int ohi) {
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J <= I; ++J) {
      i32x4 acc = zero_i4();
      if (blk_nz(I - J, olo, ohi))
        acc = OUTQ ? __builtin_amdgcn_mfma_i32_16x16x64_i8(Y.c[J].v, X.r[I].v, acc, 0, 0, 0)
                   : __builtin_amdgcn_mfma_i32_16x16x64_i8(X.r[I].v, Y.c[J].v, acc, 0, 0, 0);
      D.a[bidx(I, J)] = acc;
    }
}

// identity as quads (row and column quads coincide)
template <int NB>
__device__ __forceinline__ void eye_quads(RowQ<NB>& R, ColQ<NB>& Cq) {
  AccI<NB> e;
  const int g = lane_g(), c = lane_c();
#pragma unroll
  for (int b = 0; b < nlower(NB); ++b) e.a[b] = zero_i4();
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int v = 0; v < 4; ++v) e.a[bidx(I, I)][v] = (c == 4 * g + v) ? 1 : 0;
  to_rowq(R, e);
  to_colq(Cq, e);
}

// zero entries outside lo <= i - j <= hi of the lower blocks a[bidx(I, J)]
// (any four-element block type)
template <int NB, bool COLFORM, typename V>
__device__ __forceinline__ void band_blocks(V* a, int lo, int hi) {
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J <= I; ++J) {
      if (!blk_nz(I - J, lo, hi)) {
        a[bidx(I, J)] = V{};
      } else if (!blk_all_in(I - J, lo, hi)) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int d = COLFORM ? dcol(I - J, v) : drow(I - J, v);
          if (d < lo || d > hi) a[bidx(I, J)][v] = 0;
        }
      }
    }
}

// wave-wide maximum (the device library's DPP reduction), as a scalar
__device__ __forceinline__ int wave_max(int x) {
  return __builtin_amdgcn_readfirstlane(__ockl_wfred_max_i32(x));
}

// max |D| over the blocks that can meet the band [lo, hi] (every other block
// is zero by the structure of the computation), wave-wide
template <int NB>
__device__ __forceinline__ int amax_of(const AccI<NB>& D, int lo, int hi) {
  // the largest and the smallest value: one three-way maximum or minimum
  // takes two values, an absolute value would cost an operation each
  int mx = 0, mn = 0;
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J <= I; ++J)
      if (blk_nz(I - J, lo, hi))
#pragma unroll
        for (int v = 0; v < 4; v += 2) {
          const int a = D.a[bidx(I, J)][v], b = D.a[bidx(I, J)][v + 1];
          mx = max(max(mx, a), b);
          mn = min(min(mn, a), b);
        }
  return wave_max(max(mx, -mn));
}


// ---------------------------------------------------------------------------
// Full 64 x 64 matrices (all 4 x 4 blocks; the off-diagonal block of a
// C = 128 tile), values as int32 blocks, block (I, J) at 4 I + J.

struct FullI {
  i32x4 a[16];
};

__device__ __forceinline__ void to_rowq_full(RowQ<4>& X, const FullI& D) {
#pragma unroll
  for (int I = 0; I < 4; ++I)
#pragma unroll
    for (int K = 0; K < 4; ++K) X.r[I].v[K] = pack4(D.a[4 * I + K]);
}
// D in column form
__device__ __forceinline__ void to_colq_full(ColQ<4>& Y, const FullI& D) {
#pragma unroll
  for (int J = 0; J < 4; ++J)
#pragma unroll
    for (int K = 0; K < 4; ++K) Y.c[J].v[K] = pack4(D.a[4 * K + J]);
}
// D = X Y over the output block columns J0 .. J0 + JN - 1 (all 16 blocks
// by default; the other blocks of D are left as they are); X or Y may be
// lower: its quads carry the zero blocks.  OUTQ: row-form result.
template <bool OUTQ, int J0 = 0, int JN = 4>
__device__ __forceinline__ void mmi_full(FullI& D, const RowQ<4>& X, const ColQ<4>& Y) {
#pragma unroll
  for (int I = 0; I < 4; ++I)
#pragma unroll
    for (int J = J0; J < J0 + JN; ++J)
      D.a[4 * I + J] =
          OUTQ ? __builtin_amdgcn_mfma_i32_16x16x64_i8(Y.c[J].v, X.r[I].v, zero_i4(), 0, 0, 0)
               : __builtin_amdgcn_mfma_i32_16x16x64_i8(X.r[I].v, Y.c[J].v, zero_i4(), 0, 0, 0);
}
__device__ __forceinline__ int amax_full(const FullI& D) {
  int m = 0;
#pragma unroll
  for (int b = 0; b < 16; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) m = max(m, abs(D.a[b][v]));
  return wave_max(m);
}


// ---------------------------------------------------------------------------
// The scale rule.  A tensor of codes |q| <= Q with one power-of-two scale
// 2^e per tile; an exactly known tensor v is quantised to
// q = round-half-even(v / 2^e) with e the smallest integer at which no code
// leaves [-Q, Q], i.e. max|v| < (Q + 1/2) 2^e (Appendix G's
// q(x) = clip(round(x / Delta)) with the finest Delta = 2^e whose clip does
// nothing).  QB: 2^(QB - 1) <= Q < 2^QB.

// The shift s = e - e_v for values v = y 2^e_v held as integers y with
// max|y| = amax > 0 (int32): s is b - QB or b - QB + 1, b the bit length of
// amax (amax / 2^(b - QB) lies in [2^(QB-1), 2^QB)).
template <int Q, int QB>
__device__ __forceinline__ int shift_canon(int amax) {
  const int b = 32 - __clz(amax);
  const int s = b - QB;
  const bool over = s <= 0 ? ((int64_t)amax << -s) > Q
                           : 2 * (int64_t)amax >= ((2 * (int64_t)Q + 1) << s);
  return s + (over ? 1 : 0);
}

// The same shift from the high dword of max|y| for y held as fp64 integers
// (amax_hi > 0).  The test amax < (Q + 1/2) 2^s compares with a threshold
// of at most 16 significant bits, whose low dword is zero, so amax and its
// high dword (the value with the low dword cleared) compare alike with it.
// amax = m 2^p, m in [0.5, 1): 2^QB m < Q + 1/2 gives s = p - QB, else
// p - QB + 1.
template <int Q, int QB>
__device__ __forceinline__ int shift_canon_hi(int amax_hi) {
  const double a = __hiloint2double(amax_hi, 0);
  int p;
  const double m = frexp(a, &p);
  return p - QB + (m * (double)(1 << QB) >= (double)Q + 0.5 ? 1 : 0);
}

// round-half-even(x sc) as int32 for an fp64 integer x and a power of two sc
// with |x sc| < 2^31: x sc + 1.5 2^52 lies in [2^52, 2^53), where the fp64
// spacing is 1, so the fused addition rounds x sc half to even and the low
// dword of the sum holds the result in two's complement (1.5 2^52 has a zero
// low dword)
constexpr double kRoundMagic = 6755399441055744.0;  // 1.5 * 2^52
__device__ __forceinline__ int rne_scaled(double x, double sc) {
  return __double2loint(__builtin_fma(x, sc, kRoundMagic));
}

__device__ __forceinline__ double elem(const i32x4& x, int v) { return (double)x[v]; }
__device__ __forceinline__ double elem(const f32x4& x, int v) { return (double)x[v]; }
__device__ __forceinline__ double elem(const f64x4& x, int v) { return x[v]; }

// A term of an exact sum: the lower blocks of t (band [lo, hi]) times
// sign 2^e, absent when !p.  bits bounds |t| < 2^bits.
template <typename T> struct Term {
  const T* t;
  int e, bits, sign, lo, hi;
  bool p;
};

// the bit length of max|t| over the term's band (0 when t is zero): the
// wave maximum of the high dwords of |t| as fp64, whose frexp exponent is
// the bit length (an integer's high dword keeps its leading bit)
template <int NB, typename T>
__device__ __forceinline__ int term_bits(const Term<T>& x) {
  int mh = 0;
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J <= I; ++J)
      if (blk_nz(I - J, x.lo, x.hi)) {
        const auto q = x.t->a[bidx(I, J)];
#pragma unroll
        for (int v = 0; v < 4; ++v) mh = max(mh, __double2hiint(fabs(elem(q, v))));
      }
  mh = wave_max(mh);
  if (mh == 0) return 0;
  int p;
  frexp(__hiloint2double(mh, 0), &p);
  return p;
}

// The exponent plan of an exact sum of up to three terms, wave-uniform:
// the scale of each present term relative to the finest one kept (emin),
// and which terms are rounded to the 52-bit window.  In: each term's
// exponent e, magnitude bits b (|t| < 2^b, 2^(b-1) <= max|t|) and presence
// p.  When the present terms span at most 52 bits the sum is exact in
// fp64.  Otherwise a term whose top lies QB + 6 bits or more under the
// coarsest top is dropped: unless the kept terms cancel below a quarter of
// the coarsest one's largest value, the output's quantum is at least
// 2^(top - QB - 2), so the dropped terms together stay below an eighth of
// it and move no code.  If the kept terms still span more than 52 bits, the
// finest are rounded to the window; exactness is claimed for neither of
// these two cases (no tile of the quantiser's output on the workloads
// reaches them).
struct SumPlan {
  int emin;
  bool p[3], r[3];
};
template <int QB>
__device__ __forceinline__ SumPlan sum_plan(const int (&e)[3], const int (&b)[3],
                                            const bool (&p)[3]) {
  SumPlan pl;
  int top = -(1 << 30), emin = 1 << 30;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    pl.p[k] = p[k];
    pl.r[k] = false;
    if (p[k]) {
      top = max(top, e[k] + b[k]);
      emin = min(emin, e[k]);
    }
  }
  if (top - emin > 52) {
    // only here are b the measured magnitudes (see exact_sum, sum2_full)
    emin = 1 << 30;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      pl.p[k] = p[k] && e[k] + b[k] > top - QB - 6;
      if (pl.p[k]) emin = min(emin, e[k]);
    }
  }
  if (top - emin > 52) {
    const int floor_e = top - 52;
    emin = 1 << 30;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (pl.p[k]) {
        pl.r[k] = e[k] < floor_e;
        emin = min(emin, max(e[k], floor_e));
      }
  }
  pl.emin = emin;
  return pl;
}

// out = q(sum of the terms) over the blocks of the band [lo, hi]: the exact
// sum (every term aligned at the finest exponent among the kept ones)
// quantised once by the scale rule (Q, QB).  The values are fp64 integers.
// The plan first takes each term's bound bits; only when those span more
// than 52 bits are the terms' actual magnitudes measured (wave maxima), so
// that a zero or small term does not widen the window (sum_plan).  Returns
// the codes, their exponent and a non-zero flag; every block of out
// outside the band is set to 0.
template <int Q, int QB, int NB, typename TO, typename T1, typename T2, typename T3>
__device__ __forceinline__ void exact_sum(TO& out, int& eo, bool& nz, const Term<T1>& x,
                                          const Term<T2>& y, const Term<T3>& z, int lo, int hi) {
  int e[3] = {x.e, y.e, z.e}, b[3] = {x.bits, y.bits, z.bits};
  bool p[3] = {x.p, y.p, z.p};
  int emin = 1 << 30, top = -(1 << 30);
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (p[k]) {
      emin = min(emin, e[k]);
      top = max(top, e[k] + b[k]);
    }
  if (!p[0] && !p[1] && !p[2]) {
#pragma unroll
    for (int bb = 0; bb < nlower(NB); ++bb) out.a[bb] = {};
    eo = 0;
    nz = false;
    return;
  }
  if (top - emin > 52) {
    if (p[0]) { b[0] = term_bits<NB>(x); p[0] = b[0] > 0; }
    if (p[1]) { b[1] = term_bits<NB>(y); p[1] = b[1] > 0; }
    if (p[2]) { b[2] = term_bits<NB>(z); p[2] = b[2] > 0; }
  }
  const SumPlan pl = sum_plan<QB>(e, b, p);
  const double sx = pl.p[0] ? (double)x.sign * ldexp(1.0, x.e - pl.emin) : 0.0;
  const double sy = pl.p[1] ? (double)y.sign * ldexp(1.0, y.e - pl.emin) : 0.0;
  const double sz = pl.p[2] ? (double)z.sign * ldexp(1.0, z.e - pl.emin) : 0.0;
  // block (I, J) of the sum
  auto val = [&](int I, int J) {
    const int m = I - J, bi = bidx(I, J);
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    auto put = [&](const auto& t, bool p, bool r, double sc) {
      if (p && blk_nz(m, t.lo, t.hi)) {
        const auto q = t.t->a[bi];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double d = elem(q, v) * sc;
          acc[v] += r ? rint(d) : d;
        }
      }
    };
    put(x, pl.p[0], pl.r[0], sx);
    put(y, pl.p[1], pl.r[1], sy);
    put(z, pl.p[2], pl.r[2], sz);
    return acc;
  };
  int mh = 0;
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J <= I; ++J)
      if (blk_nz(I - J, lo, hi)) {
        const f64x4 q = val(I, J);
#pragma unroll
        for (int v = 0; v < 4; ++v) mh = max(mh, __double2hiint(fabs(q[v])));
      }
  const int amax_hi = wave_max(mh);
  nz = amax_hi > 0;
  const int s = nz ? shift_canon_hi<Q, QB>(amax_hi) : 0;
  const double sc = ldexp(1.0, -s);
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J <= I; ++J) {
      out.a[bidx(I, J)] = {};
      if (nz && blk_nz(I - J, lo, hi)) {
        const f64x4 q = val(I, J);
#pragma unroll
        for (int v = 0; v < 4; ++v) out.a[bidx(I, J)][v] = rne_scaled(q[v], sc);
      }
    }
  eo = nz ? pl.emin + s : 0;
}

template <typename T>
__device__ __forceinline__ Term<T> term(const T& t, int e, int bits, int sign, int lo, int hi,
                                        bool p) {
  return Term<T>{&t, e, bits, sign, lo, hi, p};
}
template <typename T>
__device__ __forceinline__ Term<T> no_term(const T& t) {
  return Term<T>{&t, 0, 0, 1, 1 << 20, -(1 << 20), false};  // meets no block
}

// The sum of x over the 16 lanes of one g (rotations within rows of 16 lanes).
__device__ __forceinline__ float row_sum(float x) {
  auto ror = [](float y, auto n) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, y), 0x120 + decltype(n)::value, 0xf,
                                        0xf, true));
  };
  x += ror(x, std::integral_constant<int, 8>{});
  x += ror(x, std::integral_constant<int, 4>{});
  x += ror(x, std::integral_constant<int, 2>{});
  x += ror(x, std::integral_constant<int, 1>{});
  return x;
}

// wave-wide maximum of non-negative floats, as a scalar
__device__ __forceinline__ float wave_maxf(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, __ockl_wfred_max_f32(x))));
}

// Is every column sum of |E| (codes of a lower matrix in row form, band
// [lo, C-1], exponent e) at most 1?  Then |(P E)_ij| <= max|P| for any P,
// so each residual power is bounded by the one before it.  Lane (g, c) of
// a row-form block holds row c, columns 4g + v: the sum over a block's rows
// runs over the 16 lanes of one g, the sum over block rows in the lane.
// Sums of at most 64 codes below 2^15 are exact in fp32.
template <int NB, typename V>
__device__ __forceinline__ bool colsum_at_most_one(const V* E, int e, int lo) {
  float best = 0.f;
#pragma unroll
  for (int J = 0; J < NB; ++J)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float sacc = 0.f;
#pragma unroll
      for (int I = J; I < NB; ++I)
        if (blk_nz(I - J, lo, 16 * NB - 1)) sacc += fabsf((float)E[bidx(I, J)][v]);
      best = fmaxf(best, row_sum(sacc));
    }
  return ldexpf(wave_maxf(best), e) <= 1.f;  // (underflow: at most 1)
}

// identity codes (1 on the diagonal, exponent 0)
template <int NB, typename V>
__device__ __forceinline__ void eye_codes(V* a) {
  const int g = lane_g(), c = lane_c();
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J <= I; ++J)
#pragma unroll
      for (int v = 0; v < 4; ++v) a[bidx(I, J)][v] = (I == J && c == 4 * g + v) ? 1 : 0;
}

// ---------------------------------------------------------------------------
// The integer inverse of one tile: Algorithm 1 (Section 3.4) with integer
// activations (Section 3.5, Appendix G), every operator evaluated exactly
// from its operands' codes and its result quantised once by the scale rule:
//   P_1 = L (= -A), P_n = q(P_{n-1} L),          T0 = q(T0 + P_n),
//   T0 = M^(N) (.) T0 (codes masked, scale kept),
//   E = I - q((I + A) T0),
//   P_1 = E, P_s = q(P_{s-1} E),                 T = q(T + P_s),
//   T_hat = q(T0 T)
// (T0 starts at I, T at I).  Split form (PLAIN false): the unit diagonal of
// T0, T and T_hat stays out of the codes, so their tensors are the strict
// lower parts and a product of two of them is (I + X)(I + Y) = I + (X + Y +
// X Y), one rounding of the three-term sum; E = -q(A + N0 + A N0).  Plain
// form: every tensor holds its diagonal; E = q(I - q(T0 + A T0)).
//
// In: Lm = -A as codes (row form, strictly lower) with exponent eL.  Out:
// T_hat's tensor as codes Tr (row form) and its exponent eTo.  NC, SC >= 0
// fix N and S at compile time; -1 takes them from Nrt, Srt.
//
// Ops<NB> supplies one code width: Codes (a matrix of codes, lower blocks
// a[bidx(I, J)], held as int32 or as integer-valued fp32), fragment types Row,
// Col (operands in row and column form); kQ, kQB (the code range and its bits);
// any (a code is non-zero), to_row, to_col (codes to fragments), codes
// (fragments back to codes), mulq (q of the exact product of two fragments, as
// codes and as row fragments), canon (codes to the finest scale that holds
// them), add (q of the sum of two tensors of codes, the first known to be at
// its finest scale or not), mul_sum (q of the exact sum of two tensors of codes
// and a product), row_to_col (column-form fragments of a row-form one, through
// the identity).  Every helper visits only the blocks
// that can meet the band of sub-diagonals it is given; the other blocks are
// zero by the structure of the computation.
template <template <int> class Ops, int NB, bool PLAIN, int NC = -1, int SC = -1>
__device__ __forceinline__ void int_engine(const typename Ops<NB>::Codes& Lr, int eL, int Nrt,
                                           int Srt, typename Ops<NB>::Codes& Tr, int& eTo) {
  using O = Ops<NB>;
  using Codes = typename O::Codes;
  constexpr int C = 16 * NB;
  constexpr int QB = O::kQB;
  constexpr int U0 = PLAIN ? 0 : 1;  // lowest sub-diagonal of T0's, T's and T_hat's tensors
  const int N = NC >= 0 ? NC : Nrt;
  const int S = SC >= 0 ? SC : Srt;
  RowQ<NB> Iq;
  ColQ<NB> Ic;
  eye_quads(Iq, Ic);

  const bool nzL = O::any(Lr, 1, C - 1);
  typename O::Row LRq;
  O::to_row(LRq, Lr, 1, C - 1);
  typename O::Col LCq;
  O::row_to_col(LCq, LRq, Ic, 1, C - 1);

  // ---- T0 = sum_{n=0}^{N} L^n, then masked
  Codes T0;
  int eT0 = 0;
  bool nzT0 = PLAIN;
  if constexpr (PLAIN) eye_codes<NB>(T0.a);
  else {
#pragma unroll
    for (int b = 0; b < nlower(NB); ++b) T0.a[b] = {};
  }
  if (N >= 1) {
    Codes P = Lr;
    int eP = eL;
    bool nzP = nzL;
    O::canon(P, 1, C - 1, eP, nzP);
    O::add(T0, eT0, nzT0, U0, !PLAIN, P, eP, nzP, 1, 1, U0, C - 1);
    typename O::Row PRq;
    O::to_row(PRq, P, 1, C - 1);
    auto power = [&](int n) {
      O::mulq(PRq, LCq, n, C - 1, eP + eL, P, PRq, eP, nzP);
      O::add(T0, eT0, nzT0, U0, true, P, eP, nzP, 1, n, U0, C - 1);
    };
    if constexpr (NC >= 0) {
#pragma unroll
      for (int n = 2; n <= NC; ++n) power(n);
    } else {
      for (int n = 2; n <= N; ++n) power(n);
    }
  }
  band_blocks<NB, false>(T0.a, U0, N);
  nzT0 = O::any(T0, U0, N);
  typename O::Row T0Rq;
  O::to_row(T0Rq, T0, U0, N);
  typename O::Col T0Cq;
  O::row_to_col(T0Cq, T0Rq, Ic, U0, N);

  // ---- E = I - q((I + A) T0), with (I + A) T0 = T0 - Lm T0
  constexpr int E0 = PLAIN ? 0 : 1;  // lowest sub-diagonal of E
  Codes E;
  int eE;
  bool nzE;
  if constexpr (!PLAIN) {
    // E = -(A + N0 + A N0) = Lm - N0 + Lm N0
    O::mul_sum(E, eE, nzE, term(Lr, eL, QB, 1, 1, C - 1, nzL), term(T0, eT0, QB, -1, 1, N, nzT0),
               LRq, T0Cq, eL + eT0, 1, 2, nzL && nzT0, 1, C - 1);
  } else {
    Codes M;
    int eM;
    bool nzM;
    O::mul_sum(M, eM, nzM, term(T0, eT0, QB, 1, 0, N, nzT0), no_term(T0), LRq, T0Cq, eL + eT0, -1,
               1, nzL && nzT0, 0, C - 1);
    eye_codes<NB>(E.a);
    eE = 0;
    nzE = true;
    O::add(E, eE, nzE, 0, false, M, eM, nzM, -1, 0, 0, C - 1);
  }
  typename O::Row ERq;
  O::to_row(ERq, E, E0, C - 1);
  typename O::Col ECq;
  O::row_to_col(ECq, ERq, Ic, E0, C - 1);

  // ---- T = sum_{s=0}^{S} E^s
  Codes R;
  int eR = 0;
  bool nzR = PLAIN;
  if constexpr (PLAIN) eye_codes<NB>(R.a);
  else {
#pragma unroll
    for (int b = 0; b < nlower(NB); ++b) R.a[b] = {};
  }
  if (S >= 1) {
    O::add(R, eR, nzR, U0, !PLAIN, E, eE, nzE, 1, E0, U0, C - 1);
    int eP = eE;
    bool nzP = nzE;
    typename O::Row PRq = ERq;
    // Once a residual power adds nothing to T (its exponent 2 QB + 3 or
    // more under T's, so the add leaves T's codes as they are) and every
    // column sum of |E| is at most 1, every later power is no larger, its
    // exponent no higher, and its add leaves T as it is too: the chain
    // stops there with the result it would have reached.
    const bool contracting = colsum_at_most_one<NB>(E.a, eE, E0);
    // a rolled loop: unrolled, the early exit keeps every iteration's
    // operands live at once and costs a wave per SIMD
#pragma unroll 1
    for (int s = 2; s <= S; ++s) {
      const int lo = PLAIN ? 0 : s;
      Codes P;
      O::mulq(PRq, ECq, lo, C - 1, eP + eE, P, PRq, eP, nzP);
      const bool idle = !nzP || (nzR && eR - eP >= 2 * QB + 3);
      O::add(R, eR, nzR, U0, true, P, eP, nzP, 1, lo, U0, C - 1);
      if (idle && contracting) break;
    }
  }

  // ---- T_hat = q(T0 T)
  typename O::Col RCq;
  {
    typename O::Row RRq;
    O::to_row(RRq, R, U0, C - 1);
    O::row_to_col(RCq, RRq, Ic, U0, C - 1);
  }
  bool nzT;
  if constexpr (!PLAIN) {
    // T0's codes again, from its row fragments (they hold every code exactly;
    // keeping the unpacked copy alive across the residual chain would cost a
    // wave per SIMD)
    O::codes(T0, T0Rq, U0, N);
    O::mul_sum(Tr, eTo, nzT, term(T0, eT0, QB, 1, 1, N, nzT0), term(R, eR, QB, 1, 1, C - 1, nzR),
               T0Rq, RCq, eT0 + eR, 1, 2, nzT0 && nzR, 1, C - 1);
  } else {
    typename O::Row unused;
    O::mulq(T0Rq, RCq, 0, C - 1, eT0 + eR, Tr, unused, eTo, nzT);
  }
}

// The same on int32 codes in and out, whatever the width holds codes in.
template <template <int> class Ops, int NB, bool PLAIN, int NC = -1, int SC = -1>
__device__ __forceinline__ void int_engine_i32(const AccI<NB>& Lr, int eL, int Nrt, int Srt,
                                               AccI<NB>& Tr, int& eTo) {
  typename Ops<NB>::Codes L, T;
  using E = std::remove_reference_t<decltype(L.a[0][0] + L.a[0][0])>;
#pragma unroll
  for (int b = 0; b < nlower(NB); ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) L.a[b][v] = (E)Lr.a[b][v];
  int_engine<Ops, NB, PLAIN, NC, SC>(L, eL, Nrt, Srt, T, eTo);
#pragma unroll
  for (int b = 0; b < nlower(NB); ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) Tr.a[b][v] = (int)T.a[b][v];
}

}  // namespace iq
}  // namespace gdn
