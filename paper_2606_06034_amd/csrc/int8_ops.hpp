// int8_ops.hpp -- the INT8 arithmetic of the integer inverse (Section 3.5,
// Appendix G of arXiv 2606.06034): 8-bit codes (|q| <= 127) on int8 quad
// fragments, exact int32 products and sums, quantisation by the scale rule
// of intq.hpp, and the I8Ops width the shared engine (int_engine of
// intq.hpp) runs on, plus the per-tile quantiser's exponent.  Used by
// int8.hip and by the layer forward's integer-inverse mode.
#pragma once

#include "intq.hpp"

namespace gdn {
namespace i8 {

using namespace iq;

constexpr int kQ = 127, kQB = 7;

// Codes are held as integer-valued fp32: a code is at most 127, an exact int8
// product at most 64 127^2 < 2^20, the sum of two tensors whose exponents are
// at most 16 apart below 2^23, so every value and every sum below is exact in
// fp32 (24 bits).  The vector unit is what bounds the integer inverse, and
// fp32 takes fewer of its operations than int32: the maximum of two magnitudes
// is one (three-way maximum with absolute values), an aligned sum one (a fused
// multiply-add by a power of two), a rounding one and a subtraction: x 2^-s +
// 1.5 2^23 lies where the fp32 spacing is 1, so the fused addition rounds half
// to even, and its low byte is the code's byte.
constexpr float kMagic = 12582912.f;  // 1.5 * 2^23

// 2^k as fp32, -126 <= k <= 127
__device__ __forceinline__ float pow2f(int k) {
  return __builtin_bit_cast(float, (uint32_t)(k + 127) << 23);
}

// the bytes of four codes plus kMagic
__device__ __forceinline__ int pack_biased(f32x4 x) {
  const i32x4 b = __builtin_bit_cast(i32x4, x);
  return gather_bytes<0>(b[0], b[1], b[2], b[3]);
}
__device__ __forceinline__ int packf(f32x4 x) { return pack_biased(x + kMagic); }

// The helpers below visit only the blocks that can meet a band [lo, hi] of
// sub-diagonals; every other block of their operand is exactly zero by the
// structure of the computation, so skipping it changes no result.

// max |D| over those blocks, wave-wide
template <int NB>
__device__ __forceinline__ float amaxf(const Acc<NB>& D, int lo, int hi) {
  float m = 0.f;
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J <= I; ++J)
      if (blk_nz(I - J, lo, hi))
#pragma unroll
        for (int v = 0; v < 4; ++v) m = fmaxf(m, fabsf(D.a[bidx(I, J)][v]));
  return wave_maxf(m);
}

// The scale rule's shift (shift_canon) from amax > 0, an integer: amax = m
// 2^p, m in [0.5, 1); 128 m >= 127.5 exactly when the 23 fraction bits are at
// least (127.5 / 64 - 1) 2^23.
__device__ __forceinline__ int shift_f(float amax) {
  const int b = __builtin_bit_cast(int, amax);
  return (b >> 23) - 126 - kQB + ((b & 0x7fffff) >= 0x7f0000 ? 1 : 0);
}

// D 2^-s rounded half to even, in place (exact for s <= 0)
template <int NB>
__device__ __forceinline__ void rescale(Acc<NB>& D, int s, int lo, int hi) {
  const float sc = pow2f(-s);
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J <= I; ++J)
      if (blk_nz(I - J, lo, hi))
#pragma unroll
        for (int v = 0; v < 4; ++v)
          D.a[bidx(I, J)][v] = __builtin_fmaf(D.a[bidx(I, J)][v], sc, kMagic) - kMagic;
}

// exact integer values of exponent e_in to codes by the scale rule, in
// place; exponent and non-zero flag through refs
template <int NB>
__device__ __forceinline__ void requantf(Acc<NB>& D, int lo, int hi, int e_in, int& e_out,
                                         bool& nz) {
  const float amax = amaxf(D, lo, hi);
  nz = amax > 0.f;
  if (!nz) {
    e_out = 0;
    return;
  }
  const int s = shift_f(amax);
  if (s != 0) rescale(D, s, lo, hi);
  e_out = e_in + s;
}

// the strictly lower A of one tile (row form, fp32) as codes of -A at
// exponent e (quant_exp of its maximum)
template <int NB>
__device__ __forceinline__ void quantize_neg(Acc<NB>& L, const Acc<NB>& A, int e) {
  if (e >= -120 && e <= 120) {  // 2^-e is a normal number
    const float sc = pow2f(-e);
#pragma unroll
    for (int b = 0; b < nlower(NB); ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) L.a[b][v] = __builtin_fmaf(A.a[b][v], -sc, kMagic) - kMagic;
  } else {
#pragma unroll
    for (int b = 0; b < nlower(NB); ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) L.a[b][v] = -rintf(ldexpf(A.a[b][v], -e));
  }
}

// ---------------------------------------------------------------------------

// The INT8 width for the shared integer engine (int_engine of intq.hpp).
template <int NB> struct I8Ops {
  using Codes = Acc<NB>;
  using Row = RowQ<NB>;
  using Col = ColQ<NB>;
  static constexpr int kQ = i8::kQ;
  static constexpr int kQB = i8::kQB;                                 // |code| < 2^7
  static constexpr int kAccB = 14 + (NB == 1 ? 4 : NB == 2 ? 5 : 6);  // |product| < C 2^14
  static __device__ __forceinline__ bool any(const Codes& D, int lo, int hi) {
    return amaxf(D, lo, hi) > 0.f;
  }
  static __device__ __forceinline__ void to_row(Row& X, const Codes& D, int lo, int hi) {
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int K = 0; K < 4; ++K)
        X.r[I].v[K] = (K <= I && blk_nz(I - K, lo, hi)) ? packf(D.a[bidx(I, K)]) : 0;
  }
  static __device__ __forceinline__ void to_row(Row& X, const AccI<NB>& D, int lo, int hi) {
    to_rowq(X, D, lo, hi);
  }
  static __device__ __forceinline__ void to_col(Col& Y, const AccI<NB>& D, int lo, int hi) {
    to_colq(Y, D, lo, hi);
  }
  // the codes of the blocks of X that can meet [lo, hi] (others 0)
  static __device__ __forceinline__ void codes(Codes& D, const Row& X, int lo, int hi) {
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J <= I; ++J)
        D.a[bidx(I, J)] = blk_nz(I - J, lo, hi)
                              ? __builtin_convertvector(unpack4(X.r[I].v[J]), f32x4)
                              : zero4();
  }
  // q(X Y 2^e_in) over [lo, hi] as codes and as row fragments (X and Y are
  // read before qr is written)
  static __device__ __forceinline__ void mulq(const Row& X, const Col& Y, int lo, int hi, int e_in,
                                              Codes& q, Row& qr, int& e_out, bool& nz) {
    AccI<NB> D;
    mmi<NB, true>(D, X, Y, lo, hi);
#pragma unroll
    for (int b = 0; b < nlower(NB); ++b) q.a[b] = __builtin_convertvector(D.a[b], f32x4);
    const float amax = amaxf(q, lo, hi);
    nz = amax > 0.f;
    const int s = nz ? shift_f(amax) : 0;
    const float sc = pow2f(-s);
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int K = 0; K < 4; ++K) {
        int w = 0;
        if (K <= I && blk_nz(I - K, lo, hi)) {
          f32x4 x = q.a[bidx(I, K)];
#pragma unroll
          for (int v = 0; v < 4; ++v) x[v] = __builtin_fmaf(x[v], sc, kMagic);
          w = pack_biased(x);
          q.a[bidx(I, K)] = x - kMagic;
        }
        qr.r[I].v[K] = w;
      }
    e_out = nz ? e_in + s : 0;
  }
  // codes to the finest scale that holds them (exact)
  static __device__ __forceinline__ void canon(Codes& q, int lo, int hi, int& e, bool& nz) {
    requantf(q, lo, hi, e, e, nz);
  }
  // X = q(X 2^eX + ys Y 2^eY) over [lo, hi] (X's band [xlo, hi], Y's
  // [ylo, hi]); Y is at the finest scale that holds it, and so is X when
  // xc.  Two terms with exponents 2 QB + 3 or more apart: the finer is below
  // an eighth of the output quantum and leaves the coarser's codes as they
  // are (at their finest scale); otherwise the sum is exact (below 2^23).
  static __device__ __forceinline__ void add(Codes& X, int& eX, bool& nzX, int xlo, bool xc,
                                             const Codes& Y, int eY, bool nzY, int ys, int ylo,
                                             int lo, int hi) {
    const int g = !nzY ? 64 : nzX ? eX - eY : -64;
    if (g >= 2 * kQB + 3) {
      if (!xc) canon(X, xlo, hi, eX, nzX);
      return;
    }
    auto each = [&](auto&& f) {
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = 0; J <= I; ++J)
          if (blk_nz(I - J, lo, hi)) {
            const f32x4 x = blk_nz(I - J, xlo, hi) ? X.a[bidx(I, J)] : zero4();
            const f32x4 y = blk_nz(I - J, ylo, hi) ? Y.a[bidx(I, J)] : zero4();
#pragma unroll
            for (int v = 0; v < 4; ++v) X.a[bidx(I, J)][v] = f(x[v], y[v]);
          }
    };
    const float fs = (float)ys;
    if (g <= -(2 * kQB + 3)) {
      each([&](float, float y) { return y * fs; });
      eX = eY;
      nzX = true;
      return;
    }
    const int e0 = min(eX, eY);
    if (g >= 0) {
      const float a = pow2f(g);
      each([&](float x, float y) { return __builtin_fmaf(x, a, y * fs); });
    } else {
      const float a = pow2f(-g) * fs;
      each([&](float x, float y) { return __builtin_fmaf(y, a, x); });
    }
    requantf(X, lo, hi, e0, eX, nzX);
  }
  // out = q(x + y + sign X Y 2^ep), the product on the sub-diagonals from plo
  // on and absent when !pp: terms whose tops and finest exponent span at most
  // 22 bits (three of them below 2^24) are summed exactly in fp32, wider ones
  // in fp64 (exact_sum)
  static __device__ __forceinline__ void mul_sum(Codes& out, int& eo, bool& nz,
                                                 const Term<Codes>& x, const Term<Codes>& y,
                                                 const Row& X, const Col& Y, int ep, int sign,
                                                 int plo, bool pp, int lo, int hi) {
    AccI<NB> D;
    mmi<NB, true>(D, X, Y, plo, hi);
    const Term<AccI<NB>> z = term(D, ep, kAccB, sign, plo, hi, pp);
    int emin = 1 << 30, top = -(1 << 30);
    auto span = [&](const auto& t) {
      if (t.p) {
        emin = min(emin, t.e);
        top = max(top, t.e + t.bits);
      }
    };
    span(x);
    span(y);
    span(z);
    if (emin > top || top - emin > 22) {
      exact_sum<kQ, kQB, NB>(out, eo, nz, x, y, z, lo, hi);
      return;
    }
    auto scale = [&](const auto& t) { return t.p ? t.sign * pow2f(t.e - emin) : 0.f; };
    const float sx = scale(x), sy = scale(y), sz = scale(z);
    Acc<NB> r;
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J <= I; ++J) {
        const int m = I - J, b = bidx(I, J);
        f32x4 a = zero4();
        if (blk_nz(m, lo, hi))
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            if (blk_nz(m, z.lo, z.hi)) a[v] = (float)z.t->a[b][v] * sz;
            if (blk_nz(m, x.lo, x.hi)) a[v] = __builtin_fmaf((float)x.t->a[b][v], sx, a[v]);
            if (blk_nz(m, y.lo, y.hi)) a[v] = __builtin_fmaf((float)y.t->a[b][v], sy, a[v]);
          }
        r.a[b] = a;
      }
    requantf(r, lo, hi, emin, eo, nz);
    out = r;
  }
  static __device__ __forceinline__ void row_to_col(Col& Y, const Row& X, const ColQ<NB>& Ic,
                                                    int lo, int hi) {
    AccI<NB> t;
    mmi<NB, false>(t, X, Ic, lo, hi);
    to_colq(Y, t, lo, hi);
  }
};

// e = the smallest integer at which round-half-even(amax / 2^e) <= 127
// (frexp: amax = m 2^p with m in [0.5, 1) gives amax / 2^(p - 7) = 128 m,
// which rounds past 127 when 128 m >= 127.5), 0 for amax = 0
__device__ __forceinline__ int quant_exp(float amax) {
  int e = 0;
  if (amax > 0.f) {
    int p;
    const float mant = frexpf(amax, &p);
    e = p - 7 + (mant * 128.f >= 127.5f ? 1 : 0);
  }
  return e;
}

}  // namespace i8
}  // namespace gdn
