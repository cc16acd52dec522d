// int16_ops.hpp -- the INT16 arithmetic of the integer inverse (Section 3.5,
// Appendix G of arXiv 2606.06034): 16-bit codes as two int8 limbs, products and
// sums in int32 rounded to odd (or in fp64 where the terms lie too far apart),
// quantisation by the scale rule of intq.hpp and the I16Ops width the shared
// engine (int_engine of intq.hpp) runs on, plus the per-tile quantiser's
// exponent.  Used by int16.hip and by the
// layer forward's integer-inverse mode.
#pragma once

#include "intq.hpp"

namespace gdn {
namespace i16 {

using namespace iq;

constexpr int kQmax = 32639;

// the two int8 limbs of a matrix of codes, as quads
template <int NB> struct RowL { RowQ<NB> h, l; };
template <int NB> struct ColL { ColQ<NB> h, l; };

// The limb bytes of a code c = 256 h + l (l in [-128, 127]): l's byte is
// byte 0 of c, and c + 128 = 256 h + (l + 128) with 0 <= l + 128 <= 255, so
// h's byte is byte 1 of c + 128.  Four codes of a block give one dword of a
// quad per limb.
__device__ __forceinline__ int pack_lo(i32x4 c) { return gather_bytes<0>(c[0], c[1], c[2], c[3]); }
__device__ __forceinline__ int pack_hi(i32x4 c) {
  const i32x4 u = c + 128;
  return gather_bytes<1>(u[0], u[1], u[2], u[3]);
}

// limb quads of the blocks that can meet [lo, hi] (others zero), row form
template <int NB>
__device__ __forceinline__ void to_rowl(RowL<NB>& X, const AccI<NB>& D, int lo, int hi) {
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int K = 0; K < 4; ++K) {
      const bool live = K <= I && I < NB && blk_nz(I - K, lo, hi);
      X.h.r[I].v[K] = live ? pack_hi(D.a[bidx(I, K)]) : 0;
      X.l.r[I].v[K] = live ? pack_lo(D.a[bidx(I, K)]) : 0;
    }
}
// the same in column form
template <int NB>
__device__ __forceinline__ void to_coll(ColL<NB>& Y, const AccI<NB>& D, int lo, int hi) {
#pragma unroll
  for (int J = 0; J < NB; ++J)
#pragma unroll
    for (int K = 0; K < 4; ++K) {
      const bool live = K >= J && K < NB && blk_nz(K - J, lo, hi);
      Y.h.c[J].v[K] = live ? pack_hi(D.a[bidx(K, J)]) : 0;
      Y.l.c[J].v[K] = live ? pack_lo(D.a[bidx(K, J)]) : 0;
    }
}

// The limb products of one block of X Y (row-form result): X Y = 2^16 hh +
// 2^8 mx + ll.
struct LimbBlock { i32x4 hh, mx, ll; };
template <int NB>
__device__ __forceinline__ LimbBlock limb_block(const RowL<NB>& X, const ColL<NB>& Y, int I, int J) {
  const i32x4 xh = X.h.r[I].v, xl = X.l.r[I].v, yh = Y.h.c[J].v, yl = Y.l.c[J].v, z = zero_i4();
  LimbBlock b;
  b.hh = __builtin_amdgcn_mfma_i32_16x16x64_i8(yh, xh, z, 0, 0, 0);
  b.mx = __builtin_amdgcn_mfma_i32_16x16x64_i8(yl, xh, z, 0, 0, 0);
  b.mx = __builtin_amdgcn_mfma_i32_16x16x64_i8(yh, xl, b.mx, 0, 0, 0);
  b.ll = __builtin_amdgcn_mfma_i32_16x16x64_i8(yl, xl, z, 0, 0, 0);
  return b;
}
// A product as fp64 integers, formed block by block where it is read (the
// term of an exact_sum).
template <int NB>
struct LazyProd {
  struct Blocks {
    const RowL<NB>* X;
    const ColL<NB>* Y;
    __device__ __forceinline__ f64x4 operator[](int b) const {
      int I = 0;
      while ((I + 1) * (I + 2) / 2 <= b) ++I;
      // the operand is opaque, so that each pass forms the block anew: kept
      // from one pass to the next, ten blocks would take 80 registers
      RowL<NB> x = *X;
      asm volatile("" : "+v"(x.h.r[I].v), "+v"(x.l.r[I].v));
      const LimbBlock p = limb_block(x, *Y, I, b - I * (I + 1) / 2);
      f64x4 r;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        r[v] = __builtin_fma((double)(p.hh[v] * 256 + p.mx[v]), 256.0, (double)p.ll[v]);
      return r;
    }
  } a;
};

// A product in int32.  An entry F = X Y (below 2^36) is kept as F / 128
// rounded to odd: J = 2 floor(F / 256) + (256 does not divide F), below 2^30.
// J and F / 128 lie on the same side of every even integer (and meet one only
// together), so they compare alike with, and round half to even alike to,
// every quantum 2^s with s >= 2, and so do their sums with even integers.
// Half the registers of fp64 integers, which is what lets two waves share a
// SIMD.
template <int NB>
__device__ __forceinline__ i32x4 odd_block(const RowL<NB>& X, const ColL<NB>& Y, int I, int J) {
  const i32x4 xh = X.h.r[I].v, xl = X.l.r[I].v, yh = Y.h.c[J].v, yl = Y.l.c[J].v, z = zero_i4();
  const i32x4 ll = __builtin_amdgcn_mfma_i32_16x16x64_i8(yl, xl, z, 0, 0, 0);
  const i32x4 hh = __builtin_amdgcn_mfma_i32_16x16x64_i8(yh, xh, z, 0, 0, 0);
  i32x4 f = (hh << 8) + (ll >> 8);  // floor(F / 256), completed by the mixed products
  f = __builtin_amdgcn_mfma_i32_16x16x64_i8(yl, xh, f, 0, 0, 0);
  f = __builtin_amdgcn_mfma_i32_16x16x64_i8(yh, xl, f, 0, 0, 0);
  i32x4 r;
#pragma unroll
  for (int v = 0; v < 4; ++v) r[v] = (f[v] << 1) | (int)min((uint32_t)(ll[v] & 255), 1u);
  return r;
}
// y 2^-t rounded to odd (t >= 1): floor, with the last bit set when bits were
// lost; composes with what is rounded to odd already
__device__ __forceinline__ i32x4 odd_shift(i32x4 y, int t) {
  const uint32_t mask = (1u << t) - 1;
  i32x4 r;
#pragma unroll
  for (int v = 0; v < 4; ++v)
    r[v] = (y[v] >> t) | (int)min((uint32_t)y[v] & mask, 1u);
  return r;
}
// the product itself, for |F| < 2^31
template <int NB>
__device__ __forceinline__ i32x4 exact_block(const RowL<NB>& X, const ColL<NB>& Y, int I, int J) {
  const LimbBlock p = limb_block(X, Y, I, J);
  return (p.hh << 16) + (p.mx << 8) + p.ll;
}

// Column-form limbs of a row-form matrix, through the identity (exact).
template <int NB>
__device__ __forceinline__ void row_to_col(ColL<NB>& Y, const RowL<NB>& X, const ColQ<NB>& Ic,
                                           int lo, int hi) {
  AccI<NB> t;
  mmi<NB, false>(t, X.h, Ic, lo, hi);
  to_colq(Y.h, t, lo, hi);
  mmi<NB, false>(t, X.l, Ic, lo, hi);
  to_colq(Y.l, t, lo, hi);
}

// D 2^-s, in place: a right shift by s > 0 rounded half to even (|y| + 2^(s -
// 1) stays below 2^31), or an exact left shift
template <int NB>
__device__ __forceinline__ void rescale_i32(AccI<NB>& D, int s, int lo, int hi) {
  auto each = [&](auto&& f) {
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J <= I; ++J)
        if (blk_nz(I - J, lo, hi))
#pragma unroll
          for (int v = 0; v < 4; ++v) D.a[bidx(I, J)][v] = f(D.a[bidx(I, J)][v]);
  };
  if (s > 0) {
    const int h = (1 << (s - 1)) - 1;
    each([&](int y) { return (y + h + ((y >> s) & 1)) >> s; });
  } else if (s < 0) {
    each([&](int y) { return y << -s; });
  }
}

// exact int32 values (|y| < 2^30) of exponent e_in to codes by the scale
// rule, in place; exponent and non-zero flag through refs
template <int NB>
__device__ __forceinline__ void requant_i32(AccI<NB>& D, int lo, int hi, int e_in, int& e_out,
                                            bool& nz) {
  const int amax = amax_of(D, lo, hi);
  nz = amax > 0;
  if (!nz) {
    e_out = 0;
    return;
  }
  const int s = shift_canon<kQmax, 15>(amax);
  rescale_i32(D, s, lo, hi);
  e_out = e_in + s;
}

// codes (|q| <= 32639) to the finest scale that holds them (exact left
// shift), in place
template <int NB>
__device__ __forceinline__ void canon(AccI<NB>& q, int lo, int hi, int& e, bool& nz) {
  const int amax = amax_of(q, lo, hi);
  nz = amax > 0;
  if (!nz) {
    e = 0;
    return;
  }
  const int s = shift_canon<kQmax, 15>(amax);
  if (s < 0) {
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J <= I; ++J)
        if (blk_nz(I - J, lo, hi))
#pragma unroll
          for (int v = 0; v < 4; ++v) q.a[bidx(I, J)][v] <<= -s;
  }
  e += s;
}

// ---------------------------------------------------------------------------

// The INT16 width for the shared integer engine (int_engine of intq.hpp):
// limb quads, products and sums in int32 rounded to odd, or exact in fp64.
template <int NB> struct I16Ops {
  using Codes = AccI<NB>;
  using Row = RowL<NB>;
  using Col = ColL<NB>;
  static __device__ __forceinline__ bool any(const Codes& D, int lo, int hi) {
    return amax_of(D, lo, hi) > 0;
  }
  static constexpr int kQ = kQmax;
  static constexpr int kQB = 15;                                      // |code| < 2^15
  static constexpr int kAccB = 30 + (NB == 1 ? 4 : NB == 2 ? 5 : 6);  // |product| < C 2^30
  static __device__ __forceinline__ void to_row(Row& X, const AccI<NB>& D, int lo, int hi) {
    to_rowl(X, D, lo, hi);
  }
  static __device__ __forceinline__ void to_col(Col& Y, const AccI<NB>& D, int lo, int hi) {
    to_coll(Y, D, lo, hi);
  }
  // the codes 256 h + l of the blocks of X that can meet [lo, hi] (others 0)
  static __device__ __forceinline__ void codes(AccI<NB>& D, const Row& X, int lo, int hi) {
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J <= I; ++J)
        D.a[bidx(I, J)] = blk_nz(I - J, lo, hi)
                              ? unpack4(X.h.r[I].v[J]) * 256 + unpack4(X.l.r[I].v[J])
                              : zero_i4();
  }
  // the blocks f(I, J) of the band [lo, hi], the others 0
  template <typename Fn>
  static __device__ __forceinline__ void blocks(AccI<NB>& D, int lo, int hi, Fn&& f) {
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J <= I; ++J)
        D.a[bidx(I, J)] = blk_nz(I - J, lo, hi) ? f(I, J) : zero_i4();
  }
  // q(X Y 2^e_in) over [lo, hi] as codes and as row fragments (X and Y are
  // read before qr is written).  Rounded to odd at 1 / 128 when the shift from
  // there is at least 2 (a maximum of 2^16 or more); a smaller product is below
  // 2^23 and formed in int32 as it is.
  static __device__ __forceinline__ void mulq(const Row& X, const Col& Y, int lo, int hi, int e_in,
                                              Codes& q, Row& qr, int& e_out, bool& nz) {
    blocks(q, lo, hi, [&](int I, int J) { return odd_block(X, Y, I, J); });
    int amax = amax_of(q, lo, hi), e = e_in + 7;
    if (amax < (1 << 16)) {
      blocks(q, lo, hi, [&](int I, int J) { return exact_block(X, Y, I, J); });
      amax = amax_of(q, lo, hi);
      e = e_in;
    }
    nz = amax > 0;
    const int s = nz ? shift_canon<kQmax, 15>(amax) : 0;
    rescale_i32(q, s, lo, hi);
    e_out = nz ? e + s : 0;
    to_rowl(qr, q, lo, hi);
  }
  // out = q(x + y + sign X Y 2^ep), the product on the sub-diagonals from plo
  // on and absent when !pp.  In int32: the product, rounded to odd at 1 / 128
  // (units of 2^(ep + 7)), and the terms that are even integers below 2^29
  // there; then that sum rounded to odd t bits higher, so that the coarsest
  // term stays below 2^29, and the terms that are even integers from there on.
  // Valid when every term falls on one side and the final shift is at least 2;
  // else exactly in fp64.
  static __device__ __forceinline__ void mul_sum(Codes& out, int& eo, bool& nz,
                                                 const Term<Codes>& x, const Term<Codes>& y,
                                                 const Row& X, const Col& Y, int ep, int sign,
                                                 int plo, bool pp, int lo, int hi) {
    const int kx = x.p ? x.e - ep - 7 : 1, ky = y.p ? y.e - ep - 7 : 1;  // absent: zero codes
    const int t = max(0, max(kx, ky) - 14);
    const bool cx = kx - t >= 1, cy = ky - t >= 1;  // coarse: even at the coarser unit
    if (pp && t <= 30 && (cx || (kx >= 1 && kx <= 14)) && (cy || (ky >= 1 && ky <= 14))) {
      AccI<NB> r;
      // a term's shift before and after the rounding (32: not there)
      auto put = [&](i32x4& a, const Term<Codes>& q, int m, int b, int k) {
        if (blk_nz(m, q.lo, q.hi)) a += (q.t->a[b] * q.sign) << k;
      };
      blocks(r, lo, hi, [&](int I, int J) {
        i32x4 a = zero_i4();
        if (blk_nz(I - J, plo, hi)) a = odd_block(X, Y, I, J);
        return sign < 0 ? -a : a;
      });
      auto add_term = [&](const Term<Codes>& q, int k) {
        blocks(r, lo, hi, [&](int I, int J) {
          i32x4 a = r.a[bidx(I, J)];
          put(a, q, I - J, bidx(I, J), k);
          return a;
        });
      };
      if (!cx) add_term(x, kx);
      if (!cy) add_term(y, ky);
      if (t > 0)
        blocks(r, lo, hi, [&](int I, int J) { return odd_shift(r.a[bidx(I, J)], t); });
      if (cx) add_term(x, kx - t);
      if (cy) add_term(y, ky - t);
      const int amax = amax_of(r, lo, hi);
      if (amax >= (1 << 16)) {
        const int s = shift_canon<kQmax, 15>(amax);
        rescale_i32(r, s, lo, hi);
        out = r;
        eo = ep + 7 + t + s;
        nz = true;
        return;
      }
    }
    LazyProd<NB> D{{&X, &Y}};
    exact_sum<kQ, kQB, NB>(out, eo, nz, x, y, term(D, ep, kAccB, sign, plo, hi, pp), lo, hi);
  }
  static __device__ __forceinline__ void canon(AccI<NB>& q, int lo, int hi, int& e, bool& nz) {
    i16::canon(q, lo, hi, e, nz);
  }
  // X = q(X 2^eX + ys Y 2^eY) over [lo, hi] (X's band [xlo, hi], Y's
  // [ylo, hi]); Y is at the finest scale that holds it, and so is X when
  // xc.  Exponents 2 QB + 3 or more apart: the finer term is below an
  // eighth of the output quantum and leaves the coarser's codes as they are
  // (at their finest scale); at most 14 apart: the aligned sum is below
  // 32639 (2^14 + 1) < 2^30 and exact in int32, and so is its rounding;
  // between: the finer term rounded to odd at the unit 14 bits under the
  // coarser one's, where the coarser is an even integer of 2^27 or more at its
  // maximum, so the rounding that follows shifts by 12 or more and comes out
  // as that of the exact sum.
  static __device__ __forceinline__ void add(AccI<NB>& X, int& eX, bool& nzX, int xlo, bool xc,
                                             const AccI<NB>& Y, int eY, bool nzY, int ys, int ylo,
                                             int lo, int hi) {
    int g = !nzY ? 64 : nzX ? eX - eY : -64;
    if (!xc && g > 14) {
      canon(X, xlo, hi, eX, nzX);
      if (nzY && nzX) g = eX - eY;
    }
    if (g >= 2 * kQB + 3) return;
    if (g <= -(2 * kQB + 3)) {
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = 0; J <= I; ++J)
          if (blk_nz(I - J, lo, hi))
            X.a[bidx(I, J)] = blk_nz(I - J, ylo, hi) ? Y.a[bidx(I, J)] * ys : zero_i4();
      eX = eY;
      nzX = true;
      return;
    }
    auto each = [&](auto&& f) {
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = 0; J <= I; ++J)
          if (blk_nz(I - J, lo, hi))
            X.a[bidx(I, J)] = f(blk_nz(I - J, xlo, hi) ? X.a[bidx(I, J)] : zero_i4(),
                                blk_nz(I - J, ylo, hi) ? Y.a[bidx(I, J)] * ys : zero_i4());
    };
    int e0;
    if (g > 14) {
      each([&](i32x4 x, i32x4 y) { return (x << 14) + odd_shift(y, g - 14); });
      e0 = eX - 14;
    } else if (g >= 0) {
      each([&](i32x4 x, i32x4 y) { return (x << g) + y; });
      e0 = eY;
    } else if (g >= -14) {
      each([&](i32x4 x, i32x4 y) { return (y << -g) + x; });
      e0 = eX;
    } else {
      each([&](i32x4 x, i32x4 y) { return (y << 14) + odd_shift(x, -g - 14); });
      e0 = eY - 14;
    }
    requant_i32(X, lo, hi, e0, eX, nzX);
  }
  static __device__ __forceinline__ void row_to_col(Col& Y, const Row& X, const ColQ<NB>& Ic,
                                                    int lo, int hi) {
    i16::row_to_col<NB>(Y, X, Ic, lo, hi);
  }
};

// e = the smallest integer at which round-half-even(amax / 2^e) <= 32639
// (frexp: amax = m 2^p with m in [0.5, 1) gives amax / 2^(p - 15) =
// 32768 m, which rounds past 32639 when 32768 m >= 32639.5), 0 for
// amax = 0
__device__ __forceinline__ int quant_exp(float amax) {
  int e = 0;
  if (amax > 0.f) {
    int p;
    const float mant = frexpf(amax, &p);
    e = p - 15 + (mant * 32768.f >= 32639.5f ? 1 : 0);
  }
  return e;
}

}  // namespace i16
}  // namespace gdn
