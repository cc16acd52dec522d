// state.hip -- the state pass of the layer forward: the recurrence over the
// chunks of each head and the output (forward.hpp states the products).
//
// A workgroup walks the chunks of one head in order for NSL slices of 16
// value columns, with its dk x 16 NSL part of S in registers (fp32), spread
// over recurrence waves: wave w owns the state pair q = w (its 2 x 16 state
// rows) and the row block I = w of X.  Output waves form the rows of O; the
// RS workgroups of a slice carry the same recurrence and split the row blocks
// of O between them.  Per chunk two exchanges through LDS: the state pairs
// (rounded to the compute type) before K S and Q S, and X before G X and P' X.
//
// What bounds it: a chunk's step is serial, and a CU has to take the chunk's
// operands (K, G, Q, P': 54 KB in bf16 at C = 64, dk = 128, whatever NSL)
// through its L1.  Measured on MI355X, a wave load of 1 KB costs a CU 9 ns
// when consecutive lanes read consecutive 16 bytes of whole rows, and 31 ns in
// the fragment order (lane (g, c): row c, 16 bytes at 8g), where each group of
// 16 lanes touches 16 rows.  So loader waves (two or four) copy K, Q, V and the
// gates of the chunks ahead into LDS rows by DMA in row order, and the fragments
// are read from there; G and P' lie in the workspace as fragments and come
// straight into registers.
//
// Fragment conventions (tile16.hpp): a pair over 16-blocks {2p, 2p + 1}
// gives slot s of lane (g, c) the index 32p + 16 (s / 4) + 4g + s % 4; a
// pair loaded as a run of 8 features gives slot s the feature 32q + 8g + s.
// State block m = 2q' + h' holds, for block row r = 4g + v,
//   dk = 32 q' + 8 g + 4 h' + v,
// so that the pair (block 2q', block 2q' + 1) lines up with a run of 8
// features of K and Q rows.  Value columns of slice s of a workgroup at
// column base n0: NSL = 1, n0 + n; NSL = 2, n0 + 8 (n / 4) + 4 s + n % 4, so a
// lane's 4 columns of both slices are one run of 8.
#include <atomic>
#include <type_traits>

#include "forward.hpp"
#include "launch.hpp"

namespace gdn {

// half `hf` (block 2p + hf) of slot p
__device__ __forceinline__ void slot_store_half(__bf16* s, f32x4 x, int hf, int l) {
  *(bf16x4*)(s + 8 * l + 4 * hf) = __builtin_convertvector(x, bf16x4);
}
__device__ __forceinline__ void slot_store_half(float* s, f32x4 x, int hf, int l) {
  *(f32x4*)(s + 256 * hf + 4 * l) = x;
}

// LDS writes before the barrier are visible after it; global memory is not
// waited for (no wave reads what another wrote there)
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Values a wave has read from LDS before a barrier and uses after it: held in
// registers here (a read left to the compiler may sink past the barrier, into
// the time the buffer is refilled).
__device__ __forceinline__ void hold(float& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void hold(f32x4& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void hold(bf16x4& x) {
  int2 t = __builtin_bit_cast(int2, x);
  asm volatile("" : "+v"(t.x), "+v"(t.y));
  x = __builtin_bit_cast(bf16x4, t);
}
__device__ __forceinline__ void hold(Pair<bf16x4>& x) {
  i32x4 t = __builtin_bit_cast(i32x4, x.v);
  asm volatile("" : "+v"(t));
  x.v = __builtin_bit_cast(bf16x8, t);
}
__device__ __forceinline__ void hold(Pair<f32x4>& x) {
  hold(x.a);
  hold(x.b);
}

// Pairs over the chunk's rows and their products.  NB = 1: the second block of
// the pair does not exist (zeros); in fp32 it is neither loaded nor multiplied.
template <int NB, typename F, typename TIO>
__device__ __forceinline__ Pair<F> rows_load(const TIO* s, int l) {
  if constexpr (NB == 1 && sizeof(TIO) == 4)
    return Pair<F>::make(*(const f32x4*)(s + 4 * l), zero4());
  else
    return slot_load<F>(s, l);
}
template <int NB, bool OUTQ, typename F>
__device__ __forceinline__ f32x4 rows_mma(const Pair<F>& x, const Pair<F>& y, f32x4 acc) {
  if constexpr (NB == 1 && std::is_same_v<F, f32x4>) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(OUTQ ? y.a[v] : x.a[v], OUTQ ? x.a[v] : y.a[v],
                                                 acc, 0, 0, 0);
    return acc;
  } else {
    return Pair<F>::template mma<OUTQ>(x, y, acc);
  }
}

// NSL x 4 consecutive values of a row
template <typename F, int NSL> struct Run { Pair<F> v; };
template <typename F> struct Run<F, 1> { F v; };
__device__ __forceinline__ Pair<bf16x4> lo_pair(bf16x4 x) {
  const bf16x4 z = __builtin_convertvector(zero4(), bf16x4);
  return Pair<bf16x4>{__builtin_shufflevector(x, z, 0, 1, 2, 3, 4, 5, 6, 7)};
}
__device__ __forceinline__ Pair<f32x4> lo_pair(f32x4 x) { return Pair<f32x4>::make(x, zero4()); }

// LDS rows of D values in 16-byte pieces: piece p of row r lies at position
// p ^ (r & SW), so the 16 lanes that read one piece of 16 rows meet 16
// different groups of banks.
template <int D, typename TIO>
struct SwzRows {
  static constexpr int E = 16 / sizeof(TIO);          // values a piece
  static constexpr int CPR = D / E;                   // pieces a row: 8, 16, 32
  static constexpr int SW = CPR < 16 ? CPR - 1 : 15;  // swizzle mask
  static constexpr int RPI = 64 / CPR;                // rows a wave copies at once
  // pair of features 32q + 8g .. 32q + 8g + 7 of row r
  template <typename F>
  static __device__ __forceinline__ Pair<F> pair(const TIO* s, int r, int q, int g) {
    if constexpr (sizeof(TIO) == 2) {
      return Pair<F>{*(const bf16x8*)(s + r * D + ((4 * q + g) ^ (r & SW)) * E)};
    } else {
      const int p = 8 * q + 2 * g;
      return Pair<F>{*(const f32x4*)(s + r * D + (p ^ (r & SW)) * E),
                     *(const f32x4*)(s + r * D + ((p + 1) ^ (r & SW)) * E)};
    }
  }
};

// one wave's copy of 16 bytes a lane into 1 KB of LDS at s
template <typename TIO>
__device__ __forceinline__ void dma16(const TIO* src, TIO* s) {
  __builtin_amdgcn_global_load_lds((glb_void*)src, (lds_void*)s, 16, 0, 0);
}

// The sizes of a workgroup of the state pass.
//   NSL: slices of 16 value columns; RS: workgroups that share the row blocks
//   of O; R: chunks in the LDS ring
template <int NB, int DK, typename TIO, int NSL, int RS, int R>
struct StateShape {
  static constexpr int C = 16 * NB, NQ = DK / 32, NP = npair(NB);
  static constexpr int SWV = NB > NQ ? NB : NQ;  // recurrence waves
  // loader waves: a wave issues a copy of strided rows every 27 ns, a CU takes
  // one every 10 ns.  Two only in fp32 and for the small chunks of dk = 128: a
  // third wave on a SIMD leaves 168 registers a lane, and 4 to 12 of those
  // chunks' values went to scratch
  static constexpr int LW = sizeof(TIO) == 2 && (NB >= 4 || DK == 64) ? 4 : 2;
  // row blocks of O an output wave forms: one, but in fp32 two where more
  // output waves would be the third wave on a SIMD: two slices take 200
  // registers a lane of the 168 that leaves; one slice fits, and is slower all
  // the same (us of the layer at 2048 tokens, C = 64, 17 heads 151 against 148;
  // dk = 64, 32 heads 131 against 107)
  static constexpr int OB = sizeof(TIO) == 4 && SWV + NB / RS + LW > 8 ? 2 : 1;
  static constexpr int OW = NB / RS / OB;  // output waves
  static constexpr int WAVES = SWV + OW + LW;
  // The first output and loader wave.  Waves go to the four SIMDs in turn; where
  // only the first of four recurrence waves have rows (NB < 4), the loaders come
  // before the output waves, which then have SIMDs of their own (us of the
  // layer at 2048 tokens, 4 heads, fp32: C = 32 119 -> 97, C = 16 186 -> 144;
  // bf16 within 3 %).
  static constexpr bool LFIRST = SWV == 4 && NB < 4;
  static constexpr int O0 = SWV + (LFIRST ? LW : 0), L0 = SWV + (LFIRST ? 0 : OW);
  // Workgroups a CU is to hold.  fp32, one slice each without sharing: two
  // where their LDS fits, as the launch rule counts on (run_state).
  static constexpr bool TWO =
      sizeof(TIO) == 4 && NSL == 1 && RS == 1 && (NB == 1 || (NB == 4 && DK == 64 && R == 1));
  static constexpr int PER_SIMD = (TWO ? 2 : 1) * ((WAVES + 3) / 4);  // waves
  using KR = SwzRows<DK, TIO>;
  static constexpr int KI = C / KR::RPI, QI = 16 * OW * OB / KR::RPI;  // copies a chunk
  static constexpr int VL = NSL * 16 * (int)sizeof(TIO) / 16;     // lanes a row of V
  static constexpr int VR = 64 / VL;                              // rows of V a copy
  static constexpr int VI = (C + VR - 1) / VR;
  static constexpr int VN = VI * 64 * KR::E;  // values of V in LDS (whole copies)
  // copies a loader wave and chunk; where a count does not divide, the last
  // copy is made more than once (the same bytes)
  static constexpr int KW = (KI + LW - 1) / LW, QW = (QI + LW - 1) / LW;
  static constexpr int CW = KW + QW + (VI < LW ? 1 : VI / LW + 1);
  static_assert(VI < LW || VI % LW == 0, "");
  static_assert((R - 1) * CW < 64, "vmcnt counts to 63");
};

// VARLEN: one state per (packed sequence, head); the sequence's chunks in
// order, their tiles at h * nchunks + chunk; rows of a chunk past its m
// tokens are read from row m - 1 (their columns of G and P' are zero) and not
// stored (O).  Tables that do not describe chunks of C tokens inside the T
// tokens and nchunks tiles make the sequence empty (its final state is its
// initial one).
// The grid: heads bh0 .. bh0 + nbh - 1 (bh = b H + h), padded to whole groups
// of 8: work items are dealt to the 8 XCDs in turn and XCD k takes the heads
// bh0 + k, bh0 + k + 8, ... whole, so the operands that a head's workgroups
// all read meet in one L2.
template <int NB, int DK, int DV, typename F, typename TIO, int NSL, int RS, int R, bool VARLEN>
__global__ __launch_bounds__((64 * StateShape<NB, DK, TIO, NSL, RS, R>::WAVES),
                             (StateShape<NB, DK, TIO, NSL, RS, R>::PER_SIMD)) void k_fwd_state(
    const TIO* __restrict__ ws, const TIO* __restrict__ Q, const TIO* __restrict__ K,
    const TIO* __restrict__ V, const float* __restrict__ gam, int gtiles,
    const float* __restrict__ S0, TIO* __restrict__ O, float* __restrict__ Sfin, int64_t n_tiles,
    int bh0, int nbh, int L, int H, float scale, Packed pk) {
  using SH = StateShape<NB, DK, TIO, NSL, RS, R>;
  using LY = FwdLayout<NB, DK, DV>;
  using KR = typename SH::KR;
  constexpr int C = SH::C, NQ = SH::NQ, NP = SH::NP, NS = DV / (16 * NSL);
  constexpr int SW = SH::SWV, OW = SH::OW, OB = SH::OB;
  constexpr int PS = sizeof(TIO) == 4 ? 2 : 1;  // partial sums of a product with the state
  // Register sets of G and P': bf16 loads the next chunk's while it works on
  // this one's.  fp32 loads its own at the state barrier, behind the product
  // with the state, which takes longer than the load (us of the layer at 2048
  // tokens, 16 heads, C = 64: 143 -> 136) but for the smallest (C = 32, dk = 64:
  // 72 -> 74), and half the registers.
  constexpr int GD = sizeof(TIO) == 4 && !(NB == 2 && DK == 64) ? 1 : 2;
  __shared__ __attribute__((aligned(16))) TIO sK[R][C * DK];
  __shared__ __attribute__((aligned(16))) TIO sQ[R][16 * OW * OB * DK];
  __shared__ __attribute__((aligned(16))) TIO sV[R][SH::VN];
  __shared__ __attribute__((aligned(16))) float sg[R][64];
  __shared__ __attribute__((aligned(16))) TIO xs[NSL][NQ * 512];  // state pairs
  __shared__ __attribute__((aligned(16))) TIO xv[NSL][NP * 512];  // X pairs
  const uint32_t x = blockIdx.x, xr = x >> 3;
  const int rs = (int)(xr % RS), j = (int)(xr / RS % NS);
  const int bi = (int)(xr / (RS * NS) * 8 + (x & 7));
  if (bi >= nbh) return;  // the whole workgroup, before any barrier
  const int bh = bh0 + bi, b = bh / H, h = bh - b * H;  // b: the sequence when VARLEN
  // this head's chunks: c0 .. c0 + nc - 1, the first at token tokS; len tokens
  int nc = L / C, c0 = 0, len = L;
  int64_t tokS = (int64_t)b * L;
  if constexpr (VARLEN) {
    const int t0 = pk.cu[b], t1 = pk.cu[b + 1], o0 = pk.off[b], o1 = pk.off[b + 1];
    len = t1 - t0;
    nc = o1 - o0;
    c0 = o0;
    tokS = t0;
    const bool ok = t0 >= 0 && len >= 0 && t1 <= L && o0 >= 0 && nc >= 0 && o1 <= pk.nchunks &&
                    nc == (len + C - 1) / C;
    if (!ok) nc = 0;
  }
  const int last = nc - 1;
  // tokens of chunk ck (C, or fewer in a sequence's last chunk)
  auto rows_of = [&](int ck) __attribute__((always_inline)) { return VARLEN ? min(C, len - ck * C) : C; };
  // workspace tiles: chunks first, heads inside, so that the heads, which
  // walk their chunks side by side, read one contiguous stretch
  const int64_t tile0 = ((int64_t)(VARLEN ? c0 : b * nc) * H + h);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Lane ln = lane_here();
  const int l = ln.id, gq = ln.g(), c = ln.c();
  const TIO* wsG = ws + tile0 * LY::G;
  const TIO* wsP = ws + n_tiles * LY::G + tile0 * LY::P;

  if (wv < SW) {
    // ---- recurrence wave
    const bool rows = NB >= SW || wv < NB, owner = NQ >= SW || wv < NQ;
    const int I = wv;
    const f32x4 e = eye4(ln);
    const Pair<F> id[2] = {Pair<F>::make(e, zero4()), Pair<F>::make(zero4(), e)};
    const int64_t sbase = (int64_t)bh * DK * DV;
    // state row 32 wv + 8g + 4 hf + v, value column of column c of slice s
    auto sidx = [&](int s, int hf, int v) __attribute__((always_inline)) {
      const int col = NSL == 1 ? 16 * j + c : 32 * j + 8 * (c >> 2) + 4 * s + (c & 3);
      return sbase + (int64_t)(32 * wv + 8 * gq + 4 * hf + v) * DV + col;
    };
    f32x4 st[NSL][2];
#pragma unroll
    for (int s = 0; s < NSL; ++s)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        st[s][hf] = zero4();
        if (owner && S0)
#pragma unroll
          for (int v = 0; v < 4; ++v) st[s][hf][v] = S0[sidx(s, hf, v)];
      }
    if (NB == 1 && rows) {  // block 1 of the X pair does not exist: a zero half
#pragma unroll
      for (int s = 0; s < NSL; ++s) slot_store_half(xv[s], zero4(), 1, l);
    }
    struct GOps {
      Pair<F> x[2][NP];  // G pairs of the owned state blocks
    };
    auto load_g = [&](GOps& op, int64_t ck) __attribute__((always_inline)) {
      if (owner)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int p = 0; p < NP; ++p)
            op.x[hf][p] =
                rows_load<NB, F>(wsG + ck * H * LY::G + ((2 * wv + hf) * NP + p) * 512, l);
    };
    // this chunk's K row pairs, V row and gammas, from LDS
    Pair<F> kr[NQ];
    Run<F, NSL> vr;
    f32x4 gr = zero4();
    float gl = 0.f;
    auto read_rows = [&](int buf) __attribute__((always_inline)) {
      if (rows) {
        const int r = I * 16 + c;
#pragma unroll
        for (int q = 0; q < NQ; ++q) kr[q] = KR::template pair<F>(sK[buf], r, q, gq);
        if constexpr (NSL == 1)
          vr.v = *(const F*)(sV[buf] + r * 16 + 4 * gq);
        else
          vr.v = load_row8<F>(sV[buf] + r * 32 + 8 * gq);
        gr = *(const f32x4*)(sg[buf] + I * 16 + 4 * gq);
      }
      gl = sg[buf][C - 1];
    };
    auto compute = [&](const GOps& op, GOps& nx, int cknx, int bufnx) __attribute__((always_inline)) {
      if (owner)
#pragma unroll
        for (int s = 0; s < NSL; ++s)
          slot_store(xs[s] + wv * 512, Pair<F>::make(st[s][0], st[s][1]), l);
      __builtin_amdgcn_sched_barrier(0);
      // what the step needs of the rows read earlier, formed while the other
      // waves arrive: V in column form (exact: one entry times 1), e^gamma
      f32x4 vc[NSL], eg;
      hold(gl);
      float el = __expf(gl);
      hold(el);
      if (rows) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) hold(kr[q]);
        hold(vr.v);
        hold(gr);
#pragma unroll
        for (int s = 0; s < NSL; ++s) {
          if constexpr (NSL == 1)
            vc[s] = Pair<F>::template mma<false>(lo_pair(vr.v), id[0], zero4());
          else
            vc[s] = Pair<F>::template mma<false>(vr.v, id[s], zero4());
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) eg[v] = __expf(gr[v]);
        hold(eg);
      }
      __builtin_amdgcn_sched_barrier(0);
      lds_barrier();  // state pairs published
      if (rows) {
        Pair<F> sp[NSL][NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int s = 0; s < NSL; ++s) sp[s][q] = slot_load<F>(xs[s] + q * 512, l);
        __builtin_amdgcn_sched_barrier(0);
        load_g(nx, cknx);
        __builtin_amdgcn_sched_barrier(0);
        // (fp32: two partial sums, whose roundings are smaller than one's)
        f32x4 ks[NSL][PS];
#pragma unroll
        for (int s = 0; s < NSL; ++s)
#pragma unroll
          for (int u = 0; u < PS; ++u) ks[s][u] = zero4();
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int s = 0; s < NSL; ++s)
            ks[s][q % PS] = Pair<F>::template mma<false>(kr[q], sp[s][q], ks[s][q % PS]);
#pragma unroll
        for (int s = 0; s < NSL; ++s) {
          if constexpr (PS == 2) ks[s][0] += ks[s][1];
          f32x4 xc;
#pragma unroll
          for (int v = 0; v < 4; ++v) xc[v] = vc[s][v] - eg[v] * ks[s][0][v];
          slot_store_half(xv[s] + (I >> 1) * 512, xc, I & 1, l);
        }
      } else {
        load_g(nx, cknx);
      }
      lds_barrier();  // X published; the next chunk's rows are in LDS
      Pair<F> xp[NSL][NP];
      if (owner)
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int s = 0; s < NSL; ++s) xp[s][p] = rows_load<NB, F>(xv[s] + p * 512, l);
      __builtin_amdgcn_sched_barrier(0);
      read_rows(bufnx);
      __builtin_amdgcn_sched_barrier(0);
      if (owner) {
        // fp32: the decayed state is added last, so that only the last
        // addition rounds at its size
        f32x4 old[NSL][2];
#pragma unroll
        for (int s = 0; s < NSL; ++s)
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            old[s][hf] = st[s][hf];
            st[s][hf] = PS == 2 ? zero4() : old[s][hf] * el;
          }
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int s = 0; s < NSL; ++s)
#pragma unroll
            for (int hf = 0; hf < 2; ++hf)
              st[s][hf] = rows_mma<NB, false>(op.x[hf][p], xp[s][p], st[s][hf]);
        if constexpr (PS == 2)
#pragma unroll
          for (int s = 0; s < NSL; ++s)
#pragma unroll
            for (int hf = 0; hf < 2; ++hf)
#pragma unroll
              for (int v = 0; v < 4; ++v)
                st[s][hf][v] = __builtin_fmaf(el, old[s][hf][v], st[s][hf][v]);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    // Chunk indices of loads are clamped to the last chunk (a repeated load
    // past the end is harmless), which keeps the loads free of branches.
    if (nc > 0) {
      GOps r[GD];
#pragma unroll
      for (int d = 0; d + 1 < GD; ++d) load_g(r[d], min(d, last));
      lds_barrier();  // chunk 0 is in LDS
      read_rows(0);
      int ck = 0, buf = 0;
      auto next = [&]() __attribute__((always_inline)) { return buf = buf + 1 < R ? buf + 1 : 0; };
      for (; ck + GD <= nc; ck += GD) {
#pragma unroll
        for (int d = 0; d < GD; ++d)
          compute(r[d], r[(d + GD - 1) % GD], min(ck + d + GD - 1, last), next());
      }
#pragma unroll
      for (int d = 0; d + 1 < GD; ++d)
        if (ck + d < nc) compute(r[d], r[(d + GD - 1) % GD], last, next());
    }
    if (owner && Sfin && rs == 0) {
#pragma unroll
      for (int s = 0; s < NSL; ++s)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int v = 0; v < 4; ++v) Sfin[sidx(s, hf, v)] = st[s][hf][v];
    }
  } else if (wv >= SH::O0 && wv < SH::O0 + OW) {
    // ---- output wave: OB row blocks of O; the same barriers
    const int o_ = wv - SH::O0;
    // this workgroup's block number of block n of the wave (a first and a last
    // one: the later the block, the more of P' there is), and the chunk's
    auto bno = [&](int n) __attribute__((always_inline)) { return n == 0 ? o_ : OB * OW - 1 - o_; };
    auto blkI = [&](int n) __attribute__((always_inline)) { return bno(n) * RS + rs; };
    const int64_t ldo = (int64_t)H * DV;
    TIO* ob = O + tokS * ldo + (int64_t)h * DV + 16 * NSL * j + 4 * NSL * gq + c * ldo;
    struct POps {
      Pair<F> p[OB][2];  // P' row pairs (I, p), p <= I / 2
    };
    auto load_p = [&](POps& op, int64_t ck) __attribute__((always_inline)) {
#pragma unroll
      for (int n = 0; n < OB; ++n)
#pragma unroll
        for (int p = 0; p < 2; ++p)
          if (2 * p <= blkI(n))
            op.p[n][p] = rows_load<NB, F>(wsP + ck * H * LY::P + pidx(blkI(n), p) * 512, l);
    };
    Pair<F> qr[OB][NQ];
    float gr[OB];
    auto read_rows = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
      for (int n = 0; n < OB; ++n) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          qr[n][q] = KR::template pair<F>(sQ[buf], bno(n) * 16 + c, q, gq);
        gr[n] = sg[buf][blkI(n) * 16 + c];
      }
    };
    auto compute = [&](const POps& op, int ck, POps& nx, int cknx, int bufnx) __attribute__((always_inline)) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int n = 0; n < OB; ++n) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) hold(qr[n][q]);
        hold(gr[n]);
      }
      lds_barrier();  // state pairs published
      Pair<F> sp[NSL][NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int s = 0; s < NSL; ++s) sp[s][q] = slot_load<F>(xs[s] + q * 512, l);
      __builtin_amdgcn_sched_barrier(0);
      load_p(nx, cknx);
      __builtin_amdgcn_sched_barrier(0);
      f32x4 o[OB][NSL];
#pragma unroll
      for (int n = 0; n < OB; ++n) {
        const float eg = __expf(gr[n]);
        f32x4 qs[NSL][PS];
#pragma unroll
        for (int s = 0; s < NSL; ++s)
#pragma unroll
          for (int u = 0; u < PS; ++u) qs[s][u] = zero4();
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int s = 0; s < NSL; ++s)
            qs[s][q % PS] = Pair<F>::template mma<true>(qr[n][q], sp[s][q], qs[s][q % PS]);
#pragma unroll
        for (int s = 0; s < NSL; ++s) {
          if constexpr (PS == 2) qs[s][0] += qs[s][1];
          o[n][s] = eg * qs[s][0];
          hold(o[n][s]);  // the state pairs are read before the barrier
        }
      }
      lds_barrier();  // X published; the next chunk's rows are in LDS
      Pair<F> xp[NSL][2];
#pragma unroll
      for (int p = 0; p < 2; ++p)
        if (2 * p <= (OB > 1 ? NB - 1 : blkI(0)))
#pragma unroll
          for (int s = 0; s < NSL; ++s) xp[s][p] = rows_load<NB, F>(xv[s] + p * 512, l);
      __builtin_amdgcn_sched_barrier(0);
      read_rows(bufnx);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int n = 0; n < OB; ++n) {
        const int I = blkI(n);
        // (fp32: the share of the state is added last)
        f32x4 first[NSL];
#pragma unroll
        for (int s = 0; s < NSL; ++s) {
          first[s] = o[n][s];
          if constexpr (PS == 2) o[n][s] = zero4();
        }
#pragma unroll
        for (int p = 0; p < 2; ++p)
          if (2 * p <= I)
#pragma unroll
            for (int s = 0; s < NSL; ++s)
              o[n][s] = rows_mma<NB, true>(op.p[n][p], xp[s][p], o[n][s]);
        if constexpr (PS == 2)
#pragma unroll
          for (int s = 0; s < NSL; ++s) o[n][s] += first[s];
        if (!VARLEN || I * 16 + c < rows_of(ck)) {
          TIO* op_ = ob + ((int64_t)ck * C + I * 16) * ldo;
          if constexpr (NSL == 1)
            store4(op_, scale * o[n][0]);
          else
            store_row8(op_, scale * o[n][0], scale * o[n][1]);
        }
      }
    };
    if (nc > 0) {
      POps r[GD];
#pragma unroll
      for (int d = 0; d + 1 < GD; ++d) load_p(r[d], min(d, last));
      lds_barrier();  // chunk 0 is in LDS
      read_rows(0);
      int ck = 0, buf = 0;
      auto next = [&]() __attribute__((always_inline)) { return buf = buf + 1 < R ? buf + 1 : 0; };
      for (; ck + GD <= nc; ck += GD) {
#pragma unroll
        for (int d = 0; d < GD; ++d)
          compute(r[d], ck + d, r[(d + GD - 1) % GD], min(ck + d + GD - 1, last), next());
      }
#pragma unroll
      for (int d = 0; d + 1 < GD; ++d)
        if (ck + d < nc) compute(r[d], ck + d, r[(d + GD - 1) % GD], last, next());
    }
  } else if (nc > 0) {
    // ---- loader: R chunks ahead, the copies of a chunk dealt to the LW waves.
    // Chunk ck is read between the X barrier of chunk ck - 1 and the state
    // barrier of chunk ck, so its buffer is refilled (chunk ck + R) after that
    // barrier, and it has landed when all but the copies of the R - 1 chunks
    // issued after it have.
    constexpr int LW = SH::LW;
    const int w = wv - SH::L0;
    // K and V rows: the inputs, or the workspace's copies of the tile
    const bool copies = !VARLEN && K == nullptr;
    const int64_t krow = copies ? DK : (int64_t)H * DK, vrow = copies ? DV : (int64_t)H * DV;
    const int64_t qrow = (int64_t)H * DK;
    const int64_t kstep = copies ? (int64_t)H * C * DK : C * krow;  // chunk to chunk
    const int64_t vstep = copies ? (int64_t)H * C * DV : C * vrow;
    const int64_t gstep = gtiles ? (int64_t)H * C : (int64_t)C * H, gstride = gtiles ? 1 : H;
    const TIO* kb = copies ? ws + n_tiles * (LY::G + LY::P) + tile0 * LY::KC
                           : K + tokS * krow + (int64_t)h * DK;
    const TIO* vb = (copies ? ws + n_tiles * (LY::G + LY::P + LY::KC) + tile0 * LY::VC
                            : V + tokS * vrow + (int64_t)h * DV) + 16 * NSL * j;
    const TIO* qb = Q + tokS * qrow + (int64_t)h * DK;
    const float* gb = gtiles ? gam + tile0 * C : gam + tokS * H + h;
    const int rl = l / KR::CPR;  // this lane's row and piece of a copy of K or Q
    const int pc = (l % KR::CPR) ^ ((w * KR::RPI + rl) & KR::SW);
    const int vl = l / SH::VL;
    auto copy = [&](int ck, int buf, auto clamp_tag) __attribute__((always_inline)) {
      constexpr bool CL = decltype(clamp_tag)::value;  // rows past m are row m - 1
      const int m = CL ? rows_of(ck) : C;
      auto src = [&](const TIO* base, int r0, int dr, int64_t ld) __attribute__((always_inline)) {
        if constexpr (CL) return base + min(r0 + dr, m - 1) * ld;
        return base + r0 * ld + dr * ld;  // uniform part, then the lane's
      };
      const TIO* kc = kb + ck * kstep;
#pragma unroll
      for (int n = 0; n < SH::KW; ++n) {
        const int i = SH::KI % LW ? min(w + LW * n, SH::KI - 1) : w + LW * n;
        const int pn = SH::KI % LW ? (l % KR::CPR) ^ ((i * KR::RPI + rl) & KR::SW)
                                   : pc ^ ((n * LW * KR::RPI) & KR::SW);
        dma16(src(kc, i * KR::RPI, rl, krow) + pn * KR::E, sK[buf] + i * 64 * KR::E);
      }
      const TIO* qc = qb + (int64_t)ck * C * qrow;
#pragma unroll
      for (int n = 0; n < SH::QW; ++n) {
        const int i = SH::QI % LW ? min(w + LW * n, SH::QI - 1) : w + LW * n;
        const int pn = SH::QI % LW ? (l % KR::CPR) ^ ((i * KR::RPI + rl) & KR::SW)
                                   : pc ^ ((n * LW * KR::RPI) & KR::SW);
        const int r0 = ((i * KR::RPI >> 4) * RS + rs) * 16 + ((i * KR::RPI) & 15);
        dma16(src(qc, r0, rl, qrow) + pn * KR::E, sQ[buf] + i * 64 * KR::E);
      }
      const TIO* vc = vb + ck * vstep + (l % SH::VL) * KR::E;
      const float* gc = gb + ck * gstep;
      auto copy_v = [&](int i) __attribute__((always_inline)) {
        dma16(C % SH::VR ? vc + min(i * SH::VR + vl, m - 1) * vrow : src(vc, i * SH::VR, vl, vrow),
              sV[buf] + i * 64 * KR::E);
      };
      auto copy_g = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_global_load_lds((glb_void*)(gc + min(l, m - 1) * gstride),
                                         (lds_void*)sg[buf], 4, 0, 0);
      };
      if constexpr (SH::VI < LW) {
        if (w < SH::VI) copy_v(w); else copy_g();
      } else {
#pragma unroll
        for (int n = 0; n < SH::VI / LW; ++n) copy_v(w + LW * n);
        copy_g();
      }
    };
    auto issue = [&](int ck, int buf) __attribute__((always_inline)) {
      if (VARLEN && rows_of(ck) < C)
        copy(ck, buf, std::true_type{});
      else
        copy(ck, buf, std::false_type{});
    };
#pragma unroll 1
    for (int d = 0; d < R; ++d) issue(min(d, last), d);
    int buf = 0;
#pragma unroll 1
    for (int ck = 0; ck < nc; ++ck) {
      // all but this wave's newest (R - 1) chunks of copies are done
      constexpr int N = (R - 1) * SH::CW;
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
      __builtin_amdgcn_s_barrier();  // chunk ck is in LDS
      __builtin_amdgcn_s_barrier();  // and has been read
      __builtin_amdgcn_sched_barrier(0);
      issue(min(ck + R, last), buf);
      buf = buf + 1 < R ? buf + 1 : 0;
    }
    __builtin_amdgcn_s_barrier();  // the last chunk's X barrier
    wait_vmem();                   // no copy outlives the workgroup's LDS
  }
}

// ---------------------------------------------------------------------------

// Compute units of the current device, looked up once per device.  Host threads
// may ask at the same time: each then stores the same number.
static int compute_units() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

template <int NB, int DK, int DV, typename F, typename TIO>
hipError_t run_state(const TIO* ws, const TIO* Q, const TIO* K, const TIO* V, const float* gam,
                     bool gtiles, const float* S0, TIO* O, float* Sfin, int64_t n_tiles, int B,
                     int L, int H, float scale, const Packed& pk, hipStream_t st) {
  const bool packed = pk.cu != nullptr;
  const int64_t BH = (int64_t)(packed ? pk.nseq : B) * H;
  const int cus = compute_units();
#define GDN_STATE(NSL, RS, R, VL)                                                              \
  do {                                                                                         \
    using SH = StateShape<NB, DK, TIO, NSL, RS, R>;                                            \
    constexpr int64_t per = RS * (DV / 16 / NSL), NT = 64 * SH::WAVES;                         \
    constexpr int64_t most = ((int64_t)1 << 31) / (per * NT) / 8 * 8;  /* heads a launch */    \
    for (int64_t bh = 0; bh < BH; bh += most) {                                                \
      const int64_t n = BH - bh < most ? BH - bh : most;                                       \
      hipLaunchKernelGGL((k_fwd_state<NB, DK, DV, F, TIO, NSL, RS, R, VL>),                    \
                         dim3((unsigned)((n + 7) / 8 * 8 * per)), dim3(NT), 0, st, ws, Q, K,   \
                         V, gam, (int)gtiles, S0, O, Sfin, n_tiles, (int)bh, (int)n, L, H, scale, pk);  \
    }                                                                                          \
    return hipGetLastError();                                                                  \
  } while (0)
#define GDN_STATE_V(NSL, RS, R) \
  do { if (packed) GDN_STATE(NSL, RS, R, true); else GDN_STATE(NSL, RS, R, false); } while (0)
  // Which shape (MI355X, dk = dv = 128; S_final in place rules out RS > 1: a
  // workgroup that starts late would read the new state).
  // bf16, us per chunk of 64 of the state pass, us of the layer at 4096 tokens:
  //   one slice, two workgroups sharing O, while these fit the CUs: 16 heads
  //     0.62 (one workgroup a slice 0.75; two slices, two sharing 0.72);
  //   two slices, two workgroups sharing O, while these fit, C = 64: 32 heads
  //     1.08 (one slice each 1.30, two slices without sharing 1.35); C = 32 only
  //     with dk = 128, dv = 64 (64 heads 116, one slice each 121; dv = 128, 32
  //     heads 87, 82);
  //   one slice each while these fit: in place, C = 64, 4 heads 59 (two slices
  //     65), 32 heads 77 (81); C = 32, 8 heads 67 (84); C = 16, 8 heads 114
  //     (140), 32 heads 131 (145);
  //   two slices, no sharing beyond: 64 heads 1.51 (sharing 2.12, one slice
  //     2.57).
  // fp32, us of the layer at 2048 tokens:
  //   one slice, two workgroups sharing O, while these fit the CUs: C = 64, 16
  //     heads 137 (one workgroup a slice 148);
  //   one slice, one workgroup, while these fit: C = 64, 32 heads 155;
  //   beyond, a CU has to work on two slices at once or the launch takes two
  //     rounds.  One workgroup of two slices reads the chunk's operands once for
  //     both: C = 64, 48 heads 266, one slice each 320; C = 32, dk = 128, 48
  //     heads 189, 257; C = 16, dk = 128, 48 heads 273, two workgroups of one
  //     slice a CU 284.  At C = 64, dk = 128 its LDS has room for one chunk, not
  //     two: the copies of the next one hide behind the products.
  //   Workgroups of one slice, two or three on a CU, at dk = 64 (dv = 128: C =
  //     64, 128 heads 386, two slices 403; C = 32, 65 heads 202, 222; C = 16, 64
  //     heads 171, 200), and where two slices each would just begin another
  //     round at C = 16 (dk = 128: 65 heads 395, 516; 80 heads 491, 532; 96 heads
  //     552, 545; dk = 64: 128 heads 325, 324).
  // The ring (R) of two chunks: three and four measured the same; one where two
  // do not fit the LDS that the workgroups of a CU share.
  const int64_t slices = BH * (DV / 16);
  const bool share = !(S0 && S0 == Sfin);
  if constexpr (sizeof(TIO) == 2) {
    if constexpr (NB > 1) {
      if (2 * slices <= cus && share) GDN_STATE_V(1, 2, 2);
      if constexpr (NB == 4 || (DK == 128 && DV == 64))
        if (slices <= cus && share) GDN_STATE_V(2, 2, 2);
    }
    if (slices <= cus) GDN_STATE_V(1, 1, 2);
    GDN_STATE_V(2, 1, 2);
  } else {
    if constexpr (NB > 1)
      if (2 * slices <= cus && share) GDN_STATE_V(1, 2, 2);
    if (slices <= cus) GDN_STATE_V(1, 1, 2);
    if constexpr (NB > 1 && DK == 64) {
      GDN_STATE_V(1, 1, NB == 4 ? 1 : 2);
    } else {
      if constexpr (NB == 1)
        if (2 * slices <= 5 * cus && (DK == 64 || slices > 2 * cus)) GDN_STATE_V(1, 1, 2);
      GDN_STATE_V(2, 1, NB * DK <= 256 ? 2 : 1);
    }
  }
#undef GDN_STATE_V
#undef GDN_STATE
}

#define GDN_STATE_INST(NB, DK, DV)                                                               \
  template hipError_t run_state<NB, DK, DV, bf16x4, __bf16>(                                     \
      const __bf16*, const __bf16*, const __bf16*, const __bf16*, const float*, bool,            \
      const float*, __bf16*, float*, int64_t, int, int, int, float, const Packed&, hipStream_t); \
  template hipError_t run_state<NB, DK, DV, f32x4, float>(                                       \
      const float*, const float*, const float*, const float*, const float*, bool, const float*,  \
      float*, float*, int64_t, int, int, int, float, const Packed&, hipStream_t);
#define GDN_STATE_INST_D(NB)                              \
  GDN_STATE_INST(NB, 64, 64) GDN_STATE_INST(NB, 64, 128)  \
  GDN_STATE_INST(NB, 128, 64) GDN_STATE_INST(NB, 128, 128)
GDN_STATE_INST_D(1)
GDN_STATE_INST_D(2)
GDN_STATE_INST_D(4)

}  // namespace gdn
