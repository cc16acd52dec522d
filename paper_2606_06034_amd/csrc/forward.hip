// forward.hip -- the chunk-wise Gated DeltaNet forward around the chunk
// inverse: per chunk the WY factors, then the state recurrence across the
// chunks of a head and the output (the chunk-level recurrence of Gated
// DeltaNet that Section 1 builds on; Y = T^-1 X of Appendix E).
//
// Two launches (the products of each and the workspace between them:
// forward.hpp).  Stage 1, k_fwd_chunk here: one wave per chunk, every chunk
// in parallel.  Forms T (Neumann engine, exact block-wise inverse or integer
// T_hat), then P' and G, and stores them in the workspace in exactly the
// register-fragment layouts stage 2 feeds to its MFMAs.  Stage 2, k_fwd_state
// in state.hip, walks the chunks of every head in order.
#include <mutex>
#include <type_traits>

#include "forward.hpp"
#include "int16_ops.hpp"
#include "int8_ops.hpp"
#include "launch.hpp"

namespace gdn {

// The workspace a caller provides, in elements of the IO type per chunk tile:
// G, P' and the copies of K and V of the two-call form (forward.hpp).  The
// one-call form, whose second launch reads K and V themselves, keeps the
// chunk's gates behind G and P' instead.
int64_t fwd_workspace_elems(int C, int dk, int dv) {
  const int NB = C / 16, np = (NB + 1) / 2;
  return (int64_t)NB * (dk / 32) * 512 + (int64_t)(dv / 16) * NB * 256 +
         (int64_t)(dk / 16) * np * 512 + (int64_t)npp(NB) * 512;
}

// Column-form block of a 32-feature run of X (16 rows of the chunk), made by
// an identity MFMA (exact): column n of half h is feature
// 32q + 8 (n / 4) + 4h + n % 4.
template <typename F>
__device__ __forceinline__ f32x4 run_to_col(const Pair<F>& x, int h, Lane ln) {
  const f32x4 e = eye4(ln);
  return Pair<F>::template mma<false>(x, h ? Pair<F>::make(zero4(), e) : Pair<F>::make(e, zero4()),
                                      zero4());
}

// G = K^T diag(d) T diag(beta), d = e^{gamma_last - gamma}, as row pairs per
// state block, from the column-form blocks of K (= row pairs of K^T) and NC,
// the column pairs of diag(d) (T - I) diag(beta): the unit diagonal of T
// contributes K^T diag(db), db = d beta, through the accumulator, which no
// operand rounding touches.  (As an operand in 16 bits, beta on the diagonal
// would be off by the same factor in every row where beta is constant, an
// error that adds up over keys that share a direction.)  fp32 adds that term
// last: the partial sums, and so their roundings, stay small.
template <int NB, int DK, typename F, typename TIO>
__device__ __forceinline__ void apply_g(const ColP<NB, F>& NC, const Pair<F> (&kp)[NB][DK / 32],
                                        const float* sdb, TIO* __restrict__ gf, Lane ln) {
  constexpr int NP = npair(NB);
  constexpr bool LAST = sizeof(TIO) == 4;
#pragma unroll
  for (int q = 0; q < DK / 32; ++q) {
    Pair<F> y[2][NP];
    f32x4 acc[2][2 * NP];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int J = 0; J < 2 * NP; ++J)
        acc[h][J] = J < NB ? run_to_col<F>(kp[J < NB ? J : 0][q], h, ln) : zero4();
#pragma unroll
      for (int p = 0; p < NP; ++p) y[h][p] = Pair<F>::make(acc[h][2 * p], acc[h][2 * p + 1]);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int J = 0; J < NB; ++J) {
        const f32x4 kd = acc[h][J] * *(const f32x4*)(sdb + 16 * J + 4 * ln.g());
        acc[h][J] = LAST ? zero4() : kd;
#pragma unroll
        for (int p = J / 2; p < NP; ++p)
          acc[h][J] = Pair<F>::template mma<true>(y[h][p], NC.c[p][J], acc[h][J]);
        if (LAST) acc[h][J] += kd;
      }
#pragma unroll
      for (int p = 0; p < NP; ++p)
        slot_store(gf + ((2 * q + h) * NP + p) * 512,
                   Pair<F>::make(acc[h][2 * p], acc[h][2 * p + 1]), ln.id);
    }
  }
}

// column pairs of the row-form lower blocks D (rounded to the compute type)
template <int NB, typename F>
__device__ __forceinline__ void rows_to_colp(ColP<NB, F>& Y, const Acc<NB>& D, Lane ln) {
  RowP<NB, F> R;
  to_rowp(R, D);
  Acc<NB> t;
  row_to_col(t, R, 0, 16 * NB - 1, ln);
  to_colp(Y, t);
}

// ---------------------------------------------------------------------------
// stage 1

// The inverse modes of the per-chunk launch: T_hat(N, S) in the compute
// type, the exact block-wise inverse, or T_hat(N, S) in integer arithmetic
// (16- or 8-bit codes).
enum FwdInv { kInvNeumann = 0, kInvExact = 1, kInvInt16 = 2, kInvInt8 = 3 };

// The integer inverse of one chunk inside the layer (the quantised GDN of
// Section 3.5): A in fp32 from the K row pairs with the Gram products and
// gates of gdn_build_A, quantised per tile by the quantiser's rule, the
// integer T_hat(N, S) of the shared engine, and its strict lower part
// dequantised (codes * 2^e, exact in fp32) in row form; the caller adds I.
// The codes equal those of gdn_chunk_inverse_neumann_i16_fused (_i8_fused)
// for the same chunk.
template <int NB, int DK, typename F, int INV, int NC, int SC, typename Hook>
__device__ __forceinline__ void chunk_inverse_int(const Pair<F> (&kp)[NB][DK / 32],
                                                  const float* sb, const float* sg, int N, int S,
                                                  Acc<NB>& Tr, Hook&& after_gram) {
  Acc<NB> G;
  gram_lower<NB, DK, true>(G, kp);
  after_gram();
  gate_scale<NB, true>(G, sb, sg, 1.f);
  float m = 0.f;
#pragma unroll
  for (int b = 0; b < nlower(NB); ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) m = fmaxf(m, fabsf(G.a[b][v]));
  const float amax =
      __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(__ockl_wfred_max_f32(m))));
  const int e = INV == kInvInt16 ? i16::quant_exp(amax) : i8::quant_exp(amax);
  int eT;
  if constexpr (INV == kInvInt16) {
    iq::AccI<NB> Lr, Ti;
#pragma unroll
    for (int b = 0; b < nlower(NB); ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) Lr.a[b][v] = -(int)rintf(ldexpf(G.a[b][v], -e));
    iq::int_engine<i16::I16Ops, NB, false, NC, SC>(Lr, e, N, S, Ti, eT);
#pragma unroll
    for (int b = 0; b < nlower(NB); ++b) Tr.a[b] = __builtin_convertvector(Ti.a[b], f32x4);
  } else {
    Acc<NB> Lr;
    i8::quantize_neg(Lr, G, e);
    iq::int_engine<i8::I8Ops, NB, false, NC, SC>(Lr, e, N, S, Tr, eT);
  }
#pragma unroll
  for (int b = 0; b < nlower(NB); ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) Tr.a[b][v] = ldexpf(Tr.a[b][v], eT);
}

// VARLEN: packed sequences (B = 1, L = T tokens, chunk tables pk); a chunk's
// rows past its m tokens are read from row m - 1 and carry beta = 0 and zero
// keys, so their columns of G and P' vanish and the state pass never stores
// their outputs.  split: the state pass is a call of its own; K and V go into
// the workspace for it, the gates do not (it is given them).
template <int NB, int DK, int DV, typename F, bool SMALLN, int NC, int SC, typename TIO,
          int INV, bool VARLEN = false>
__global__ __launch_bounds__(64) void k_fwd_chunk(const TIO* __restrict__ Q,
                                                  const TIO* __restrict__ K,
                                                  const TIO* __restrict__ V,
                                                  const float* __restrict__ beta,
                                                  const float* __restrict__ g,
                                                  TIO* __restrict__ ws, int64_t n_tiles, int L,
                                                  int H, int N, int S, int split, Packed pk) {
  constexpr int C = 16 * NB;
  // bf16: Q arrives in LDS by DMA while registers are busy
  constexpr bool PREF = sizeof(TIO) == 2;
  using LY = FwdLayout<NB, DK, DV>;
  __shared__ __attribute__((aligned(16))) float sb[C], sg[C], sd[C], sdb[C];
  __shared__ __attribute__((aligned(16))) __bf16 sx[PREF ? NB * (DK / 32) * 512 : 8];
  Chunk ch;
  if constexpr (VARLEN)
    ch = Chunk::packed(blockIdx.x, H, C, L, pk.cu, pk.off, pk.nseq, pk.nchunks);
  else
    ch = Chunk(blockIdx.x, L, H, C);
  const int m = VARLEN ? ch.m : C;
  if (VARLEN && m <= 0) return;
  const Lane ln = lane_here();
  const GateRows<C> gr = fetch_gates<C>(beta, g, ch, L, H, m);
  // workspace tile: chunks first, heads inside (the state pass walks the
  // heads side by side)
  const int64_t tile = VARLEN ? (int64_t)blockIdx.x
                              : ((int64_t)ch.b * (L / C) + ch.t0 / C) * H + ch.h;
  TIO* gf = ws + tile * LY::G;
  TIO* pf = ws + n_tiles * LY::G + tile * LY::P;
  TIO* rest = ws + n_tiles * (LY::G + LY::P);
  const int64_t ldk = (int64_t)H * DK, ldv = (int64_t)H * DV;

  Pair<F> kp[NB][DK / 32];
  load_rows<NB, DK>(kp, K + ch.row(0, L, H, DK), ldk, ln, m);
  stash_gates<C>(gr, sb, sg);
  for (int r = ln.id; r < C; r += 64) {
    sd[r] = __expf(sg[C - 1] - sg[r]);
    sdb[r] = sd[r] * sb[r];
    if (!split) ((float*)rest)[tile * C + r] = sg[r];
  }
  __syncthreads();
  auto prefetch_q = [&]() {
    if constexpr (PREF) {
      __builtin_amdgcn_sched_barrier(0);
      prefetch_rows_lds<NB, DK>((const __bf16*)Q + ch.row(0, L, H, DK), ldk, sx, ln, m);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  Acc<NB> Tr;
  if constexpr (INV == kInvInt16 || INV == kInvInt8)
    chunk_inverse_int<NB, DK, F, INV, NC, SC>(kp, sb, sg, N, S, Tr, prefetch_q);
  else
    chunk_inverse<NB, DK, F, SMALLN, NC, SC, INV == kInvExact>(kp, sb, sg, N, S, Tr, prefetch_q);
  // (T - I) diag(beta)
#pragma unroll
  for (int I = 0; I < NB; ++I) Tr.a[bidx(I, I)] = band_block<false>(Tr.a[bidx(I, I)], 0, 1, C);
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J <= I; ++J) Tr.a[bidx(I, J)] *= *(const f32x4*)(sb + 16 * J + 4 * ln.g());

  // P = (Q K^T) (.) D, lower blocks in row form, and P' = P T diag(beta) = P
  // diag(beta) + P (T - I) diag(beta), the first term not rounded (as in apply_g)
  {
    Acc<NB> Pm;
#pragma unroll
    for (int b = 0; b < nlower(NB); ++b) Pm.a[b] = zero4();
    if constexpr (PREF) wait_vmem();
#pragma unroll
    for (int q = 0; q < DK / 32; ++q) {
      Pair<F> qp[NB];
#pragma unroll
      for (int I = 0; I < NB; ++I) {
        if constexpr (PREF)
          qp[I] = LdsRows<DK>{sx, ln.id}(I, q);
        else
          qp[I] = load_row8<F>(Q + ch.row(min(I * 16 + ln.c(), m - 1), L, H, DK) + 32 * q +
                               8 * ln.g());
      }
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = 0; J <= I; ++J)
          Pm.a[bidx(I, J)] = Pair<F>::template mma<true>(qp[I], kp[J][q], Pm.a[bidx(I, J)]);
    }
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J <= I; ++J)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = I * 16 + ln.c(), j = J * 16 + 4 * ln.g() + v;
          // formed either way, then chosen: a branch around each of the diagonal
          // blocks' exponentials would keep the others from overlapping
          const float x = Pm.a[bidx(I, J)][v] * __expf(sg[i] - sg[j]);
          Pm.a[bidx(I, J)][v] = I > J || i >= j ? x : 0.f;
        }
    RowP<NB, F> PR;
    to_rowp(PR, Pm);
    ColP<NB, F> TC;
    rows_to_colp(TC, Tr, ln);
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J <= I; ++J) Pm.a[bidx(I, J)] *= *(const f32x4*)(sb + 16 * J + 4 * ln.g());
    if constexpr (sizeof(TIO) == 2) {
      mm<NB, true, true>(Pm, PR, 0, C - 1, TC, 1, C - 1, 0, C - 1);
    } else {
      Acc<NB> D;
      mm<NB, true, false>(D, PR, 0, C - 1, TC, 1, C - 1, 0, C - 1);
#pragma unroll
      for (int b = 0; b < nlower(NB); ++b) Pm.a[b] += D.a[b];
    }
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int p = 0; 2 * p <= I; ++p)
        slot_store(pf + pidx(I, p) * 512, Pair<F>::make(blk(Pm, I, 2 * p), blk(Pm, I, 2 * p + 1)),
                   ln.id);
  }

  // G (row i of T is row c of its block)
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J <= I; ++J) Tr.a[bidx(I, J)] *= sd[16 * I + ln.c()];
  ColP<NB, F> TC;
  rows_to_colp(TC, Tr, ln);
  apply_g<NB, DK, F>(TC, kp, sdb, gf, ln);

  if (!VARLEN && split) {
    TIO* kc = rest + tile * LY::KC;
    TIO* vc = rest + n_tiles * LY::KC + tile * LY::VC;
#pragma unroll
    for (int I = 0; I < NB; ++I) {
      const int r = I * 16 + ln.c();
#pragma unroll
      for (int q = 0; q < DK / 32; ++q)
        store_row8(kc + r * DK + 32 * q + 8 * ln.g(), kp[I][q].lo(), kp[I][q].hi());
#pragma unroll
      for (int q = 0; q < DV / 32; ++q) {
        const Pair<F> x = load_row8<F>(V + ch.row(r, L, H, DV) + 32 * q + 8 * ln.g());
        store_row8(vc + r * DV + 32 * q + 8 * ln.g(), x.lo(), x.hi());
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The scratch of the allocation-free layer forward (gdn_chunk_forward_noalloc):
// the workspace between the two launches, held in a file-scope device array
// of kForwardScratchBytes that every device the library runs on keeps until
// the process ends.  In host code the array's name is only a stand-in for
// its device address: forward_scratch() looks that address up once per
// device (hipGetSymbolAddress with the device current) and hands it out, and
// only that address is ever passed to a kernel.

static __device__ __align__(256) unsigned char scratch[kForwardScratchBytes];

hipError_t forward_scratch(void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// launchers

template <int NB> struct FwdOrder;
template <> struct FwdOrder<1> { static constexpr int N = 3, S = 2; };
template <> struct FwdOrder<2> { static constexpr int N = 3, S = 4; };
template <> struct FwdOrder<4> { static constexpr int N = 3, S = 8; };

template <int NB, int DK, int DV, typename F, typename TIO>
static hipError_t run_forward_nb(const void* Q, const void* K, const void* V, const float* beta,
                                 const float* g, const float* S0, void* O, float* Sfin, void* ws,
                                 int B, int L, int H, int N, int S, int mode, float scale,
                                 int phases, hipStream_t st, const Packed& pk) {
  constexpr int DN = FwdOrder<NB>::N, DS = FwdOrder<NB>::S;
  const bool packed = pk.cu != nullptr;
  const int64_t n = packed ? (int64_t)pk.nchunks * H : (int64_t)B * H * (L / (16 * NB));
  const int split = phases != 3;  // the two launches are separate calls
#define GDN_FWD1(SM, NC_, SC_, EX)                                                             \
  do {                                                                                         \
    if (packed)                                                                                \
      hipLaunchKernelGGL((k_fwd_chunk<NB, DK, DV, F, SM, NC_, SC_, TIO, EX, true>),            \
                         dim3((unsigned)n), dim3(64), 0, st, (const TIO*)Q, (const TIO*)K,     \
                         (const TIO*)V, beta, g, (TIO*)ws, n, L, H, N, S, split, pk);                 \
    else                                                                                       \
      hipLaunchKernelGGL((k_fwd_chunk<NB, DK, DV, F, SM, NC_, SC_, TIO, EX, false>),           \
                         dim3((unsigned)n), dim3(64), 0, st, (const TIO*)Q, (const TIO*)K,     \
                         (const TIO*)V, beta, g, (TIO*)ws, n, L, H, N, S, split, pk);                 \
  } while (0)
  if ((phases & 1) && n > 0) {
    if (mode == kInvExact) {
      GDN_FWD1(true, 0, 0, kInvExact);
    } else if (mode == kInvInt16 || mode == kInvInt8) {
      // the integer modes run the default order with dk = dv = 128
      if constexpr (DK == 128 && DV == 128) {
        if (N != DN || S != DS) return hipErrorNotSupported;
        if (mode == kInvInt16)
          GDN_FWD1(true, DN, DS, kInvInt16);
        else
          GDN_FWD1(true, DN, DS, kInvInt8);
      } else {
        return hipErrorNotSupported;
      }
    } else if (N == DN && S == DS) {
      GDN_FWD1(true, DN, DS, kInvNeumann);
    } else if (N <= 15) {
      GDN_FWD1(true, -1, -1, kInvNeumann);
    } else {
      GDN_FWD1(false, -1, -1, kInvNeumann);
    }
  }
#undef GDN_FWD1
  if (phases & 2) {
    using LY = FwdLayout<NB, DK, DV>;
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // one call: K and V themselves, the gates as the first launch left them
    const float* gam = split ? g : (const float*)((const TIO*)ws + n * (LY::G + LY::P));
    return run_state<NB, DK, DV, F, TIO>((const TIO*)ws, (const TIO*)Q,
                                         split ? nullptr : (const TIO*)K,
                                         split ? nullptr : (const TIO*)V, gam, !split, S0,
                                         (TIO*)O, Sfin, n, B, L, H, scale, pk, st);
  }
  return hipGetLastError();
}

template <typename F, typename TIO>
static hipError_t run_forward(const void* Q, const void* K, const void* V, const float* beta,
                              const float* g, const float* S0, void* O, float* Sfin, void* ws,
                              int B, int L, int H, int dk, int dv, int C, int N, int S,
                              int mode, float scale, int phases, hipStream_t st,
                              const Packed& pk) {
#define GDN_FWD_NB(NB_)                                                                      \
  GDN_DK_SWITCH(dk, GDN_DV_SWITCH(dv, {                                                      \
    return run_forward_nb<NB_, DK, DV, F, TIO>(Q, K, V, beta, g, S0, O, Sfin, ws, B, L, H, N, \
                                              S, mode, scale, phases, st, pk);               \
  }))
  switch (C) {
    case 16: GDN_FWD_NB(1) break;
    case 32: GDN_FWD_NB(2) break;
    case 64: GDN_FWD_NB(4) break;
  }
#undef GDN_FWD_NB
  return hipErrorNotSupported;
}

static hipError_t forward_dtype(const void* Q, const void* K, const void* V, const float* beta,
                                const float* g, const float* S0, void* O, float* Sfin, void* ws,
                                int B, int L, int H, int dk, int dv, int C, int N, int S,
                                int mode, float scale, int dtype, int phases, hipStream_t st,
                                const Packed& pk) {
  if (dtype == 0)
    return run_forward<f32x4, float>(Q, K, V, beta, g, S0, O, Sfin, ws, B, L, H, dk, dv, C, N, S,
                                     mode, scale, phases, st, pk);
  if (dtype == 1)
    return run_forward<bf16x4, __bf16>(Q, K, V, beta, g, S0, O, Sfin, ws, B, L, H, dk, dv, C, N,
                                       S, mode, scale, phases, st, pk);
  return hipErrorNotSupported;
}

hipError_t launch_forward(const void* Q, const void* K, const void* V, const float* beta,
                          const float* g, const float* S0, void* O, float* Sfin, void* ws, int B,
                          int L, int H, int dk, int dv, int C, int N, int S, int mode,
                          float scale, int dtype, int phases, hipStream_t st) {
  return forward_dtype(Q, K, V, beta, g, S0, O, Sfin, ws, B, L, H, dk, dv, C, N, S, mode, scale,
                       dtype, phases, st, Packed{});
}

hipError_t launch_forward_varlen(const void* Q, const void* K, const void* V, const float* beta,
                                 const float* g, const float* S0, void* O, float* Sfin, void* ws,
                                 const int* cu, const int* off, int nseq, int nchunks, int Ttok,
                                 int H, int dk, int dv, int C, int N, int S, int mode,
                                 float scale, int dtype, hipStream_t st) {
  return forward_dtype(Q, K, V, beta, g, S0, O, Sfin, ws, 1, Ttok, H, dk, dv, C, N, S, mode,
                       scale, dtype, 3, st, Packed{cu, off, nseq, nchunks});
}

}  // namespace gdn
