// forward.hpp -- what the two launches of the chunk-wise layer forward share
// (forward.hip, the per-chunk launch; state.hip, the state pass): the
// workspace layout and its fragment slots.
//
// With gamma the within-chunk cumulative log-decay (the g input), per chunk
//   T = (I + A)^-1, T' = T diag(beta), P = (Q K^T) (.) D,
//   D_ij = e^{gamma_i - gamma_j} for i >= j, else 0,
// the state pass works with the chunk's own K, V and Q and two products of
// the per-chunk launch,
//   G = K^T diag(e^{gamma_last - gamma}) T',   P' = P T'
// (formed with (T - I) diag(beta) as the operand; the unit diagonal's share, K^T
// diag(e^{gamma_last - gamma} beta) and P diag(beta), is added unrounded):
// with S the [dk, dv] state entering the chunk,
//   X  = V - diag(e^gamma) K S,
//   O  = scale (diag(e^gamma) Q S + P' X),
//   S' = e^{gamma_last} S + G X,
// which is the chunk recurrence with V_new = U - W S = T' X (W = T diag(beta
// e^gamma) K, U = T diag(beta) V) folded into G and P'.  Against a workspace
// of W, U, K^T and P this moves 22 KB instead of 55 KB per C = 64 chunk (bf16,
// dk = dv = 128) each way.  In 16 bits the rounded operands are the state (times K
// and Q), (T - I) diag(beta), P, and then G, P' and X; K, Q and V enter as given.
//
// Workspace parts per chunk tile, in elements of the IO type.  A slot is one
// pair per lane (64 x 8 elements).
//   G : (DK / 16) x npair(NB) slots, G row pairs (state block m, p)
//   P : npp(NB) slots, P' row pairs (I, p) with 2p <= I
//   K, V: copies of the chunk's rows [C][DK], [C][DV], written and read only
//     when the two launches are separate calls (the second has no K and V
//     arguments)
#pragma once

#include "wy.hpp"

namespace gdn {

__host__ __device__ constexpr int npp(int NB) {
  int n = 0;
  for (int I = 0; I < NB; ++I) n += I / 2 + 1;
  return n;
}
// sum over i < I of (i / 2 + 1), in closed form (I may be a runtime value)
__host__ __device__ constexpr int pidx(int I, int p) {
  return I + (I / 2) * ((I - 1) / 2) + p;
}
template <int NB, int DK, int DV>
struct FwdLayout {
  static constexpr int64_t G = (DK / 16) * npair(NB) * 512;
  static constexpr int64_t P = npp(NB) * 512;
  static constexpr int64_t KC = 16 * NB * DK;
  static constexpr int64_t VC = 16 * NB * DV;
};

// One fragment slot: a pair per lane, 64 x 8 values.  bf16: lane-major runs
// of 8 (16 bytes per lane); fp32: the lo halves of all lanes, then the hi
// halves (16 bytes per lane each), so that every slot is a whole number of
// 1 KB runs of 16 bytes per lane.
__device__ __forceinline__ void slot_store(__bf16* s, const Pair<bf16x4>& x, int l) {
  *(bf16x8*)(s + 8 * l) = x.v;
}
__device__ __forceinline__ void slot_store(float* s, const Pair<f32x4>& x, int l) {
  *(f32x4*)(s + 4 * l) = x.a;
  *(f32x4*)(s + 256 + 4 * l) = x.b;
}
template <typename F, typename TIO>
__device__ __forceinline__ Pair<F> slot_load(const TIO* s, int l);
template <>
__device__ __forceinline__ Pair<bf16x4> slot_load<bf16x4, __bf16>(const __bf16* s, int l) {
  return Pair<bf16x4>{*(const bf16x8*)(s + 8 * l)};
}
template <>
__device__ __forceinline__ Pair<f32x4> slot_load<f32x4, float>(const float* s, int l) {
  return Pair<f32x4>{*(const f32x4*)(s + 4 * l), *(const f32x4*)(s + 256 + 4 * l)};
}

// The state pass over a prepared workspace (state.hip).  K, V: the inputs
// [B, L, H, d], or nullptr to read the workspace's copies.  gam: the gates,
// as the input [B, L, H] or (gtiles) as rows of C per chunk tile.
template <int NB, int DK, int DV, typename F, typename TIO>
hipError_t run_state(const TIO* ws, const TIO* Q, const TIO* K, const TIO* V, const float* gam,
                     bool gtiles, const float* S0, TIO* O, float* Sfin, int64_t n_tiles, int B,
                     int L, int H, float scale, const Packed& pk, hipStream_t st);

}  // namespace gdn
