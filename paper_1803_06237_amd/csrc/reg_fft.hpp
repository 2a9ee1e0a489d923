// Transforms of length 8 L by groups of L lanes holding 8 values each in registers (the
// cross-section passes of xyr.hip and jmr.hip).  Lane a holds x[a + L b], takes an 8-point DFT
// over b, twiddles by W^(a k), exchanges (a, k) with the group through LDS and finishes with
// 8 / L transforms of L points, giving X[k1 + 8 k2] for k1 = (8 / L) a + e at position e L + k2.
// The inverse runs mirrored.  A group's lanes lie in one wave, whose LDS accesses complete in
// program order, so wave barriers order the exchange.
#pragma once
#include "fft_device.hpp"

namespace vie {

// hand-off element (c, y, kx) of one plane: row (c, y), column swizzled so that the LY rows
// a column group reads at once lie in different banks
template <int LX, int LY>
__device__ __forceinline__ int rhand(int c, int y, int kx) {
  constexpr int M1 = 8 * LX, Y = 4 * LY;
  const int sw = LY == 8 ? (y & 7) << 1 : (y & 3) * 10;
  return (c * Y + y) * M1 + (kx ^ (sw & (M1 - 1)));
}
// row exchange element (a, k) of group f inside the row's 8 L slots
template <int L>
__device__ __forceinline__ int rrow(int a, int k, int f) {
  if (L == 8) return (k ^ (f & 3)) * 8 + ((k + a) & 7);
  if (L == 4) return ((k + f) & 7) * 4 + (a ^ ((k >> 1) & 3));
  return ((k + f) & 7) * 2 + (a ^ ((k >> 2) & 1));
}
// column exchange element (a, k) of column kx: entries of components c0, c0 + 1, chosen so
// that the lanes of a group differ in y & (LY - 1) when writing and when reading
template <int LX, int LY>
__device__ __forceinline__ int rcol(int c0, int a, int k, int kx) {
  return rhand<LX, LY>(c0 + (k & 1), (k >> 1) * LY + ((a + k * LY / 8) & (LY - 1)), kx);
}

// 8 / L transforms of L points on v[0..L), v[L..2 L), ...
template <typename T, bool INV, int L>
__device__ __forceinline__ void dft_tail(cx<T>* v) {
#pragma unroll
  for (int e = 0; e < 8 / L; ++e) {
    if constexpr (L == 2) dft2<T, INV>(v + 2 * e);
    else if constexpr (L == 4) dft4<T, INV>(v + 4 * e);
    else if constexpr (L == 8) dft8<T, INV>(v);
  }
}

// Forward transform of a group: in, lane a holds x[a + L b] (PADDED: for b < 4, the rest is
// zero padding); out, v[e L + k2] = X[(8 / L) a + e + 8 k2].  at(a, k): the exchange slot in S;
// tw[TS k] = W^k.
template <typename T, int L, bool PADDED = true, int TS = 1, typename AT>
__device__ __forceinline__ void group_fwd(cx<T>* v, const cx<T>* tw, int a, cx<T>* S, AT at) {
  if constexpr (PADDED) dft8_padded<T>(v);
  else dft8<T, false>(v);
  if constexpr (L > 1) {
#pragma unroll
    for (int k = 1; k < 8; ++k) v[k] = cmul(v[k], tw[TS * a * k]);
#pragma unroll
    for (int k = 0; k < 8; ++k) S[at(a, k)] = v[k];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int e = 0; e < 8 / L; ++e)
#pragma unroll
      for (int s = 0; s < L; ++s) v[e * L + s] = S[at(s, (8 / L) * a + e)];
    __builtin_amdgcn_wave_barrier();
    dft_tail<T, false, L>(v);
  }
}

// The inverse, mirrored: v[b] = x[a + L b] (of a padded transform only b < 4 is wanted).
template <typename T, int L, int TS = 1, typename AT>
__device__ __forceinline__ void group_inv(cx<T>* v, const cx<T>* tw, int a, cx<T>* S, AT at) {
  if constexpr (L > 1) {
    dft_tail<T, true, L>(v);
#pragma unroll
    for (int e = 0; e < 8 / L; ++e)
#pragma unroll
      for (int s = 0; s < L; ++s) {
        const int k1 = (8 / L) * a + e;
        S[at(s, k1)] = s == 0 ? v[e * L] : cmulc(v[e * L + s], tw[TS * s * k1]);
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = S[at(a, k)];
    __builtin_amdgcn_wave_barrier();
  }
  dft8<T, true>(v);
}

// The value as the compiler must materialise it here (it would otherwise carry parts of the
// Green product into the inverse transforms and need half as many registers again).
template <typename T>
__device__ __forceinline__ void pin(cx<T>& v) {
  asm volatile("" : "+v"(v.x), "+v"(v.y));
}

}  // namespace vie
