// Register-resident DFTs of 8, 10, 12, 15 and 16 points, natural order in and out:
// X[k] = sum_n v[n] exp(-+2 pi i n k / N).
//
// 10 = 2 x 5, 12 = 3 x 4 and 15 = 3 x 5 by the prime-factor maps n = (N2 n1 + N1 n2) mod N and
// k = the residue that is k1 mod N1 and k2 mod N2, which leave no twiddles; 16 = 4 x 4 with
// twiddles; 3 and 5 points by the symmetric and antisymmetric sums of the conjugate pairs.
// dft_half: v[n] = 0 for n >= N / 2 (zero padding), the butterflies of those inputs left out.
#pragma once
#include "fft_device.hpp"

namespace vie {

// (a, b, c) -> 3-point DFT
template <typename T, bool INV>
__device__ __forceinline__ void dft3(cx<T>& a, cx<T>& b, cx<T>& c) {
  const T h = (T)0.5, s = (T)0.86602540378443864676;   // sin(2 pi / 3)
  const cx<T> p = cadd(b, c), m = cscale(rot90<INV>(csub(b, c)), s);
  const cx<T> q{a.x - h * p.x, a.y - h * p.y};
  a = cadd(a, p);
  b = cadd(q, m);
  c = csub(q, m);
}

// v[0..5) -> 5-point DFT
template <typename T, bool INV>
__device__ __forceinline__ void dft5(cx<T>* v) {
  const T c1 = (T)0.30901699437494742410, c2 = (T)-0.80901699437494742410;   // cos(2 pi / 5), cos(4 pi / 5)
  const T s1 = (T)0.95105651629515357212, s2 = (T)0.58778525229247312917;    // sin(2 pi / 5), sin(4 pi / 5)
  const cx<T> p1 = cadd(v[1], v[4]), p2 = cadd(v[2], v[3]);
  const cx<T> m1 = rot90<INV>(csub(v[1], v[4])), m2 = rot90<INV>(csub(v[2], v[3]));
  const cx<T> a{v[0].x + c1 * p1.x + c2 * p2.x, v[0].y + c1 * p1.y + c2 * p2.y};
  const cx<T> b{v[0].x + c2 * p1.x + c1 * p2.x, v[0].y + c2 * p1.y + c1 * p2.y};
  const cx<T> d{s1 * m1.x + s2 * m2.x, s1 * m1.y + s2 * m2.y};
  const cx<T> e{s2 * m1.x - s1 * m2.x, s2 * m1.y - s1 * m2.y};
  v[0] = cadd(v[0], cadd(p1, p2));
  v[1] = cadd(a, d);
  v[4] = csub(a, d);
  v[2] = cadd(b, e);
  v[3] = csub(b, e);
}

// 4-point DFT of (a, b, 0, 0)
template <typename T, bool INV>
__device__ __forceinline__ void dft4_half(cx<T>* v) {
  const cx<T> a = v[0], b = v[1], r = rot90<INV>(b);
  v[0] = cadd(a, b);
  v[1] = cadd(a, r);
  v[2] = csub(a, b);
  v[3] = csub(a, r);
}

// W_16^k = exp(-+2 pi i k / 16) for the products of two indices below 4
template <typename T, bool INV>
__device__ __forceinline__ cx<T> twiddle16(cx<T> z, int k) {
  const T r = (T)0.70710678118654752440, c = (T)0.92387953251128675613, s = (T)0.38268343236508977173;
  const cx<T> w = k == 1 ? cx<T>{c, -s} : k == 2 ? cx<T>{r, -r} : k == 3 ? cx<T>{s, -c} : k == 6 ? cx<T>{-r, -r} : cx<T>{-c, s};
  if (k == 0) return z;
  if (k == 4) return rot90<INV>(z);
  return INV ? cmulc(z, w) : cmul(z, w);
}

template <typename T, bool INV, bool HALF>
__device__ __forceinline__ void dft16(cx<T>* v) {
  cx<T> y[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int b = 0; b < (HALF ? 2 : 4); ++b) y[a][b] = v[a + 4 * b];
    if constexpr (HALF) dft4_half<T, INV>(y[a]);
    else dft4<T, INV>(y[a]);
#pragma unroll
    for (int k = 1; k < 4; ++k) y[a][k] = twiddle16<T, INV>(y[a][k], a * k);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    cx<T> z[4] = {y[0][k], y[1][k], y[2][k], y[3][k]};
    dft4<T, INV>(z);
#pragma unroll
    for (int m = 0; m < 4; ++m) v[k + 4 * m] = z[m];
  }
}

template <typename T, bool INV, bool HALF>
__device__ __forceinline__ void dft10(cx<T>* v) {
  // n = (5 n1 + 2 n2) mod 10, k = (5 k1 + 6 k2) mod 10
  cx<T> y[2][5];
#pragma unroll
  for (int n2 = 0; n2 < 5; ++n2) {
    const int na = 2 * n2, nb = (5 + 2 * n2) % 10;
    if (HALF) {   // exactly one of the pair is below 5
      const bool lo = na < 5;
      y[0][n2] = lo ? v[na] : v[nb];
      y[1][n2] = lo ? v[na] : cx<T>{-v[nb].x, -v[nb].y};
    } else {
      y[0][n2] = cadd(v[na], v[nb]);
      y[1][n2] = csub(v[na], v[nb]);
    }
  }
  dft5<T, INV>(y[0]);
  dft5<T, INV>(y[1]);
#pragma unroll
  for (int k = 0; k < 10; ++k) v[k] = y[k % 2][k % 5];
}

template <typename T, bool INV, bool HALF>
__device__ __forceinline__ void dft12(cx<T>* v) {
  // n = (4 n1 + 3 n2) mod 12, k = the residue that is k1 mod 3 and k2 mod 4
  cx<T> y[3][4];
#pragma unroll
  for (int n1 = 0; n1 < 3; ++n1) {
    if constexpr (HALF) {
      // the two inputs below 6: n2 = 0, 1 (0, 3), n2 = 3, 0 (1, 4), n2 = 2, 3 (2, 5)
      const cx<T> a = n1 == 0 ? v[0] : n1 == 1 ? v[1] : v[2];
      const cx<T> b = n1 == 0 ? v[3] : n1 == 1 ? v[4] : v[5];
      cx<T> z[4] = {a, b, a, b};
      dft4_half<T, INV>(z);   // as if at n2 = 0, 1; a shift of n2 by d multiplies output k2 by (-+i)^(d k2)
      constexpr int shift[3] = {0, 3, 2};
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) {
        const int q = shift[n1] * k2 % 4;
        y[n1][k2] = q == 0 ? z[k2] : q == 1 ? rot90<INV>(z[k2]) : q == 2 ? cx<T>{-z[k2].x, -z[k2].y} : rot90<!INV>(z[k2]);
      }
    } else {
#pragma unroll
      for (int n2 = 0; n2 < 4; ++n2) y[n1][n2] = v[(4 * n1 + 3 * n2) % 12];
      dft4<T, INV>(y[n1]);
    }
  }
#pragma unroll
  for (int k2 = 0; k2 < 4; ++k2) dft3<T, INV>(y[0][k2], y[1][k2], y[2][k2]);
#pragma unroll
  for (int k = 0; k < 12; ++k) v[k] = y[k % 3][k % 4];
}

template <typename T, bool INV>
__device__ __forceinline__ void dft15(cx<T>* v) {
  // n = (5 n1 + 3 n2) mod 15, k = the residue that is k1 mod 3 and k2 mod 5
  cx<T> y[3][5];
#pragma unroll
  for (int n1 = 0; n1 < 3; ++n1) {
#pragma unroll
    for (int n2 = 0; n2 < 5; ++n2) y[n1][n2] = v[(5 * n1 + 3 * n2) % 15];
    dft5<T, INV>(y[n1]);
  }
#pragma unroll
  for (int k2 = 0; k2 < 5; ++k2) dft3<T, INV>(y[0][k2], y[1][k2], y[2][k2]);
#pragma unroll
  for (int k = 0; k < 15; ++k) v[k] = y[k % 3][k % 5];
}

template <typename T, bool INV, int N>
__device__ __forceinline__ void dft_codelet(cx<T>* v) {
  if constexpr (N == 8) dft8<T, INV>(v);
  else if constexpr (N == 10) dft10<T, INV, false>(v);
  else if constexpr (N == 12) dft12<T, INV, false>(v);
  else if constexpr (N == 15) dft15<T, INV>(v);
  else {
    static_assert(N == 16);
    dft16<T, INV, false>(v);
  }
}

// forward, N even, v[n] taken as zero for n >= N / 2
template <typename T, int N>
__device__ __forceinline__ void dft_half(cx<T>* v) {
  if constexpr (N == 8) dft8_padded<T>(v);
  else if constexpr (N == 10) dft10<T, false, true>(v);
  else if constexpr (N == 12) dft12<T, false, true>(v);
  else {
    static_assert(N == 16);
    dft16<T, false, true>(v);
  }
}

}  // namespace vie
