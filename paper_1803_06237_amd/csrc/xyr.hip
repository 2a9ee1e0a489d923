// Pass 2 of the matvec for circulant cross-sections of 8 to 64 by 8 to 32 points (and 16 or
// 32 by 64): per kz plane, zero-padded 2-D FFT of the three current components, the 3x3
// symmetric product with the Green spectrum, inverse 2-D FFT and crop (Section III-A: N is
// block Toeplitz, its product a circular convolution).  The solver's operators on the core's
// bounding box and most odd grids have such cross-sections.
//
// Transforms by groups of lanes in registers, see reg_fft.hpp:
//  A: the 3 n2 forward x transforms (inputs x < M1 / 2), one per group of LX lanes;
//  B: one column kx of the three components per group of LY lanes: forward, Green product,
//     inverse;
//  C: the 3 n2 inverse x transforms, crop to x < n1, store.
// The only LDS is the row/column hand-off (3 M2 / 2 rows of M1 frequencies): a row exchanges
// in its own slot, a column in its own entries of components 0 and 1, free once the column is
// in registers.  A workgroup takes as many planes as its threads have columns for, so small
// cross-sections keep whole waves busy and several workgroups share a CU (48 KiB of LDS for
// 256 threads in FP64 at every size).
// The generic LDS pass it replaces has one plane per workgroup and a barrier pair per radix-8
// stage; measurements at xyr_fits.
#include <hip/hip_runtime.h>

#include "block_maps.hpp"
#include "fft_device.hpp"
#include "reg_fft.hpp"
#include "vie_internal.hpp"

namespace vie {

namespace {

// Planes positions first .. first + planes - 1 of the paired order, R: planes hand-offs.
// DEEP: all of a column's spectrum values are loaded before its transforms (one memory
// latency instead of eight; their registers leave one workgroup per SIMD).
template <typename T, int LX, int LY, bool DEEP>
__device__ __forceinline__ void xyr_planes(cx<T>* __restrict__ U, const cx<T>* __restrict__ goct, const Geom& g,
                                           const cx<T>* __restrict__ tw1, const cx<T>* __restrict__ tw2, int first,
                                           int planes, cx<T>* R) {
  constexpr int M1 = 8 * LX, M2 = 8 * LY, Y = 4 * LY, kHand = 3 * Y * M1;
  const int n1 = g.n1, n2 = g.n2;
  const int nthreads = blockDim.x;
  const long plane = 3L * n1 * n2;

  // ---------------- A: forward x transforms, row task = (plane, c, y)
  // (each stage takes a fresh opaque thread index, so that its per-lane LDS address terms
  // are computed where they are used instead of all at the start)
  {
    const int t = opaque_tid();
    const int a = t % LX, q = t / LX;
#pragma unroll 1
    for (int task = q; task < planes * 3 * n2; task += nthreads / LX) {
      const int y = task % n2, c = (task / n2) % 3, pl = task / (3 * n2);
      if (first + pl >= g.M3) break;
      const cx<T>* row = U + paired_plane(first + pl, g.M3) * plane + (long)(c * n2 + y) * n1;
      cx<T> v[8];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int x = a + LX * b;
        const cx<T> in = row[x < n1 ? x : n1 - 1];
        v[b] = cx<T>{x < n1 ? in.x : (T)0, x < n1 ? in.y : (T)0};
      }
      cx<T>* Rp = R + pl * kHand;
      group_fwd<T, LX>(v, tw1, a, Rp + (c * Y + y) * M1, [&](int aa, int k) { return rrow<LX>(aa, k, q & 7); });
#pragma unroll
      for (int e = 0; e < 8 / LX; ++e)
#pragma unroll
        for (int k2 = 0; k2 < LX; ++k2) Rp[rhand<LX, LY>(c, y, (8 / LX) * a + e + 8 * k2)] = v[e * LX + k2];
    }
  }
  __syncthreads();

  // ---------------- B: columns (plane, kx), forward, Green product, inverse
  {
    const int t = opaque_tid();
    const int a = t % LY, col = t / LY, kx = col % M1, pl = col / M1;
    if (pl < planes && first + pl < g.M3) {
      cx<T>* Rp = R + pl * kHand;
      const int kz = paired_plane(first + pl, g.M3);
      // spectrum folded to the stored octant; point i = e LY + m is ky = (8 / LY) a + e + 8 m
      const int k3 = kz <= g.M3 / 2 ? kz : g.M3 - kz;
      const T s3 = kz <= g.M3 / 2 ? (T)1 : (T)-1;
      const int k1 = kx <= M1 / 2 ? kx : M1 - kx;
      const T s1 = kx <= M1 / 2 ? (T)1 : (T)-1;
      const cx<T>* G3 = goct + ((long)k3 * g.H2 * g.H1 + k1) * 6;
      auto green = [&](int i, cx<T>* G) {
        const int ky = (8 / LY) * a + i / LY + 8 * (i % LY);
        const cx<T>* Gp = G3 + (long)(ky <= M2 / 2 ? ky : M2 - ky) * g.H1 * 6;
#pragma unroll
        for (int q = 0; q < 6; ++q) G[q] = Gp[q];
      };
      cx<T> G[DEEP ? 8 : 1][6];
      if constexpr (DEEP)
#pragma unroll
        for (int i = 0; i < 8; ++i) green(i, G[i]);
      cx<T> v[3][8];
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int y = a + LY * b;
          v[c][b] = y < n2 ? Rp[rhand<LX, LY>(c, y, kx)] : cx<T>{(T)0, (T)0};
        }
      auto at = [&](int aa, int k) { return rcol<LX, LY>(0, aa, k, kx); };
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        group_fwd<T, LY>(v[c], tw2, a, Rp, at);
        // components one after the other: interleaving their transforms runs the kernel
        // out of registers
        if constexpr (!DEEP) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int ky = (8 / LY) * a + i / LY + 8 * (i % LY);
        const T s2 = ky <= M2 / 2 ? (T)1 : (T)-1;
        if constexpr (!DEEP) green(i, G[0]);
        const cx<T>* Gi = G[DEEP ? i : 0];
        const cx<T> gxx = Gi[0], gyy = Gi[3], gzz = Gi[5];
        const cx<T> gxy = cscale(Gi[1], s1 * s2), gxz = cscale(Gi[2], s1 * s3), gyz = cscale(Gi[4], s2 * s3);
        const cx<T> ux = v[0][i], uy = v[1][i], uz = v[2][i];
        v[0][i] = cadd(cadd(cmul(gxx, ux), cmul(gxy, uy)), cmul(gxz, uz));
        v[1][i] = cadd(cadd(cmul(gxy, ux), cmul(gyy, uy)), cmul(gyz, uz));
        v[2][i] = cadd(cadd(cmul(gxz, ux), cmul(gyz, uy)), cmul(gzz, uz));
        if constexpr (!DEEP) {
          pin<T>(v[0][i]);
          pin<T>(v[1][i]);
          pin<T>(v[2][i]);
          // one point's spectrum loads in flight at a time (see registers above)
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        group_inv<T, LY>(v[c], tw2, a, Rp, at);
        if constexpr (!DEEP) __builtin_amdgcn_sched_barrier(0);
      }
      // stored after all three inverse transforms: the exchange reuses the entries of
      // components 0 and 1
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int y = a + LY * b;
          if (y < n2) Rp[rhand<LX, LY>(c, y, kx)] = v[c][b];
        }
    }
  }
  __syncthreads();

  // ---------------- C: inverse x transforms, crop, store
  {
    const int t = opaque_tid();
    const int a = t % LX, q = t / LX;
#pragma unroll 1
    for (int task = q; task < planes * 3 * n2; task += nthreads / LX) {
      const int y = task % n2, c = (task / n2) % 3, pl = task / (3 * n2);
      if (first + pl >= g.M3) break;
      cx<T>* Rp = R + pl * kHand;
      cx<T> v[8];
#pragma unroll
      for (int e = 0; e < 8 / LX; ++e)
#pragma unroll
        for (int k2 = 0; k2 < LX; ++k2) v[e * LX + k2] = Rp[rhand<LX, LY>(c, y, (8 / LX) * a + e + 8 * k2)];
      group_inv<T, LX>(v, tw1, a, Rp + (c * Y + y) * M1, [&](int aa, int k) { return rrow<LX>(aa, k, q & 7); });
      cx<T>* row = U + paired_plane(first + pl, g.M3) * plane + (long)(c * n2 + y) * n1;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int x = a + LX * b;
        if (x < n1) row[x] = v[b];
      }
    }
  }
}

// waves per SIMD the registers are held to: three workgroups of 256 threads per CU in FP64
// (their LDS), four in FP32; one fewer for 64-point columns; one in the DEEP form
template <typename T, int LY, bool DEEP>
constexpr int kXyrWaves = DEEP ? 1 : (sizeof(T) == 8 ? 3 : 4) - (LY == 8 ? 1 : 0);

template <typename T, int LX, int LY, bool DEEP>
__global__ __launch_bounds__(256, (kXyrWaves<T, LY, DEEP>)) void k_xyr(cx<T>* __restrict__ U, const cx<T>* __restrict__ goct,
                                                             Geom g, const cx<T>* __restrict__ tw1,
                                                             const cx<T>* __restrict__ tw2) {
  extern __shared__ unsigned char smem_raw[];
  const int planes = blockDim.x / (8 * LX * LY);
  xyr_planes<T, LX, LY, DEEP>(U, goct, g, tw1, tw2, blockIdx.x * planes, planes, reinterpret_cast<cx<T>*>(smem_raw));
}

// items: groups of `planes` planes of each system
template <typename T, int LX, int LY>
__global__ __launch_bounds__(256, (kXyrWaves<T, LY, false>)) void k_xyr_batch(const PassDesc* __restrict__ d,
                                                                   const int* __restrict__ prefix, int nsys,
                                                                   int total) {
  extern __shared__ unsigned char smem_raw[];
  const int planes = blockDim.x / (8 * LX * LY);
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    int lo = 0, hi = nsys - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (prefix[mid] <= item) lo = mid;
      else hi = mid - 1;
    }
    const PassDesc& D = d[lo];
    if (D.active && *D.active == 0) continue;
    xyr_planes<T, LX, LY, false>((cx<T>*)D.U, (const cx<T>*)D.goct, D.g, (const cx<T>*)D.twx, (const cx<T>*)D.twy,
                          (item - prefix[lo]) * planes, planes, reinterpret_cast<cx<T>*>(smem_raw));
    __syncthreads();
  }
}

// threads of a workgroup: 256, fewer where the whole pass would then have under 256 workgroups
// (64 at least, and enough for one plane's columns)
int xyr_threads(int M1, int M2, int M3) {
  const int per = M1 * (M2 / 8);
  int t = 256;
  while (t > 64 && t / 2 >= per && (long)M3 * per / t < 256) t /= 2;
  return t;
}

template <typename T>
size_t xyr_lds(int M1, int M2, int threads) {
  return (size_t)(threads / (M1 * (M2 / 8))) * 3 * (M2 / 2) * M1 * sizeof(cx<T>);
}

#define VIE_XYR_SHAPES(X) \
  X(1, 1) X(2, 1) X(4, 1) X(8, 1) X(1, 2) X(2, 2) X(4, 2) X(8, 2) X(1, 4) X(2, 4) X(4, 4) X(1, 8) X(2, 8) X(4, 8)

}  // namespace

// Measured with events around the pass, against the generic pass (us in FP64 / FP32):
// 64 x 16 x 1024: 24.5 / 18.0, was 59.5 / 50.9; 32 x 32 x 1024: 25.2 / 18.1, was 42.8 / 34.8;
// 32 x 64 x 1024: 38.3 / 23.4, was 81.5 / 44.4; 8 x 8 x 64: 9.1 / 8.2, was 10.0 / 9.5.
bool xyr_fits_batch(const Geom& g) {
  return g.M1 >= 8 && g.M2 >= 8 && g.M1 <= 64 && g.M2 <= 64 && !(g.M1 == 64 && g.M2 == 64);
}
// Single products: 64 x 32 is k_xy6432's, with one plane per workgroup compiled in (38.4
// against 39.4 us at 64 x 32 x 1024).  Up to 16 x 32 x 256 the generic pass has one plane on
// each CU and its 512 threads finish the few transforms sooner than the chain of one lane's
// three columns here (16 x 16 x 64: 11.7 against 13.0 us; from 512 planes on 14.9 against 13.6).
bool xyr_fits(const Geom& g) {
  if (g.M1 <= 16 && (g.M2 == 16 || g.M2 == 32) && g.M3 <= 256) return false;
  return xyr_fits_batch(g) && !(g.M1 == 64 && g.M2 == 32);
}

int xyr_planes_per_group(const Geom& g) { return xyr_threads(g.M1, g.M2, 1 << 20) / (g.M1 * (g.M2 / 8)); }

template <typename T>
hipError_t launch_xyr(const Geom& g, void* U, const void* goct, const void* tw1, const void* tw2, hipStream_t s) {
  if (!xyr_fits(g)) return hipErrorInvalidValue;
  const int threads = xyr_threads(g.M1, g.M2, g.M3);
  const int planes = threads / (g.M1 * (g.M2 / 8));
  const dim3 grid((g.M3 + planes - 1) / planes);
  // at most one workgroup per CU: nothing hides the spectrum's latency but the loads themselves
  const bool deep = grid.x <= 256;
  const size_t lds = xyr_lds<T>(g.M1, g.M2, threads);
#define VIE_XYR(LX, LY)                                                                                   \
  if (g.M1 == 8 * LX && g.M2 == 8 * LY) {                                                                 \
    if (deep)                                                                                             \
      hipLaunchKernelGGL((k_xyr<T, LX, LY, true>), grid, dim3(threads), lds, s, (cx<T>*)U,                \
                         (const cx<T>*)goct, g, (const cx<T>*)tw1, (const cx<T>*)tw2);                    \
    else                                                                                                  \
      hipLaunchKernelGGL((k_xyr<T, LX, LY, false>), grid, dim3(threads), lds, s, (cx<T>*)U,               \
                         (const cx<T>*)goct, g, (const cx<T>*)tw1, (const cx<T>*)tw2);                    \
    return hipGetLastError();                                                                             \
  }
  VIE_XYR_SHAPES(VIE_XYR)
#undef VIE_XYR
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_xyr_batch(int M1, int M2, const PassDesc* d, const int* prefix, int nsys, int total, hipStream_t s) {
  const int threads = xyr_threads(M1, M2, 1 << 20);
  const size_t lds = xyr_lds<T>(M1, M2, threads);
  const dim3 grid(total < 4096 ? total : 4096);
#define VIE_XYR(LX, LY)                                                                                      \
  if (M1 == 8 * LX && M2 == 8 * LY) {                                                                        \
    hipLaunchKernelGGL((k_xyr_batch<T, LX, LY>), grid, dim3(threads), lds, s, d, prefix, nsys, total);       \
    return hipGetLastError();                                                                                \
  }
  VIE_XYR_SHAPES(VIE_XYR)
  VIE_XYR(8, 4)
#undef VIE_XYR
  return hipErrorInvalidValue;
}

template hipError_t launch_xyr<double>(const Geom&, void*, const void*, const void*, const void*, hipStream_t);
template hipError_t launch_xyr<float>(const Geom&, void*, const void*, const void*, const void*, hipStream_t);
template hipError_t launch_xyr_batch<double>(int, int, const PassDesc*, const int*, int, int, hipStream_t);
template hipError_t launch_xyr_batch<float>(int, int, const PassDesc*, const int*, int, int, hipStream_t);

}  // namespace vie
