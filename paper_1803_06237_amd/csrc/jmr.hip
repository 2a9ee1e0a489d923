// Cross-section pass of the JM product (jm.hip) with every transform in registers: per kz plane
// the zero-padded 2-D FFT of the six components, the coupled product
//   out_e = N u_e + i kappa K u_m,   out_m = N u_m - i kappa K u_e
// at every frequency, the inverse 2-D FFT and the crop; U_e and U_m are read and overwritten in
// place.  The scheme is that of xyr.hip with the two halves on neighbouring lanes: a column
// group has LY pairs of lanes, lane 2 a + h holding the three components of half h, so a thread
// keeps three columns as in the J-VIE pass; it forms N u and K u of its own half and swaps K u
// with its neighbour by a lane permutation.
// Hand-off: 6 M2 / 2 rows of M1 / SPLIT frequencies.  SPLIT = 2 is for 64 x 64, whose full rows
// do not fit in LDS in FP64 (196 KiB): with x_n = 0 for n >= M1 / 2 the even frequencies are the
// M1/2-point transform of the rows and the odd ones that of the rows twisted by W^n, W =
// exp(-2 pi i / M1), and the inverse with the crop adds the two half-length inverses, the second
// untwisted; the workgroup does both in turn, U holding the first half's outputs meanwhile.
// Against the fused pass over LDS transforms (k_jm_xy, kept for sections with a side under 8
// points): see jmr_fits.
#include <hip/hip_runtime.h>

#include "block_maps.hpp"
#include "fft_device.hpp"
#include "reg_fft.hpp"
#include "vie_internal.hpp"

namespace vie {

namespace {

// the value of the neighbouring lane (lane ^ 1)
__device__ __forceinline__ float swap_pair(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));   // quad_perm [1, 0, 3, 2]
}
__device__ __forceinline__ double swap_pair(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)b, 0xB1, 0xF, 0xF, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), 0xB1, 0xF, 0xF, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <typename V>
__device__ __forceinline__ V swap_pair2(V v) {
  return V{swap_pair(v.x), swap_pair(v.y)};
}

template <typename T, int LX, int LY, int SPLIT>
__device__ __forceinline__ void jmr_planes(cx<T>* __restrict__ Ue, cx<T>* __restrict__ Um,
                                           const cx<T>* __restrict__ goct, const cx<T>* __restrict__ koct,
                                           const Geom& g, T kappa, const cx<T>* __restrict__ tw1,
                                           const cx<T>* __restrict__ tw2, int first, int planes, cx<T>* R) {
  constexpr int Mx = 8 * LX, M1 = Mx * SPLIT, M2 = 8 * LY, Y = 4 * LY, kHand = 6 * Y * Mx;
  constexpr int kIn = 4 * SPLIT;                // inputs per lane of a row: x < M1 / 2
  const int n1 = g.n1, n2 = g.n2;
  const int nthreads = blockDim.x;
  const long plane = 3L * n1 * n2;
  if (planes > g.M3 - first) planes = g.M3 - first;
  // row task (plane, component, y) on the LX lanes q
  const int tasks = planes * 6 * n2;
  struct Row {
    cx<T>* u;
    cx<T>* Rp;
    int c, y;
  };
  auto row_of = [&](int task) {
    const int y = task % n2, c = (task / n2) % 6, pl = task / (6 * n2);
    const int kz = paired_plane(first + pl, g.M3);
    return Row{(c < 3 ? Ue : Um) + kz * plane + (long)((c < 3 ? c : c - 3) * n2 + y) * n1, R + pl * kHand, c, y};
  };
  // forward transform of a row (odd: of the odd frequencies) into the hand-off
  auto forward = [&](const Row& r, cx<T>* v, bool odd, int a, int q) {
    if (SPLIT == 2 && odd)
#pragma unroll
      for (int b = 0; b < 8; ++b) v[b] = cmul(v[b], tw1[a + LX * b]);
    group_fwd<T, LX, SPLIT == 1, SPLIT>(v, tw1, a, r.Rp + (r.c * Y + r.y) * Mx,
                                        [&](int aa, int k) { return rrow<LX>(aa, k, q & 7); });
#pragma unroll
    for (int e = 0; e < 8 / LX; ++e)
#pragma unroll
      for (int k2 = 0; k2 < LX; ++k2) r.Rp[rhand<LX, LY>(r.c, r.y, (8 / LX) * a + e + 8 * k2)] = v[e * LX + k2];
  };
  auto load_row = [&](const Row& r, cx<T>* v, int a) {
#pragma unroll
    for (int b = 0; b < kIn; ++b) {
      const int x = a + LX * b;
      const cx<T> in = r.u[x < n1 ? x : n1 - 1];
      v[b] = cx<T>{x < n1 ? in.x : (T)0, x < n1 ? in.y : (T)0};
    }
  };

  // ---------------- A: forward x transforms
  {
    const int t = opaque_tid();
    const int a = t % LX, q = t / LX;
#pragma unroll 1
    for (int task = q; task < tasks; task += nthreads / LX) {
      const Row r = row_of(task);
      cx<T> v[8];
      load_row(r, v, a);
      forward(r, v, false, a, q);
    }
  }
  __syncthreads();

#pragma unroll 1
  for (int half = 0; half < SPLIT; ++half) {
    // ---------------- B: columns (plane, kx, half h), forward, product, inverse
    {
      const int t = opaque_tid();
      const int h = t & 1, a = (t >> 1) % LY, col = (t >> 1) / LY, kc = col % Mx, pl = col / Mx;
      if (pl < planes) {
        cx<T>* Rp = R + pl * kHand;
        const int kz = paired_plane(first + pl, g.M3);
        const int kx = SPLIT * kc + half;
        const int k3 = kz <= g.M3 / 2 ? kz : g.M3 - kz;
        const T s3 = kz <= g.M3 / 2 ? (T)1 : (T)-1;
        const int k1 = kx <= M1 / 2 ? kx : M1 - kx;
        const T s1 = kx <= M1 / 2 ? (T)1 : (T)-1;
        const T kap = h == 0 ? kappa : -kappa;
        const long o3 = (long)k3 * g.H2 * g.H1 + k1;
        cx<T> v[3][8];
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const int y = a + LY * b;
            v[c][b] = y < n2 ? Rp[rhand<LX, LY>(3 * h + c, y, kc)] : cx<T>{(T)0, (T)0};
          }
        auto at = [&](int aa, int k) { return rcol<LX, LY>(3 * h, aa, k, kc); };
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          group_fwd<T, LY>(v[c], tw2, a, Rp, at);
          __builtin_amdgcn_sched_barrier(0);   // components in turn: registers
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int ky = (8 / LY) * a + i / LY + 8 * (i % LY);
          const T s2 = ky <= M2 / 2 ? (T)1 : (T)-1;
          const long f = o3 + (long)(ky <= M2 / 2 ? ky : M2 - ky) * g.H1;
          const cx<T>* G = goct + f * 6;
          const cx<T>* K = koct + f * 3;
          const cx<T> gxx = G[0], gyy = G[3], gzz = G[5];
          const cx<T> gxy = cscale(G[1], s1 * s2), gxz = cscale(G[2], s1 * s3), gyz = cscale(G[4], s2 * s3);
          // i kappa K (of this half's sign for the neighbour: out_m takes -i kappa K u_e)
          const cx<T> kxy = cscale(K[0], kap * s3), kxz = cscale(K[1], kap * s2), kyz = cscale(K[2], kap * s1);
          const cx<T> ux = v[0][i], uy = v[1][i], uz = v[2][i];
          // K antisymmetric; times i, and minus for the neighbour of half 0
          cx<T> kx_ = cadd(cmul(kxy, uy), cmul(kxz, uz)), ky_ = csub(cmul(kyz, uz), cmul(kxy, ux));
          cx<T> kz_ = cadd(cmul(kxz, ux), cmul(kyz, uy));
          kx_ = swap_pair2(cx<T>{kx_.y, -kx_.x});
          ky_ = swap_pair2(cx<T>{ky_.y, -ky_.x});
          kz_ = swap_pair2(cx<T>{-kz_.y, kz_.x});
          v[0][i] = cadd(cadd(cadd(cmul(gxx, ux), cmul(gxy, uy)), cmul(gxz, uz)), kx_);
          v[1][i] = cadd(cadd(cadd(cmul(gxy, ux), cmul(gyy, uy)), cmul(gyz, uz)), ky_);
          v[2][i] = cadd(cadd(cadd(cmul(gxz, ux), cmul(gyz, uy)), cmul(gzz, uz)), kz_);
          pin<T>(v[0][i]);
          pin<T>(v[1][i]);
          pin<T>(v[2][i]);
          __builtin_amdgcn_sched_barrier(0);   // one point's spectra in flight: registers
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          group_inv<T, LY>(v[c], tw2, a, Rp, at);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const int y = a + LY * b;
            if (y < n2) Rp[rhand<LX, LY>(3 * h + c, y, kc)] = v[c][b];
          }
      }
    }
    __syncthreads();

    // ---------------- C: inverse x transforms; crop and store, the first half also sends the
    // row's odd frequencies (its lanes store the elements that they have read)
    {
      const int t = opaque_tid();
      const int a = t % LX, q = t / LX;
#pragma unroll 1
      for (int task = q; task < tasks; task += nthreads / LX) {
        const Row r = row_of(task);
        cx<T> v[8], w[8];
        if (SPLIT == 2) load_row(r, w, a);
#pragma unroll
        for (int e = 0; e < 8 / LX; ++e)
#pragma unroll
          for (int k2 = 0; k2 < LX; ++k2)
            v[e * LX + k2] = r.Rp[rhand<LX, LY>(r.c, r.y, (8 / LX) * a + e + 8 * k2)];
        group_inv<T, LX, SPLIT>(v, tw1, a, r.Rp + (r.c * Y + r.y) * Mx,
                                [&](int aa, int k) { return rrow<LX>(aa, k, q & 7); });
        const bool last = half == SPLIT - 1;
#pragma unroll
        for (int b = 0; b < kIn; ++b) {
          const int x = a + LX * b;
          if (SPLIT == 2 && last) v[b] = cadd(w[b], cmulc(v[b], tw1[x]));
          if (x < n1) r.u[x] = v[b];
        }
        if (SPLIT == 2 && !last) forward(r, w, true, a, q);
      }
    }
    if (SPLIT == 2) __syncthreads();
  }
}

// waves per SIMD: two in FP64 (192 bytes of LDS and over 200 registers a thread), four in FP32
template <typename T>
constexpr int kJmrWaves = sizeof(T) == 8 ? 2 : 4;

template <typename T, int LX, int LY, int SPLIT, int THREADS>
__global__ __launch_bounds__(THREADS, kJmrWaves<T>) void k_jmr(
    cx<T>* __restrict__ Ue, cx<T>* __restrict__ Um, const cx<T>* __restrict__ goct, const cx<T>* __restrict__ koct,
    Geom g, T kappa, const cx<T>* __restrict__ tw1, const cx<T>* __restrict__ tw2) {
  extern __shared__ unsigned char smem_raw[];
  const int planes = blockDim.x / (16 * LX * LY);
  jmr_planes<T, LX, LY, SPLIT>(Ue, Um, goct, koct, g, kappa, tw1, tw2, blockIdx.x * planes, planes,
                               reinterpret_cast<cx<T>*>(smem_raw));
}

// threads of a workgroup: one plane's column lanes if those are more than 256, else 256, fewer
// where the pass would then have under 256 workgroups (64 at least, and one plane's columns)
int jmr_threads(int Mx, int M2, int M3) {
  const int per = Mx * (M2 / 8) * 2;
  int t = per > 256 ? per : 256;
  while (t > 64 && t / 2 >= per && (long)M3 * per / t < 256) t /= 2;
  return t;
}

#define VIE_JMR_SHAPES(X)                                                                              \
  X(1, 1, 1, 256) X(2, 1, 1, 256) X(4, 1, 1, 256) X(8, 1, 1, 256) X(1, 2, 1, 256) X(2, 2, 1, 256)      \
  X(4, 2, 1, 256) X(8, 2, 1, 256) X(1, 4, 1, 256) X(2, 4, 1, 256) X(4, 4, 1, 256) X(8, 4, 1, 512)      \
  X(1, 8, 1, 256) X(2, 8, 1, 256) X(4, 8, 1, 512)                                                      \
  X((sizeof(T) == 8 ? 4 : 8), 8, (sizeof(T) == 8 ? 2 : 1), (sizeof(T) == 8 ? 512 : 1024))

template <typename T>
int jmr_split(const Geom& g) {
  return sizeof(T) == 8 && g.M1 == 64 && g.M2 == 64 ? 2 : 1;
}

template <typename T>
size_t jmr_lds(const Geom& g, int threads) {
  const int Mx = g.M1 / jmr_split<T>(g);
  return (size_t)(threads / (Mx * (g.M2 / 8) * 2)) * 6 * (g.M2 / 2) * Mx * sizeof(cx<T>);
}

}  // namespace

// Whole product with the LDS pass and with this one, us: every pair of sides gains at 8 to 1024
// planes.  FP64 16 x 16 x 1024 75 and 60, 32 x 32 x 1024 144 and 91, 64 x 32 x 1024 266 and 138,
// 64 x 64 x 1024 577 and 291; FP32 32 x 32 x 1024 93 and 67, 64 x 32 x 1024 173 and 88,
// 64 x 64 x 1024 277 and 136 (in two halves as in FP64: 253); with 8 planes, bound by the
// launches, 5 to 20 %.
bool jmr_fits(const Geom& g) { return g.M1 >= 8 && g.M2 >= 8 && g.M1 <= 64 && g.M2 <= 64; }

template <typename T>
hipError_t launch_jmr(const Geom& g, void* Ue, void* Um, const void* goct, const void* koct, double kappa,
                      const void* tw1, const void* tw2, hipStream_t s) {
  using C = cx<T>;
  if (!jmr_fits(g)) return hipErrorInvalidValue;
  const int split = jmr_split<T>(g), Mx = g.M1 / split;
  const int threads = jmr_threads(Mx, g.M2, g.M3);
  const int planes = threads / (Mx * (g.M2 / 8) * 2);
  const dim3 grid((g.M3 + planes - 1) / planes);
  const size_t lds = jmr_lds<T>(g, threads);
#define VIE_JMR(LX, LY, SP, TH)                                                                               \
  if (Mx == 8 * LX && g.M2 == 8 * LY && split == SP) {                                                        \
    hipLaunchKernelGGL((k_jmr<T, LX, LY, SP, TH>), grid, dim3(threads), lds, s, (C*)Ue, (C*)Um, (const C*)goct, \
                       (const C*)koct, g, (T)kappa, (const C*)tw1, (const C*)tw2);                            \
    return hipGetLastError();                                                                                 \
  }
  VIE_JMR_SHAPES(VIE_JMR)
#undef VIE_JMR
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t allow_lds_jmr() {
  hipError_t e = hipSuccess;
#define VIE_JMR(LX, LY, SP, TH)                                                                                     \
  if (!e)                                                                                                           \
    e = hipFuncSetAttribute((const void*)k_jmr<T, LX, LY, SP, TH>, hipFuncAttributeMaxDynamicSharedMemorySize,      \
                            TH / (16 * LX * LY) * 6 * 4 * LY * 8 * LX * (int)sizeof(cx<T>));
  VIE_JMR_SHAPES(VIE_JMR)
#undef VIE_JMR
  return e;
}

template hipError_t launch_jmr<double>(const Geom&, void*, void*, const void*, const void*, double, const void*,
                                       const void*, hipStream_t);
template hipError_t launch_jmr<float>(const Geom&, void*, void*, const void*, const void*, double, const void*,
                                      const void*, hipStream_t);
template hipError_t allow_lds_jmr<double>();
template hipError_t allow_lds_jmr<float>();

}  // namespace vie
