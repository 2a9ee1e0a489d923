// Krylov building blocks launched on a stream (implementations in krylov.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "fft_device.hpp"

namespace vie {

// ||w||^2 / ||h||^2 of an FP64 Arnoldi step below which it needs the extra sweep (krylov.hip)
constexpr double kCancel2 = 0.01;

// Sums of NV (a power of two up to 64) values per lane over the wave: lane l gets that of value *idx, with half
// as many exchanges per halving step as values left (17 in all for 16 values instead of 96).
template <int NV, int H>
__device__ __forceinline__ void wave_fold(double (&v)[NV], int lane, int& id) {
  if constexpr (H >= 1) {
    constexpr int bit = NV / 2 / H;              // 1, 2, 4, ...
    const bool up = (lane & bit) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const double send = up ? v[i] : v[i + H], keep = up ? v[i + H] : v[i];
      v[i] = keep + __shfl_xor(send, bit, 64);
    }
    id |= up ? H : 0;
    wave_fold<NV, H / 2>(v, lane, id);
  }
}
template <int NV>
__device__ __forceinline__ double wave_sum_many(double (&v)[NV], int lane, int* idx) {
  *idx = 0;
  wave_fold<NV, NV / 2>(v, lane, *idx);
  double r = v[0];
#pragma unroll
  for (int o = NV; o < 64; o <<= 1) r += __shfl_xor(r, o, 64);
  return r;
}

// Rows i0 .. i0 + 63 of h = 2 raw - G raw by a workgroup of kProjThreads, G hermitian with
// G_ij, i < j, at H[i ldh + j] and its diagonal in gd.  The products with k > i run along the
// lanes of the wave that has row i and those with k <= i along lanes of rows, split over the
// waves, so that both read H in whole lines (with lanes of rows throughout the first kind read a
// line per lane: batched FP64 steps of one system, cycles of 500, 206 us, now 190 with the
// extra sweep's launches).
constexpr int kProjThreads = 1024;
struct ProjLds {
  double2 lower[kProjThreads / 64][64];
  double upper[64][2];
};
__device__ __forceinline__ void project_rows(const double2* __restrict__ raw, const double2* __restrict__ gd,
                                             const double2* __restrict__ H, int ldh, int nv, int i0,
                                             double2* __restrict__ h, ProjLds& lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int kW = kProjThreads / 64, kRows = 64 / kW;
  double a[2 * kRows];
#pragma unroll
  for (int q = 0; q < 2 * kRows; ++q) a[q] = 0.0;
  const int r0 = i0 + wave * kRows;
  for (int k = r0 + 1 + lane; k < nv; k += 64) {
    const double2 r = raw[k];
#pragma unroll
    for (int q = 0; q < kRows; ++q)
      if (k > r0 + q) {
        const double2 g = H[(long)(r0 + q) * ldh + k];
        a[2 * q] += g.x * r.x - g.y * r.y;
        a[2 * q + 1] += g.x * r.y + g.y * r.x;
      }
  }
  int idx;
  const double t = wave_sum_many<2 * kRows>(a, lane, &idx);
  if (lane < 2 * kRows) lds.upper[wave * kRows + (idx >> 1)][idx & 1] = t;
  const int i = i0 + lane;
  double2 s{0.0, 0.0};
  if (i < nv)
    for (int k = wave; k <= i; k += kW) {
      const double2 r = raw[k];
      double2 g = k == i ? gd[i] : H[(long)k * ldh + i];   // conj G_ki
      g.y = k == i ? g.y : -g.y;
      s.x += g.x * r.x - g.y * r.y;
      s.y += g.x * r.y + g.y * r.x;
    }
  lds.lower[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && i < nv) {
    double2 u{lds.upper[lane][0], lds.upper[lane][1]};
    for (int k = 0; k < kW; ++k) {
      u.x += lds.lower[k][lane].x;
      u.y += lds.lower[k][lane].y;
    }
    const double2 r = raw[i];
    h[i] = double2{2.0 * r.x - u.x, 2.0 * r.y - u.y};
  }
  __syncthreads();
}

// Device data of one GMRES cycle: the reduction partials (arnoldi_partials), the raw dots and
// the Gram diagonal (m + 1 values each), the projections h, the Hessenberg matrix
// (column-major, leading dimension ldh; the Gram entries G_ij, i < j, at row j of column i),
// the rotations, the right-hand side g and its entries before their last rotation, the gate of
// the extra sweep.
struct ArnoldiData {
  double2 *partial, *raw, *gd, *h, *H;
  int ldh;
  double* cs;
  double2 *sn, *g, *pend;
  int* gate;
};

template <typename T>
struct KrylovOps {
  // out[0].x = ||w||^2 (FP64 accumulation); partial needs partial_blocks(n) entries
  static hipError_t nrm2sq(const cx<T>* w, long n, double2* partial, double2* out, hipStream_t s);
  // w += sign * sum_i coef[i] V_i
  template <typename TW>
  static hipError_t maxpy(const cx<T>* V, long ldv, int nv, const double2* coef, double sign, cx<TW>* w, long n,
                          hipStream_t s);
  // Arnoldi step j after w = A v_j: w orthogonalised against V_0 .. V_j and normalised (it is
  // V_{j+1}), Hessenberg column, rotation and g updated; state (pinned host memory, 4 values):
  // residual estimate, ||w||, 1 if something is not finite, 1 if the step cancelled too much
  // for the merged sweeps.  again: a further sweep where the device finds that; a step that
  // reports it without is to be repeated from w = A v_j with it.
  static hipError_t orthogonalise(const cx<T>* V, int j, cx<T>* w, long n, const ArnoldiData& d, double bnorm,
                                  bool again, double* state, hipStream_t s);
  // dst = src / sqrt(sumsq->x)
  static hipError_t scale(const cx<T>* src, cx<T>* dst, long n, const double2* sumsq, hipStream_t s);
  static hipError_t zero(cx<T>* dst, long n, hipStream_t s);
  static hipError_t trisolve(const double2* H, int ldh, const double2* g, int k, double2* y, hipStream_t s);
  static hipError_t set_g(double2* pend, const double2* sumsq, hipStream_t s);
};

template <typename TS, typename TD>
hipError_t convert(const cx<TS>* src, cx<TD>* dst, long n, hipStream_t s);

// The voxel columns (i1, i2) where the contrast is non-zero on some slice.  A
// maps vectors supported on these columns (all slices, all three components) to
// vectors supported there, so Krylov vectors can be stored compressed:
// comp[(a s + p) n3 + i3] = full[a][col[p]][i3] with col[p] = i1 n2 + i2.
struct Support {
  const int* col;   // device, s entries, increasing
  int s;
  long n12;         // n1 n2
  int n3;
  long size() const { return 3L * s * n3; }
};
// comp = full on the support (sub != nullptr: comp = sub - full on the support; may alias comp)
template <typename T>
hipError_t gather(const Support& u, const cx<T>* full, cx<T>* comp, const cx<T>* sub, hipStream_t s);
// full on the support = comp (other entries untouched)
template <typename T>
hipError_t scatter(const Support& u, const cx<T>* comp, cx<T>* full, hipStream_t s);
// full on the support = 0
template <typename T>
hipError_t zero_support(const Support& u, cx<T>* full, hipStream_t s);
// flags[c] = 1 if chi[c][i3] != 0 for some i3, else 0 (c < n12)
hipError_t column_flags(const double2* chi, long n12, int n3, int* flags, hipStream_t s);

int partial_blocks(long n);
// partials of a cycle of dimension m on vectors of n elements
size_t arnoldi_partials(long n, int m);

}  // namespace vie
