// GMRES(m) and flexible GMRES(m) on the device (Section V-D: the discrete J-VIE
// is solved by GMRES with matrix-vector products only).
//
// Arnoldi is classical Gram-Schmidt applied twice, with the two sweeps merged.  With
// h1 = V^H w and G = V^H V the second sweep's coefficients are V^H (w - V h1) = h1 - G h1, so
// w'' = w - V h with h = 2 h1 - G h1 needs one pass over the basis for the dots and one for
// the update instead of two each; G's new column V^H v_j comes out of the same dot pass (v_j
// is its last vector).  Four kernels a step: k_mdot2 (dots with w and with v_j), k_proj (their
// sums, h; two launches in long cycles), k_maxpy_nrm (w'' and block sums of |w''|^2), k_finish (norm, v_{j+1}, Hessenberg
// column, rotation, estimate to host memory).  Measured per step with the sweeps apart (dots
// and update of the second gated by a cancellation test): ten kernels and a copy, 110 us at
// n = 276480 and j ~ 20, 33 us at n = 1536 and j ~ 25; merged 60 and 18 us.
//
// The merged second sweep corrects for G != I but takes V^H w' from the rounded dots of w
// instead of measuring it, so V^H v_{j+1} is of order eps ||h|| / ||w''|| (two measured sweeps:
// eps).  On guides ||w''|| is 0.3 to 0.5 of ||h||.  Where it is below a tenth of it (kCancel2) in
// FP64, one more sweep measures V^H w'' and subtracts it, which bounds the loss by 10 eps at
// any cancellation (without it a permittivity of 1e-10 in one voxel, ratios of 1e-10, made a
// cycle of 15 steps end at 27 times the minimal residual, the basis no longer one).  k_finish reports such a step; the
// solver repeats it with the extra sweep and queues that, gated on the device by the same
// test (k_gate), for the steps that follow.  FP32 vectors do not need it: their dots are FP64
// sums of exact products, so what the merging leaves out is below their own rounding until
// w'' is nothing but the rounding of w.
// The Hessenberg matrix is kept in upper-triangular form with complex Givens rotations by one
// device thread; the host reads only the residual estimate |g_{j+1}| / ||b|| after each step.
// G_ij, i < j, lies in the unused strict lower triangle of that matrix.  Reductions are
// two-stage and in a fixed order, so results are bitwise reproducible run to run.  All
// reductions and Hessenberg data are FP64; basis vectors are FP64 (cx<double>)
// or FP32 (cx<float>, the inner solve of the mixed tier).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>

#include "fft_device.hpp"
#include "krylov.hpp"

namespace vie {

constexpr int kThreads = 256;
constexpr int kEPT = 2;                     // elements per thread held in registers (reductions)
constexpr int kChunk = kThreads * kEPT;     // elements per block (reductions)
constexpr int kGroup = 4;                   // basis vectors per block of the multi-dot
constexpr int kDotEPT = 4;                  // elements per thread and round of the multi-dot
constexpr int kDotChunk = kThreads * kDotEPT;
constexpr int kDotBlocks = 256;             // most blocks (partials) per vector group of the multi-dot
constexpr int kAxpyBlocks = 2048;           // most blocks (partials) of k_maxpy_nrm

__device__ __forceinline__ double2 to_d(double2 v) { return v; }
__device__ __forceinline__ double2 to_d(float2 v) { return double2{(double)v.x, (double)v.y}; }
template <typename V> __device__ __forceinline__ V from_d(double2 v);
template <> __device__ __forceinline__ double2 from_d<double2>(double2 v) { return v; }
template <> __device__ __forceinline__ float2 from_d<float2>(double2 v) { return float2{(float)v.x, (float)v.y}; }

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  return v;
}

// Block-wide sum of NV double values per thread; result valid in thread 0.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = wave_sum(v[i]);
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < NV; ++i) lds[wave * NV + i] = v[i];
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 0; i < NV; ++i) {
      double s = 0;
      for (int w = 0; w < kThreads / 64; ++w) s += lds[w * NV + i];
      v[i] = s;
    }
  }
  __syncthreads();
}

// partial[(2 i + s) nblk + blk] = the block's share of V_i^H w (s = 0) and of V_i^H V_{nv-1}
// (s = 1), for the kGroup vectors i of blockIdx.y; GATED: nothing where *gate == 0
template <typename T, bool GATED>
__global__ __launch_bounds__(kThreads) void k_mdot2(const cx<T>* __restrict__ V, long ldv, int nv,
                                                     const cx<T>* __restrict__ w, long n,
                                                     double2* __restrict__ partial, const int* __restrict__ gate) {
  if (GATED && *gate == 0) return;
  constexpr int kVals = 4 * kGroup;
  __shared__ double lds[kThreads / 64][kVals];
  const cx<T>* vj = V + (long)(nv - 1) * ldv;
  const int i0 = blockIdx.y * kGroup;
  double acc[kVals];
#pragma unroll
  for (int q = 0; q < kVals; ++q) acc[q] = 0.0;
  for (long b0 = (long)blockIdx.x * kDotChunk; b0 < n; b0 += (long)gridDim.x * kDotChunk) {
    // loads from clamped, always valid addresses (w and v_j count as zero past the end), so
    // that all of a round are in flight together instead of one per branch
    long e[kDotEPT];
    double2 wv[kDotEPT], vv[kDotEPT];
#pragma unroll
    for (int k = 0; k < kDotEPT; ++k) {
      const long at = b0 + threadIdx.x + (long)k * kThreads;
      e[k] = at < n ? at : n - 1;
      wv[k] = to_d(w[e[k]]);
      vv[k] = to_d(vj[e[k]]);
      if (at >= n) wv[k] = vv[k] = double2{0.0, 0.0};
    }
#pragma unroll
    for (int q = 0; q < kGroup; ++q) {
      const cx<T>* Vi = V + (long)(i0 + q < nv ? i0 + q : nv - 1) * ldv;
      double2 a[kDotEPT];
#pragma unroll
      for (int k = 0; k < kDotEPT; ++k) a[k] = to_d(Vi[e[k]]);
#pragma unroll
      for (int k = 0; k < kDotEPT; ++k) {
        acc[4 * q] += a[k].x * wv[k].x + a[k].y * wv[k].y;
        acc[4 * q + 1] += a[k].x * wv[k].y - a[k].y * wv[k].x;
        acc[4 * q + 2] += a[k].x * vv[k].x + a[k].y * vv[k].y;
        acc[4 * q + 3] += a[k].x * vv[k].y - a[k].y * vv[k].x;
      }
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int idx;
  const double r = wave_sum_many<kVals>(acc, lane, &idx);
  if (lane < kVals) lds[wave][idx] = r;
  __syncthreads();
  // value 4 q + 2 s + c: component c of partial (2 (i0 + q) + s)
  if (threadIdx.x < kVals && i0 + (int)(threadIdx.x >> 2) < nv) {
    double t = 0.0;
    for (int k = 0; k < kThreads / 64; ++k) t += lds[k][threadIdx.x];
    const long row = 2L * i0 + (threadIdx.x >> 1);
    reinterpret_cast<double*>(partial)[2 * (row * gridDim.x + blockIdx.x) + (threadIdx.x & 1)] = t;
  }
}

// The sums of k_mdot2's partials (raw = V^H w into `raw`, the new Gram column into gd[j] and
// H's lower triangle), j = nv - 1
__device__ __forceinline__ void dot_sums(const double2* __restrict__ partial, int nblk, int nv,
                                         double2* __restrict__ raw, double2* __restrict__ gd,
                                         double2* __restrict__ H, int ldh) {
  // 8 lanes per value: one round of loads for up to 64 vectors, kDotBlocks / 8 per lane
  const int sub = threadIdx.x & 7;
  for (int v = (blockIdx.x * kProjThreads + threadIdx.x) >> 3; v < 2 * nv; v += gridDim.x * (kProjThreads / 8)) {
    double2 s{0.0, 0.0};
#pragma unroll 8
    for (int b = sub; b < nblk; b += 8) {
      const double2 p = partial[(long)v * nblk + b];
      s.x += p.x;
      s.y += p.y;
    }
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
      s.x += __shfl_xor(s.x, o, 64);
      s.y += __shfl_xor(s.y, o, 64);
    }
    if (sub == 0) {
      const int i = v >> 1;
      if ((v & 1) == 0) raw[i] = s;
      else if (i < nv - 1) H[(long)i * ldh + nv - 1] = s;
      else gd[i] = s;
    }
  }
}

// Sums and h = 2 raw - G raw by one workgroup.  Its share grows with nv^2: past kProjOne vectors
// the sums and the rows are two launches over as many workgroups as they fill (an average step
// at n = 12288, us: cycles of 150 steps 57.5 with 64, 59.8 with 192, of 200 65.6 and 69.4; of
// 1000 152, by one workgroup throughout 380).
constexpr int kProjOne = 64;
__global__ __launch_bounds__(kProjThreads) void k_proj(const double2* __restrict__ partial, int nblk, int nv,
                                                       double2* __restrict__ raw, double2* __restrict__ gd,
                                                       double2* __restrict__ H, int ldh, double2* __restrict__ h) {
  __shared__ ProjLds lds;
  dot_sums(partial, nblk, nv, raw, gd, H, ldh);
  __syncthreads();
  for (int i0 = 0; i0 < nv; i0 += 64) project_rows(raw, gd, H, ldh, nv, i0, h, lds);
}
__global__ __launch_bounds__(kProjThreads) void k_dot_sums(const double2* __restrict__ partial, int nblk, int nv,
                                                           double2* __restrict__ raw, double2* __restrict__ gd,
                                                           double2* __restrict__ H, int ldh) {
  dot_sums(partial, nblk, nv, raw, gd, H, ldh);
}
__global__ __launch_bounds__(kProjThreads) void k_proj_rows(const double2* __restrict__ raw,
                                                            const double2* __restrict__ gd,
                                                            const double2* __restrict__ H, int ldh, int nv,
                                                            double2* __restrict__ h) {
  __shared__ ProjLds lds;
  project_rows(raw, gd, H, ldh, nv, blockIdx.x * 64, h, lds);
}

// *gate = 1 where ||w''||^2, the sum of nblk partials, is too small a part of ||h||^2
__global__ __launch_bounds__(kThreads) void k_gate(const double* __restrict__ partial, int nblk,
                                                   const double2* __restrict__ h, int nv, int* __restrict__ gate) {
  __shared__ double lds[(kThreads / 64) * 2];
  double v[2] = {0.0, 0.0};
  for (int b = threadIdx.x; b < nblk; b += kThreads) v[0] += partial[b];
  for (int i = threadIdx.x; i < nv; i += kThreads) v[1] += h[i].x * h[i].x + h[i].y * h[i].y;
  block_sum<2>(v, lds);
  if (threadIdx.x == 0) *gate = v[0] < kCancel2 * v[1] ? 1 : 0;
}

// The extra sweep's coefficients from k_mdot2's partials: c = V^H w'', and h += c
__global__ __launch_bounds__(kThreads) void k_proj_again(const double2* __restrict__ partial, int nblk, int nv,
                                                         double2* __restrict__ c, double2* __restrict__ h,
                                                         const int* __restrict__ gate) {
  if (*gate == 0) return;
  const int sub = threadIdx.x & 7, i = blockIdx.x * (kThreads / 8) + (threadIdx.x >> 3);
  double2 s{0.0, 0.0};
  if (i < nv)
    for (int b = sub; b < nblk; b += 8) {
      const double2 p = partial[2L * i * nblk + b];
      s.x += p.x;
      s.y += p.y;
    }
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) {
    s.x += __shfl_xor(s.x, o, 64);
    s.y += __shfl_xor(s.y, o, 64);
  }
  if (sub == 0 && i < nv) {
    c[i] = s;
    h[i] = double2{h[i].x + s.x, h[i].y + s.y};
  }
}

// out[i] = sum_b partial[i * nblk + b], one workgroup per i, fixed order
__global__ __launch_bounds__(kThreads) void k_reduce(const double2* __restrict__ partial, int nblk,
                                                      double2* __restrict__ out) {
  __shared__ double lds[(kThreads / 64) * 2];
  const int i = blockIdx.x;
  double v[2] = {0.0, 0.0};
  for (int b = threadIdx.x; b < nblk; b += kThreads) {
    const double2 p = partial[(long)i * nblk + b];
    v[0] += p.x;
    v[1] += p.y;
  }
  block_sum<2>(v, lds);
  if (threadIdx.x == 0) out[i] = double2{v[0], v[1]};
}

// w += sign * sum_i coef[i] V_i, one element per thread (loads of the nv vectors
// are independent, so they overlap)
template <typename T, typename TW>
__global__ __launch_bounds__(kThreads) void k_maxpy(const cx<T>* __restrict__ V, long ldv, int nv,
                                                     const double2* __restrict__ coef, double sign,
                                                     cx<TW>* __restrict__ w, long n) {
  __shared__ double2 c[512];
  for (int i = threadIdx.x; i < nv && i < 512; i += kThreads) c[i] = double2{sign * coef[i].x, sign * coef[i].y};
  __syncthreads();
  const long e = (long)blockIdx.x * kThreads + threadIdx.x;
  if (e >= n) return;
  double2 acc = to_d(w[e]);
  const cx<T>* Ve = V + e;
#pragma unroll 4
  for (int i = 0; i < nv; ++i) {
    const double2 ci = c[i];
    const double2 a = to_d(Ve[(long)i * ldv]);
    acc.x += ci.x * a.x - ci.y * a.y;
    acc.y += ci.x * a.y + ci.y * a.x;
  }
  w[e] = from_d<cx<TW>>(acc);
}

// partial[blk] = sum |w|^2 over the block's chunk
template <typename T>
__global__ __launch_bounds__(kThreads) void k_nrm2_partial(const cx<T>* __restrict__ w, long n,
                                                            double2* __restrict__ partial) {
  __shared__ double lds[(kThreads / 64) * 2];
  const long e0 = (long)blockIdx.x * kChunk + threadIdx.x;
  double v[2] = {0.0, 0.0};
#pragma unroll
  for (int k = 0; k < kEPT; ++k) {
    const long e = e0 + (long)k * kThreads;
    if (e < n) {
      const double2 a = to_d(w[e]);
      v[0] += a.x * a.x + a.y * a.y;
    }
  }
  block_sum<2>(v, lds);
  if (threadIdx.x == 0) partial[blockIdx.x] = double2{v[0], 0.0};
}

// dst = src * (1/norm) where norm = sqrt(sumsq->x); dst may alias src
template <typename T>
__global__ __launch_bounds__(kThreads) void k_scale(const cx<T>* src, cx<T>* dst, long n,
                                                     const double2* __restrict__ sumsq) {
  const double nr = sqrt(sumsq->x);
  const double s = nr > 0.0 ? 1.0 / nr : 0.0;
  for (long e = (long)blockIdx.x * kThreads + threadIdx.x; e < n; e += (long)gridDim.x * kThreads) {
    const double2 a = to_d(src[e]);
    dst[e] = from_d<cx<T>>(double2{a.x * s, a.y * s});
  }
}

template <typename TS, typename TD>
__global__ __launch_bounds__(kThreads) void k_copy(const cx<TS>* __restrict__ src, cx<TD>* __restrict__ dst,
                                                    long n) {
  for (long e = (long)blockIdx.x * kThreads + threadIdx.x; e < n; e += (long)gridDim.x * kThreads)
    dst[e] = from_d<cx<TD>>(to_d(src[e]));
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_zero(cx<T>* __restrict__ dst, long n) {
  for (long e = (long)blockIdx.x * kThreads + threadIdx.x; e < n; e += (long)gridDim.x * kThreads)
    dst[e] = cx<T>{(T)0, (T)0};
}

// w -= sum_i h_i V_i and, of the stored result, the block partial sums of |w|^2; GATED: nothing
// where *gate == 0
template <typename T, bool GATED>
__global__ __launch_bounds__(kThreads) void k_maxpy_nrm(const cx<T>* __restrict__ V, long ldv, int nv,
                                                         const double2* __restrict__ h, cx<T>* __restrict__ w, long n,
                                                         double* __restrict__ partial, const int* __restrict__ gate) {
  if (GATED && *gate == 0) return;
  extern __shared__ unsigned char smem_raw[];
  double2* c = reinterpret_cast<double2*>(smem_raw);   // nv values, zeros up to a multiple of 8
  __shared__ double lds[kThreads / 64];
  for (int i = threadIdx.x; i < nv + 7; i += kThreads) c[i] = i < nv ? h[i] : double2{0.0, 0.0};
  __syncthreads();
  double v[1] = {0.0};
  for (long e = (long)blockIdx.x * kThreads + threadIdx.x; e < n; e += (long)gridDim.x * kThreads) {
    double2 acc = to_d(w[e]);
    const cx<T>* Ve = V + e;
    for (int i = 0; i < nv; i += 8) {   // eight loads in flight (the last vector again past the end)
      double2 a[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) a[k] = to_d(Ve[(long)(i + k < nv ? i + k : nv - 1) * ldv]);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const double2 ci = c[i + k];
        acc.x -= ci.x * a[k].x - ci.y * a[k].y;
        acc.y -= ci.x * a[k].y + ci.y * a[k].x;
      }
    }
    const cx<T> out = from_d<cx<T>>(acc);
    w[e] = out;
    const double2 o = to_d(out);
    v[0] += o.x * o.x + o.y * o.y;
  }
  block_sum<1>(v, lds);
  if (threadIdx.x == 0) partial[blockIdx.x] = v[0];
}

// Column j of the Hessenberg matrix (hs[0..j] = the projections, hn = ||w||) through the previous
// rotations, the new rotation and g, by one thread: it sweeps the rotations down the column with
// the running entry in a register (the loads of hs, cs, sn do not depend on the sweep, so they
// are issued ahead).  pend[j] is the rotated right-hand side's entry before rotation j, so that
// a step can be repeated.  state: see k_finish.
__device__ __forceinline__ void hessenberg_column(double2* hs, double hn, double* __restrict__ cs,
                                                  double2* __restrict__ sn, double2* __restrict__ gvec,
                                                  double2* __restrict__ pend, int j, double bnorm,
                                                  double* __restrict__ state) {
  // previous rotations: [c s; -conj(s) c] on (h_i, h_{i+1})
  double2 a = hs[0];
  for (int i = 0; i < j; ++i) {
    const double2 b = hs[i + 1];
    const double c = cs[i];
    const double2 s = sn[i];
    hs[i] = double2{c * a.x + (s.x * b.x - s.y * b.y), c * a.y + (s.x * b.y + s.y * b.x)};
    a = double2{-(s.x * a.x + s.y * a.y) + c * b.x, -(s.x * a.y - s.y * a.x) + c * b.y};
  }
  // new rotation zeroing h_{j+1} = ||w||
  const double2 b = double2{hn, 0.0};
  const double na = hypot(a.x, a.y), nb = hypot(b.x, b.y);
  double c;
  double2 sv, r;
  if (nb == 0.0) {
    c = 1.0;
    sv = double2{0.0, 0.0};
    r = a;
  } else if (na == 0.0) {
    c = 0.0;
    sv = double2{1.0, 0.0};
    r = b;
  } else {
    const double t = hypot(na, nb);
    const double2 ph = double2{a.x / na, a.y / na};
    c = na / t;
    // s = ph * conj(b) / t
    sv = double2{(ph.x * b.x + ph.y * b.y) / t, (ph.y * b.x - ph.x * b.y) / t};
    r = double2{ph.x * t, ph.y * t};
  }
  cs[j] = c;
  sn[j] = sv;
  hs[j] = r;
  const double2 gj = pend[j];
  // g_{j+1} = -conj(s) g_j ; g_j = c g_j
  const double2 gn = double2{-(sv.x * gj.x + sv.y * gj.y), -(sv.x * gj.y - sv.y * gj.x)};
  pend[j + 1] = gn;
  gvec[j] = double2{c * gj.x, c * gj.y};
  const double est = hypot(gn.x, gn.y) / bnorm;
  state[0] = est;
  state[1] = hn;
  state[2] = (isfinite(est) && isfinite(hn) && isfinite(r.x) && isfinite(r.y)) ? 0.0 : 1.0;
  __threadfence_system();
}

// End of an Arnoldi step.  Every workgroup sums the nblk partials of ||w||^2 (same order, same
// result) and scales its share of w; workgroup 0 also does the Hessenberg bookkeeping: column
// j = (h, ||w||) through the previous rotations, the new rotation, g.  state (host memory):
// [0] residual estimate |g_{j+1}| / bnorm, [1] ||w|| (breakdown when 0), [2] = 1 if any value
// is non-finite, [3] = 1 if the step cancelled too much for the merged sweeps alone.  After the
// extra sweep, *gate != 0, the partials are those of its update.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_finish(cx<T>* __restrict__ w, long n,
                                                      const double* __restrict__ partial, int nblk,
                                                      const int* __restrict__ gate, const double2* __restrict__ h,
                                                      double2* __restrict__ H, int ldh, double* __restrict__ cs,
                                                      double2* __restrict__ sn, double2* __restrict__ gvec,
                                                      double2* __restrict__ pend, int j, double bnorm,
                                                      double* __restrict__ state) {
  extern __shared__ unsigned char smem_raw[];
  double2* hs = reinterpret_cast<double2*>(smem_raw);   // j + 2 entries (workgroup 0)
  __shared__ double lds[kThreads / 64];
  __shared__ double s_norm;
  const bool again = gate && *gate != 0;
  if (again) partial += nblk;
  double v[1] = {0.0};
  for (int b = threadIdx.x; b < nblk; b += kThreads) v[0] += partial[b];
  block_sum<1>(v, lds);
  if (threadIdx.x == 0) s_norm = sqrt(v[0]);
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i <= j; i += kThreads) hs[i] = h[i];
  __syncthreads();
  const double hn = s_norm;
  const double scale = hn > 0.0 ? 1.0 / hn : 0.0;
  for (long e = (long)blockIdx.x * kThreads + threadIdx.x; e < n; e += (long)gridDim.x * kThreads) {
    const double2 a = to_d(w[e]);
    w[e] = from_d<cx<T>>(double2{a.x * scale, a.y * scale});
  }
  if (blockIdx.x != 0) return;
  if (threadIdx.x == 0) hessenberg_column(hs, hn, cs, sn, gvec, pend, j, bnorm, state);
  if (threadIdx.x >= 64 && threadIdx.x < 128) {   // meanwhile the second wave: the cancellation
    double hh = 0.0;
    for (int i = threadIdx.x - 64; i <= j; i += 64) hh += h[i].x * h[i].x + h[i].y * h[i].y;
    hh = wave_sum(hh);
    if (threadIdx.x == 64) state[3] = again || hn * hn < kCancel2 * hh ? 1.0 : 0.0;
  }
  __syncthreads();
  double2* col = H + (long)j * ldh;
  for (int i = threadIdx.x; i <= j; i += kThreads) col[i] = hs[i];
}

// y = R^{-1} g for the leading k x k upper triangle of H, column by column from the last: one
// workgroup, the right-hand side in LDS, every thread updating its rows with the new y_i.  A
// triangle of up to kTriLds columns, within the default limit of 64 KiB, is staged in LDS first
// (by one thread from global memory the solve took 133 us at k = 50, a load latency per entry).
constexpr int kTriLds = 63;
__global__ __launch_bounds__(kThreads) void k_trisolve(const double2* __restrict__ H, int ldh,
                                                        const double2* __restrict__ gvec, int k,
                                                        double2* __restrict__ y) {
  extern __shared__ unsigned char smem_raw[];
  double2* r = reinterpret_cast<double2*>(smem_raw);   // k values
  double2* R = r + k;                                   // k x k, where k <= kTriLds
  const bool staged = k <= kTriLds;
  for (int i = threadIdx.x; i < k; i += kThreads) r[i] = gvec[i];
  if (staged)
    for (int e = threadIdx.x; e < k * k; e += kThreads) R[e] = H[(long)(e / k) * ldh + e % k];
  __syncthreads();
  const double2* A = staged ? R : H;
  const long ld = staged ? k : ldh;
  for (int i = k - 1; i >= 0; --i) {
    const double2 s = r[i], d = A[(long)i * ld + i];
    const double dd = d.x * d.x + d.y * d.y;
    const double2 yi = double2{(s.x * d.x + s.y * d.y) / dd, (s.y * d.x - s.x * d.y) / dd};
    if (threadIdx.x == 0) y[i] = yi;
    for (int l = threadIdx.x; l < i; l += kThreads) {
      const double2 a = A[(long)i * ld + l];
      r[l] = double2{r[l].x - (a.x * yi.x - a.y * yi.y), r[l].y - (a.x * yi.y + a.y * yi.x)};
    }
    __syncthreads();
  }
}

__global__ void k_set_g(double2* pend, const double2* sumsq) { pend[0] = double2{sqrt(sumsq->x), 0.0}; }

// ---- support compression ------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kThreads) void k_gather(const cx<T>* __restrict__ full, cx<T>* comp, const cx<T>* sub,
                                                      const int* __restrict__ col, int s, long n12, int n3) {
  const long total = 3L * s * n3;
  for (long e = (long)blockIdx.x * kThreads + threadIdx.x; e < total; e += (long)gridDim.x * kThreads) {
    const long row = e / n3;
    const int t = (int)(e - row * n3);
    const int a = (int)(row / s), p = (int)(row - (long)a * s);
    const cx<T> v = full[((long)a * n12 + col[p]) * n3 + t];
    comp[e] = sub ? cx<T>{sub[e].x - v.x, sub[e].y - v.y} : v;
  }
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_scatter(const cx<T>* __restrict__ comp, cx<T>* __restrict__ full,
                                                       const int* __restrict__ col, int s, long n12, int n3,
                                                       int zero) {
  const long total = 3L * s * n3;
  for (long e = (long)blockIdx.x * kThreads + threadIdx.x; e < total; e += (long)gridDim.x * kThreads) {
    const long row = e / n3;
    const int t = (int)(e - row * n3);
    const int a = (int)(row / s), p = (int)(row - (long)a * s);
    full[((long)a * n12 + col[p]) * n3 + t] = zero ? cx<T>{(T)0, (T)0} : comp[e];
  }
}

__global__ __launch_bounds__(kThreads) void k_column_flags(const double2* __restrict__ chi, long n12, int n3,
                                                            int* __restrict__ flags) {
  const long c = (long)blockIdx.x * kThreads + threadIdx.x;
  if (c >= n12) return;
  const double2* z = chi + c * n3;
  int any = 0;
  for (int t = 0; t < n3; ++t) any |= (z[t].x != 0.0 || z[t].y != 0.0) ? 1 : 0;
  flags[c] = any;
}

// ------------------------------------------------------------------ host-side helpers

static inline int nblocks(long n) { return (int)((n + kChunk - 1) / kChunk); }

template <typename T>
hipError_t KrylovOps<T>::nrm2sq(const cx<T>* w, long n, double2* partial, double2* out, hipStream_t s) {
  const int nb = nblocks(n);
  hipLaunchKernelGGL((k_nrm2_partial<T>), dim3(nb), dim3(kThreads), 0, s, w, n, partial);
  hipLaunchKernelGGL(k_reduce, dim3(1), dim3(kThreads), 0, s, partial, nb, out);
  return hipGetLastError();
}

template <typename T>
template <typename TW>
hipError_t KrylovOps<T>::maxpy(const cx<T>* V, long ldv, int nv, const double2* coef, double sign, cx<TW>* w,
                               long n, hipStream_t s) {
  for (int i0 = 0; i0 < nv; i0 += 512) {
    const int cnt = nv - i0 < 512 ? nv - i0 : 512;
    hipLaunchKernelGGL((k_maxpy<T, TW>), dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, s,
                       V + (long)i0 * ldv, ldv, cnt,
                       coef + i0, sign, w, n);
  }
  return hipGetLastError();
}

// every block the same number of rounds
static int axpy_blocks(long n) {
  const long b = (n + kThreads - 1) / kThreads, rounds = (b + kAxpyBlocks - 1) / kAxpyBlocks;
  return (int)((b + rounds - 1) / rounds);
}
static int dot_blocks(long n) { return (int)std::min<long>(kDotBlocks, (n + kDotChunk - 1) / kDotChunk); }

// Coefficients in LDS: past 64 KiB, the default limit (cycles of more than 4000 steps), a kernel
// has to be told, on the device that it runs on; so for each such launch.
static hipError_t allow_coefs(const void* kernel, size_t bytes) {
  return bytes <= 4000 * sizeof(double2)
             ? hipSuccess
             : hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <typename T>
hipError_t KrylovOps<T>::orthogonalise(const cx<T>* V, int j, cx<T>* w, long n, const ArnoldiData& d, double bnorm,
                                       bool again, double* state, hipStream_t s) {
  const int nv = j + 1, nd = dot_blocks(n), na = axpy_blocks(n);
  double* norms = reinterpret_cast<double*>(d.partial);   // of the update and of the extra sweep's
  double2* dots = d.partial + na;
  int* gate = again ? d.gate : nullptr;
  const dim3 dgrid(nd, (nv + kGroup - 1) / kGroup);
  const size_t coef = (size_t)(nv + 7) * sizeof(double2);
  for (const void* k : {(const void*)k_maxpy_nrm<T, false>, (const void*)k_maxpy_nrm<T, true>, (const void*)k_finish<T>})
    if (hipError_t e = allow_coefs(k, coef)) return e;
  hipLaunchKernelGGL((k_mdot2<T, false>), dgrid, dim3(kThreads), 0, s, V, n, nv, w, n, dots, (const int*)nullptr);
  if (nv <= kProjOne) {
    hipLaunchKernelGGL(k_proj, dim3(1), dim3(kProjThreads), 0, s, dots, nd, nv, d.raw, d.gd, d.H, d.ldh, d.h);
  } else {
    hipLaunchKernelGGL(k_dot_sums, dim3((16 * nv + kProjThreads - 1) / kProjThreads), dim3(kProjThreads), 0, s, dots,
                       nd, nv, d.raw, d.gd, d.H, d.ldh);
    hipLaunchKernelGGL(k_proj_rows, dim3((nv + 63) / 64), dim3(kProjThreads), 0, s, d.raw, d.gd, d.H, d.ldh, nv, d.h);
  }
  hipLaunchKernelGGL((k_maxpy_nrm<T, false>), dim3(na), dim3(kThreads), coef, s, V, n, nv, d.h, w, n, norms,
                     (const int*)nullptr);
  if (again) {
    hipLaunchKernelGGL(k_gate, dim3(1), dim3(kThreads), 0, s, norms, na, d.h, nv, gate);
    hipLaunchKernelGGL((k_mdot2<T, true>), dgrid, dim3(kThreads), 0, s, V, n, nv, w, n, dots, (const int*)gate);
    hipLaunchKernelGGL(k_proj_again, dim3((nv + kThreads / 8 - 1) / (kThreads / 8)), dim3(kThreads), 0, s, dots, nd,
                       nv, d.raw, d.h, (const int*)gate);
    hipLaunchKernelGGL((k_maxpy_nrm<T, true>), dim3(na), dim3(kThreads), coef, s, V, n, nv, d.raw, w, n, norms + na,
                       (const int*)gate);
  }
  hipLaunchKernelGGL((k_finish<T>), dim3(na), dim3(kThreads), (size_t)(j + 2) * sizeof(double2), s, w, n, norms,
                     na, (const int*)gate, d.h, d.H, d.ldh, d.cs, d.sn, d.g, d.pend, j, bnorm, state);
  return hipGetLastError();
}

template <typename T>
hipError_t KrylovOps<T>::scale(const cx<T>* src, cx<T>* dst, long n, const double2* sumsq, hipStream_t s) {
  hipLaunchKernelGGL((k_scale<T>), dim3(2048), dim3(kThreads), 0, s, src, dst, n, sumsq);
  return hipGetLastError();
}

template <typename T>
hipError_t KrylovOps<T>::zero(cx<T>* dst, long n, hipStream_t s) {
  hipLaunchKernelGGL((k_zero<T>), dim3(2048), dim3(kThreads), 0, s, dst, n);
  return hipGetLastError();
}

template <typename T>
hipError_t KrylovOps<T>::trisolve(const double2* H, int ldh, const double2* g, int k, double2* y, hipStream_t s) {
  const size_t lds = sizeof(double2) * (size_t)(k + (k <= kTriLds ? k * k : 0));
  hipLaunchKernelGGL(k_trisolve, dim3(1), dim3(kThreads), lds, s, H, ldh, g, k, y);
  return hipGetLastError();
}

template <typename T>
hipError_t KrylovOps<T>::set_g(double2* pend, const double2* sumsq, hipStream_t s) {
  hipLaunchKernelGGL(k_set_g, dim3(1), dim3(1), 0, s, pend, sumsq);
  return hipGetLastError();
}

template <typename TS, typename TD>
hipError_t convert(const cx<TS>* src, cx<TD>* dst, long n, hipStream_t s) {
  hipLaunchKernelGGL((k_copy<TS, TD>), dim3(2048), dim3(kThreads), 0, s, src, dst, n);
  return hipGetLastError();
}

template struct KrylovOps<double>;
template struct KrylovOps<float>;
template hipError_t KrylovOps<double>::maxpy<double>(const cx<double>*, long, int, const double2*, double,
                                                     cx<double>*, long, hipStream_t);
template hipError_t KrylovOps<float>::maxpy<float>(const cx<float>*, long, int, const double2*, double,
                                                   cx<float>*, long, hipStream_t);
template hipError_t convert<double, float>(const cx<double>*, cx<float>*, long, hipStream_t);
template hipError_t convert<float, double>(const cx<float>*, cx<double>*, long, hipStream_t);
template hipError_t convert<double, double>(const cx<double>*, cx<double>*, long, hipStream_t);

int partial_blocks(long n) { return nblocks(n); }
size_t arnoldi_partials(long n, int m) {
  return std::max<size_t>(2 * (size_t)(m + 1) * dot_blocks(n) + axpy_blocks(n), nblocks(n));
}

static inline int grid_for(long n) {
  const long b = (n + kThreads - 1) / kThreads;
  return (int)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

template <typename T>
hipError_t gather(const Support& u, const cx<T>* full, cx<T>* comp, const cx<T>* sub, hipStream_t s) {
  if (u.s == 0) return hipSuccess;
  hipLaunchKernelGGL((k_gather<T>), dim3(grid_for(u.size())), dim3(kThreads), 0, s, full, comp, sub, u.col, u.s,
                     u.n12, u.n3);
  return hipGetLastError();
}

template <typename T>
hipError_t scatter(const Support& u, const cx<T>* comp, cx<T>* full, hipStream_t s) {
  if (u.s == 0) return hipSuccess;
  hipLaunchKernelGGL((k_scatter<T>), dim3(grid_for(u.size())), dim3(kThreads), 0, s, comp, full, u.col, u.s, u.n12,
                     u.n3, 0);
  return hipGetLastError();
}

template <typename T>
hipError_t zero_support(const Support& u, cx<T>* full, hipStream_t s) {
  if (u.s == 0) return hipSuccess;
  hipLaunchKernelGGL((k_scatter<T>), dim3(grid_for(u.size())), dim3(kThreads), 0, s, nullptr, full, u.col, u.s,
                     u.n12, u.n3, 1);
  return hipGetLastError();
}

hipError_t column_flags(const double2* chi, long n12, int n3, int* flags, hipStream_t s) {
  hipLaunchKernelGGL(k_column_flags, dim3((unsigned)((n12 + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, chi,
                     n12, n3, flags);
  return hipGetLastError();
}

template hipError_t gather<double>(const Support&, const cx<double>*, cx<double>*, const cx<double>*, hipStream_t);
template hipError_t gather<float>(const Support&, const cx<float>*, cx<float>*, const cx<float>*, hipStream_t);
template hipError_t scatter<double>(const Support&, const cx<double>*, cx<double>*, hipStream_t);
template hipError_t scatter<float>(const Support&, const cx<float>*, cx<float>*, hipStream_t);
template hipError_t zero_support<double>(const Support&, cx<double>*, hipStream_t);
template hipError_t zero_support<float>(const Support&, cx<float>*, hipStream_t);

}  // namespace vie
