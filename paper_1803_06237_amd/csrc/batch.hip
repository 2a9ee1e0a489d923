// Batched solves: many systems (uneven grids, each its own plan) advanced in
// lockstep by GMRES(m) or, for the mixed tier, FP64 flexible GMRES(m) whose
// preconditioner is a fixed number of FP32 GMRES steps (Section V-D solves the
// discrete J-VIE with GMRES; the batching, the tiers and the graph capture are
// this library's design).
//
// Every kernel covers the whole batch in one launch: the work of system s is the
// item range [prefix[s], prefix[s+1]) and each workgroup walks items with a grid
// stride.  Convergence is tracked on the device: a system whose residual
// estimate reaches tol clears its flag and every later kernel of the cycle skips
// it, so a whole restart cycle needs no host synchronisation; the second is
// captured as a HIP graph and replayed from then on.  The host synchronises once per cycle to
// read the true residuals.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/vie.h"
#include "fft_device.hpp"
#include "krylov.hpp"
#include "vie_internal.hpp"

namespace vie {

namespace {

constexpr int kT = 256;
constexpr int kE = 4;
constexpr int kC = kT * kE;   // elements per chunk

__device__ __forceinline__ double2 d2(double2 v) { return v; }
__device__ __forceinline__ double2 d2(float2 v) { return double2{(double)v.x, (double)v.y}; }
template <typename V> __device__ __forceinline__ V fromd(double2 v);
template <> __device__ __forceinline__ double2 fromd<double2>(double2 v) { return v; }
template <> __device__ __forceinline__ float2 fromd<float2>(double2 v) { return float2{(float)v.x, (float)v.y}; }

__device__ __forceinline__ int find_item(const int* prefix, int nsys, int item) {
  int lo = 0, hi = nsys - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= item) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

template <int NV>
__device__ __forceinline__ void bsum(double (&v)[NV], double* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < NV; ++i)
    for (int o = 32; o > 0; o >>= 1) v[i] += __shfl_down(v[i], o, 64);
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < NV; ++i) lds[wave * NV + i] = v[i];
  __syncthreads();
  if (threadIdx.x == 0)
    for (int i = 0; i < NV; ++i) {
      double s = 0;
      for (int w = 0; w < kT / 64; ++w) s += lds[w * NV + i];
      v[i] = s;
    }
  __syncthreads();
}

}  // namespace

// Per-system Krylov state (device memory).
struct KDesc {
  void* V;          // (m + 1) * n basis vectors
  void* Z;          // m * n preconditioned vectors (flexible) or null
  void* x;          // solution
  const void* b;    // right-hand side
  void* r;          // residual buffer (cycle start vector)
  long n;
  int nchunk;
  double2* partial; // 2 (m + 1) * nchunk
  double* norms;    // 2 nchunk: ||w||^2 after the update and after the extra sweep's
  double2* h;       // projections of the step
  double2* raw;     // V^H w
  double2* gd;      // Gram diagonal
  double2* sumsq;   // [0] ||w||^2 of the current vector, [1] ||b||^2
  double2* H;       // (m + 1) * m, column-major; Gram entry G_ij, i < j, at row j of column i
  double* cs;
  double2* sn;
  double2* g;
  double2* y;
  int* act;         // active in the current step
  int* go;          // act as the step's projections found it (act may clear while it ends)
  int* again;       // the step needs the extra sweep (FP64)
  const int* act0;  // active for the cycle
  int* kdone;       // Arnoldi steps of the current cycle
  int* iters;       // accumulated steps
  double* est;      // residual estimate |g_{k}| / ||b||
  double tol;
};

// Support compression of one system: Krylov vectors hold the 3 s n3 values of the
// support columns, comp[(a s + p) n3 + i3] = full[a][col[p]][i3], and the product
// runs on the full-length buffers fx (zero off the support) and fy.  fx is null where the
// support is every column: the product then runs on the vectors themselves.
struct SDesc {
  const int* col;   // s increasing column indices i1 n2 + i2
  int s;
  int n3;
  long n12;
  void* fx;
  void* fy;
};

// vector selector: 0 -> V_j, 1 -> Z_j, 2 -> x, 3 -> b, 4 -> r
template <typename T>
__device__ __forceinline__ cx<T>* vsel(const KDesc& D, int which, int j) {
  switch (which) {
    case 0: return (cx<T>*)D.V + (long)j * D.n;
    case 1: return (cx<T>*)D.Z + (long)j * D.n;
    case 2: return (cx<T>*)D.x;
    case 3: return (cx<T>*)D.b;
    default: return (cx<T>*)D.r;
  }
}

// Arnoldi steps as in the single solver (krylov.hip): the two Gram-Schmidt sweeps merged by
// the Gram matrix G = V^H V, h = 2 V^H w - G V^H w, one dot pass and one update pass over the
// basis per step.  (With the sweeps apart, in workgroups that walked all vectors of a chunk:
// 117 us of dots and updates per FP32 step of eight systems of 968k unknowns together; now 28.)
// An FP64 step that cancels too much is measured against the basis once more, as there: k_b_gate
// decides it per system, and dots, their sums and the update run again (AGAIN) for those systems.

// partial[(2 i + s) nchunk + chunk] = V_i^H w (s = 0) and V_i^H V_j (s = 1) over the chunk, for
// the four vectors i of blockIdx.y; w = V_{j+1}
template <typename T, bool AGAIN>
__global__ __launch_bounds__(kT) void k_b_mdot(const KDesc* __restrict__ d, const int* __restrict__ prefix, int nsys,
                                               int j) {
  __shared__ double lds[kT / 64][16];
  const int item = blockIdx.x;
  const int s = find_item(prefix, nsys, item);
  const KDesc& D = d[s];
  if (*(AGAIN ? D.again : D.act) == 0) return;
  const int chunk = item - prefix[s], i0 = blockIdx.y * 4;
  const long n = D.n;
  const cx<T>* V = (const cx<T>*)D.V;
  const cx<T>* vj = V + (long)j * n;
  const cx<T>* w = vj + n;
  // loads from clamped, always valid addresses: all in flight together
  long e[kE];
  double2 wv[kE], vv[kE];
#pragma unroll
  for (int k = 0; k < kE; ++k) {
    const long at = (long)chunk * kC + threadIdx.x + (long)k * kT;
    e[k] = at < n ? at : n - 1;
    wv[k] = d2(w[e[k]]);
    vv[k] = d2(vj[e[k]]);
    if (at >= n) wv[k] = vv[k] = double2{0.0, 0.0};
  }
  double acc[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const cx<T>* Vi = V + (long)(i0 + q <= j ? i0 + q : j) * n;
    double2 a[kE];
#pragma unroll
    for (int k = 0; k < kE; ++k) a[k] = d2(Vi[e[k]]);
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      acc[4 * q] += a[k].x * wv[k].x + a[k].y * wv[k].y;
      acc[4 * q + 1] += a[k].x * wv[k].y - a[k].y * wv[k].x;
      acc[4 * q + 2] += a[k].x * vv[k].x + a[k].y * vv[k].y;
      acc[4 * q + 3] += a[k].x * vv[k].y - a[k].y * vv[k].x;
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int idx;
  const double r = wave_sum_many<16>(acc, lane, &idx);
  if (lane < 16) lds[wave][idx] = r;
  __syncthreads();
  if (threadIdx.x < 16 && i0 + (int)(threadIdx.x >> 2) <= j) {
    double t = 0.0;
    for (int k = 0; k < kT / 64; ++k) t += lds[k][threadIdx.x];
    const long row = 2L * i0 + (threadIdx.x >> 1);
    reinterpret_cast<double*>(D.partial)[2 * (row * D.nchunk + chunk) + (threadIdx.x & 1)] = t;
  }
}

// Sums of the dots, the new Gram column and h, one workgroup per system (as k_proj)
__global__ __launch_bounds__(kProjThreads) void k_b_proj(const KDesc* __restrict__ d, int j, int m) {
  __shared__ ProjLds lds;
  const KDesc& D = d[blockIdx.x];
  const int on = *D.act;
  if (threadIdx.x == 0) *D.go = on;
  if (on == 0) return;
  const int nv = j + 1, ldh = m + 1, sub = threadIdx.x & 7;
  for (int v = threadIdx.x >> 3; v < 2 * nv; v += kProjThreads / 8) {
    double2 s{0.0, 0.0};
#pragma unroll 8
    for (int b = sub; b < D.nchunk; b += 8) {
      const double2 p = D.partial[(long)v * D.nchunk + b];
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
      if ((v & 1) == 0) D.raw[i] = s;
      else if (i < j) D.H[(long)i * ldh + j] = s;
      else D.gd[i] = s;
    }
  }
  __syncthreads();
  for (int i0 = 0; i0 < nv; i0 += 64) project_rows(D.raw, D.gd, D.H, ldh, nv, i0, D.h, lds);
}

// again = 1 where ||w||^2 is too small a part of ||h||^2, one workgroup per system
__global__ __launch_bounds__(kT) void k_b_gate(const KDesc* __restrict__ d, int j) {
  __shared__ double lds[(kT / 64) * 2];
  const KDesc& D = d[blockIdx.x];
  if (*D.go == 0) {
    if (threadIdx.x == 0) *D.again = 0;
    return;
  }
  double v[2] = {0.0, 0.0};
  for (int c = threadIdx.x; c < D.nchunk; c += kT) v[0] += D.norms[c];
  for (int i = threadIdx.x; i <= j; i += kT) v[1] += D.h[i].x * D.h[i].x + D.h[i].y * D.h[i].y;
  bsum<2>(v, lds);
  if (threadIdx.x == 0) *D.again = v[0] < kCancel2 * v[1] ? 1 : 0;
}

// The extra sweep's coefficients: raw = V^H w, and h += raw; one workgroup per system
__global__ __launch_bounds__(kProjThreads) void k_b_proj_again(const KDesc* __restrict__ d, int j) {
  const KDesc& D = d[blockIdx.x];
  if (*D.again == 0) return;
  const int sub = threadIdx.x & 7;
  for (int i = threadIdx.x >> 3; i <= j; i += kProjThreads / 8) {
    double2 s{0.0, 0.0};
    for (int b = sub; b < D.nchunk; b += 8) {
      const double2 p = D.partial[2L * i * D.nchunk + b];
      s.x += p.x;
      s.y += p.y;
    }
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
      s.x += __shfl_xor(s.x, o, 64);
      s.y += __shfl_xor(s.y, o, 64);
    }
    if (sub == 0) {
      D.raw[i] = s;
      D.h[i] = double2{D.h[i].x + s.x, D.h[i].y + s.y};
    }
  }
}

// w = V_{j+1} -= sum_{i <= j} h_i V_i (AGAIN: raw_i) and norms[chunk] = ||w||^2 over the chunk
template <typename T, bool AGAIN>
__global__ __launch_bounds__(kT) void k_b_orth(const KDesc* __restrict__ d, const int* __restrict__ prefix, int nsys,
                                               int j) {
  __shared__ double2 c[512];
  __shared__ double lds[kT / 64];
  const int item = blockIdx.x;
  const int s = find_item(prefix, nsys, item);
  const KDesc& D = d[s];
  if (*(AGAIN ? D.again : D.go) == 0) return;
  const double2* coef = AGAIN ? D.raw : D.h;
  for (int i = threadIdx.x; i <= j + 1; i += kT) c[i] = i <= j ? coef[i] : double2{0.0, 0.0};
  __syncthreads();
  const long n = D.n;
  const int chunk = item - prefix[s];
  const cx<T>* V = (const cx<T>*)D.V;
  cx<T>* w = (cx<T>*)D.V + (long)(j + 1) * n;
  long e[kE];
  double2 acc[kE];
#pragma unroll
  for (int k = 0; k < kE; ++k) {
    const long at = (long)chunk * kC + threadIdx.x + (long)k * kT;
    e[k] = at < n ? at : n - 1;
    acc[k] = d2(w[e[k]]);
  }
  for (int i = 0; i <= j; i += 2) {   // eight loads in flight (the last vector again past the end)
    const cx<T>* Vi = V + (long)i * n;
    const cx<T>* Vk = V + (long)(i < j ? i + 1 : i) * n;
    double2 a[kE], b[kE];
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      a[k] = d2(Vi[e[k]]);
      b[k] = d2(Vk[e[k]]);
    }
    const double2 ca = c[i], cb = c[i + 1];
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      acc[k].x -= ca.x * a[k].x - ca.y * a[k].y;
      acc[k].y -= ca.x * a[k].y + ca.y * a[k].x;
      acc[k].x -= cb.x * b[k].x - cb.y * b[k].y;
      acc[k].y -= cb.x * b[k].y + cb.y * b[k].x;
    }
  }
  double v[1] = {0.0};
#pragma unroll
  for (int k = 0; k < kE; ++k) {
    const long at = (long)chunk * kC + threadIdx.x + (long)k * kT;
    if (at < n) {
      const cx<T> out = fromd<cx<T>>(acc[k]);
      w[at] = out;
      const double2 o = d2(out);
      v[0] += o.x * o.x + o.y * o.y;
    }
  }
  bsum<1>(v, lds);
  if (threadIdx.x == 0) D.norms[(AGAIN ? D.nchunk : 0) + chunk] = v[0];
}

// partial[chunk] = ||v||^2 over the chunk, v selected by (which, j); act_sel: 0 -> act, 1 -> act0
template <typename T>
__global__ __launch_bounds__(kT) void k_b_nrm2(const KDesc* __restrict__ d, const int* __restrict__ prefix, int nsys,
                                               int total, int which, int j, int act_sel) {
  __shared__ double lds[(kT / 64) * 2];
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int s = find_item(prefix, nsys, item);
    const KDesc& D = d[s];
    if ((act_sel ? *D.act0 : *D.act) == 0) continue;
    const int chunk = item - prefix[s];
    const long e0 = (long)chunk * kC + threadIdx.x;
    const cx<T>* v = vsel<T>(D, which, j);
    double acc[2] = {0.0, 0.0};
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      const long e = e0 + (long)k * kT;
      if (e < D.n) {
        const double2 a = d2(v[e]);
        acc[0] += a.x * a.x + a.y * a.y;
      }
    }
    bsum<2>(acc, lds);
    if (threadIdx.x == 0) D.partial[chunk] = double2{acc[0], 0.0};
  }
}

// sumsq[slot] = sum of partial[0..nchunk)
__global__ __launch_bounds__(kT) void k_b_nrm2_fin(const KDesc* __restrict__ d, int nsys, int slot, int act_sel) {
  __shared__ double lds[(kT / 64) * 2];
  for (int s = blockIdx.x; s < nsys; s += gridDim.x) {
    const KDesc& D = d[s];
    if ((act_sel ? *D.act0 : *D.act) == 0) continue;
    double v[2] = {0.0, 0.0};
    for (int c = threadIdx.x; c < D.nchunk; c += kT) v[0] += D.partial[c].x;
    bsum<2>(v, lds);
    if (threadIdx.x == 0) D.sumsq[slot] = double2{v[0], 0.0};
  }
}

// dst = src / sqrt(sumsq[0])
template <typename T>
__global__ __launch_bounds__(kT) void k_b_scale(const KDesc* __restrict__ d, const int* __restrict__ prefix, int nsys,
                                                int total, int wsrc, int jsrc, int jdst, int act_sel) {
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int s = find_item(prefix, nsys, item);
    const KDesc& D = d[s];
    if ((act_sel ? *D.act0 : *D.act) == 0) continue;
    const double nr = sqrt(D.sumsq[0].x);
    const double f = nr > 0.0 ? 1.0 / nr : 0.0;
    const cx<T>* src = vsel<T>(D, wsrc, jsrc);
    cx<T>* dst = (cx<T>*)D.V + (long)jdst * D.n;
    const long e0 = (long)(item - prefix[s]) * kC + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      const long e = e0 + (long)k * kT;
      if (e < D.n) {
        const double2 a = d2(src[e]);
        dst[e] = fromd<cx<T>>(double2{a.x * f, a.y * f});
      }
    }
  }
}

// cycle start: g = (beta, 0, ...), step flags from the cycle flags
__global__ void k_b_init(const KDesc* __restrict__ d, int nsys, int m) {
  for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < nsys; s += gridDim.x * blockDim.x) {
    const KDesc& D = d[s];
    *D.act = *D.act0;
    *D.kdone = 0;
    if (*D.act0 == 0) continue;
    for (int i = 0; i <= m; ++i) D.g[i] = double2{0.0, 0.0};
    D.g[0] = double2{sqrt(D.sumsq[0].x), 0.0};
  }
}

// End of step j: every workgroup sums its system's parts of ||w||^2 and scales its chunk of
// V_{j+1}; the system's first one also does the Hessenberg column, the rotations, the residual
// estimate and the step mask.
template <typename T>
__global__ __launch_bounds__(kT) void k_b_finish(const KDesc* __restrict__ d, const int* __restrict__ prefix, int nsys,
                                                 int j, int m) {
  __shared__ double lds[kT / 64];
  __shared__ double2 h[512];
  __shared__ double s_norm;
  const int item = blockIdx.x;
  const int s = find_item(prefix, nsys, item);
  const KDesc& D = d[s];
  if (*D.go == 0) return;
  const int chunk = item - prefix[s];
  double v[1] = {0.0};
  const double* norms = D.norms + (sizeof(T) == 8 && *D.again != 0 ? D.nchunk : 0);
  for (int c = threadIdx.x; c < D.nchunk; c += kT) v[0] += norms[c];
  bsum<1>(v, lds);
  if (threadIdx.x == 0) s_norm = sqrt(v[0]);
  if (chunk == 0)
    for (int i = threadIdx.x; i <= j; i += kT) h[i] = D.h[i];
  __syncthreads();
  const double hn = s_norm, f = hn > 0.0 ? 1.0 / hn : 0.0;
  cx<T>* w = (cx<T>*)D.V + (long)(j + 1) * D.n;
#pragma unroll
  for (int k = 0; k < kE; ++k) {
    const long e = (long)chunk * kC + threadIdx.x + (long)k * kT;
    if (e < D.n) {
      const double2 a = d2(w[e]);
      w[e] = fromd<cx<T>>(double2{a.x * f, a.y * f});
    }
  }
  if (chunk != 0) return;
  if (threadIdx.x == 0) {
    double2 a = h[0];
    for (int i = 0; i < j; ++i) {
      const double2 bb = h[i + 1];
      const double c = D.cs[i];
      const double2 sn = D.sn[i];
      h[i] = double2{c * a.x + (sn.x * bb.x - sn.y * bb.y), c * a.y + (sn.x * bb.y + sn.y * bb.x)};
      a = double2{-(sn.x * a.x + sn.y * a.y) + c * bb.x, -(sn.x * a.y - sn.y * a.x) + c * bb.y};
    }
    const double2 bb = double2{hn, 0.0};
    const double na = hypot(a.x, a.y), nb = hypot(bb.x, bb.y);
    double c;
    double2 sn, r;
    if (nb == 0.0) {
      c = 1.0;
      sn = double2{0.0, 0.0};
      r = a;
    } else if (na == 0.0) {
      c = 0.0;
      sn = double2{1.0, 0.0};
      r = bb;
    } else {
      const double t = hypot(na, nb);
      const double2 ph = double2{a.x / na, a.y / na};
      c = na / t;
      sn = double2{(ph.x * bb.x + ph.y * bb.y) / t, (ph.y * bb.x - ph.x * bb.y) / t};
      r = double2{ph.x * t, ph.y * t};
    }
    D.cs[j] = c;
    D.sn[j] = sn;
    h[j] = r;
    const double2 gj = D.g[j];
    D.g[j + 1] = double2{-(sn.x * gj.x + sn.y * gj.y), -(sn.x * gj.y - sn.y * gj.x)};
    D.g[j] = double2{c * gj.x, c * gj.y};
    const double bn = sqrt(D.sumsq[1].x);
    const double est = hypot(D.g[j + 1].x, D.g[j + 1].y) / (bn > 0 ? bn : 1.0);
    *D.est = est;
    *D.kdone = j + 1;
    *D.iters += 1;
    if (!(est > D.tol) || hn == 0.0 || !isfinite(est)) *D.act = 0;
  }
  __syncthreads();
  double2* col = D.H + (long)j * (m + 1);
  for (int i = threadIdx.x; i <= j; i += kT) col[i] = h[i];
}

// y = R^{-1} g over the kdone leading columns, one workgroup per system: the right-hand side in
// LDS, every thread updating its rows with the new y_i
__global__ __launch_bounds__(kT) void k_b_trisolve(const KDesc* __restrict__ d, int m) {
  __shared__ double2 r[512];
  const KDesc& D = d[blockIdx.x];
  if (*D.act0 == 0) return;
  const int k = *D.kdone;
  for (int i = threadIdx.x; i < k; i += kT) r[i] = D.g[i];
  __syncthreads();
  for (int i = k - 1; i >= 0; --i) {
    const double2* A = D.H + (long)i * (m + 1);
    const double2 acc = r[i], dd = A[i];
    const double q = dd.x * dd.x + dd.y * dd.y;
    const double2 yi = q > 0 ? double2{(acc.x * dd.x + acc.y * dd.y) / q, (acc.y * dd.x - acc.x * dd.y) / q}
                             : double2{0.0, 0.0};
    if (threadIdx.x == 0) D.y[i] = yi;
    for (int l = threadIdx.x; l < i; l += kT) {
      const double2 a = A[l];
      r[l] = double2{r[l].x - (a.x * yi.x - a.y * yi.y), r[l].y - (a.x * yi.y + a.y * yi.x)};
    }
    __syncthreads();
  }
}

// x += sum_{i < kdone} y_i basis_i (basis = Z if flexible else V)
template <typename T>
__global__ __launch_bounds__(kT) void k_b_update(const KDesc* __restrict__ d, const int* __restrict__ prefix, int nsys,
                                                 int total) {
  __shared__ double2 c[512];
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int s = find_item(prefix, nsys, item);
    const KDesc& D = d[s];
    if (*D.act0 == 0) continue;
    const int k = *D.kdone;
    __syncthreads();
    for (int i = threadIdx.x; i < k; i += kT) c[i] = D.y[i];
    __syncthreads();
    const cx<T>* basis = (const cx<T>*)(D.Z ? D.Z : D.V);
    cx<T>* x = (cx<T>*)D.x;
    const long e0 = (long)(item - prefix[s]) * kC + threadIdx.x;
#pragma unroll
    for (int kk = 0; kk < kE; ++kk) {
      const long e = e0 + (long)kk * kT;
      if (e >= D.n) continue;
      double2 acc = d2(x[e]);
      for (int i = 0; i < k; ++i) {
        const double2 a = d2(basis[(long)i * D.n + e]);
        acc.x += c[i].x * a.x - c[i].y * a.y;
        acc.y += c[i].x * a.y + c[i].y * a.x;
      }
      x[e] = fromd<cx<T>>(acc);
    }
  }
}

// dst(vector of Dd selected by (wd, jd)) = src(vector of Ds selected by (ws, js)), type converted;
// skipped when the source system's step flag is off.  zero = 1 writes zeros instead.
template <typename TS, typename TD>
__global__ __launch_bounds__(kT) void k_b_copy(const KDesc* __restrict__ ds, const KDesc* __restrict__ dd,
                                               const int* __restrict__ prefix, int nsys, int total, int ws, int js,
                                               int wd, int jd, int zero, int act_sel) {
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int s = find_item(prefix, nsys, item);
    const KDesc& S = ds[s];
    const KDesc& Dd = dd[s];
    if ((act_sel ? *S.act0 : *S.act) == 0) continue;
    const cx<TS>* src = vsel<TS>(S, ws, js);
    cx<TD>* dst = vsel<TD>(Dd, wd, jd);
    const long e0 = (long)(item - prefix[s]) * kC + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      const long e = e0 + (long)k * kT;
      if (e < Dd.n) dst[e] = zero ? cx<TD>{(TD)0, (TD)0} : fromd<cx<TD>>(d2(src[e]));
    }
  }
}

__device__ __forceinline__ long full_index(const SDesc& S, long e) {
  const long row = e / S.n3;
  const int t = (int)(e - row * S.n3);
  const int a = (int)(row / S.s), p = (int)(row - (long)a * S.s);
  return ((long)a * S.n12 + S.col[p]) * S.n3 + t;
}

// fx on the support = the compressed vector selected by (which, j); the entries
// off the support stay as they are (zero)
template <typename T>
__global__ __launch_bounds__(kT) void k_b_scatter(const KDesc* __restrict__ d, const SDesc* __restrict__ sd,
                                                  const int* __restrict__ prefix, int nsys, int total, int which,
                                                  int j, int act_sel) {
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int s = find_item(prefix, nsys, item);
    const KDesc& D = d[s];
    if ((act_sel ? *D.act0 : *D.act) == 0) continue;
    const SDesc& S = sd[s];
    if (!S.fx) continue;
    const cx<T>* src = vsel<T>(D, which, j);
    cx<T>* fx = (cx<T>*)S.fx;
    const long e0 = (long)(item - prefix[s]) * kC + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      const long e = e0 + (long)k * kT;
      if (e < D.n) fx[full_index(S, e)] = src[e];
    }
  }
}

// the compressed vector selected by (which, j) = fy on the support; sub = 1:
// = b - fy on the support (the residual of the cycle start)
template <typename T>
__global__ __launch_bounds__(kT) void k_b_gather(const KDesc* __restrict__ d, const SDesc* __restrict__ sd,
                                                 const int* __restrict__ prefix, int nsys, int total, int which,
                                                 int j, int sub, int act_sel) {
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int s = find_item(prefix, nsys, item);
    const KDesc& D = d[s];
    if ((act_sel ? *D.act0 : *D.act) == 0) continue;
    const SDesc& S = sd[s];
    if (!S.fx) continue;
    cx<T>* dst = vsel<T>(D, which, j);
    const cx<T>* b = (const cx<T>*)D.b;
    const cx<T>* fy = (const cx<T>*)S.fy;
    const long e0 = (long)(item - prefix[s]) * kC + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kE; ++k) {
      const long e = e0 + (long)k * kT;
      if (e < D.n) {
        const cx<T> v = fy[full_index(S, e)];
        dst[e] = sub ? cx<T>{b[e].x - v.x, b[e].y - v.y} : v;
      }
    }
  }
}

}  // namespace vie

// =============================================================================
// host side
// =============================================================================
using namespace vie;

namespace {

struct SysPlan : SolveView {};   // the operator of one system; U64, U32 are the batch's own

template <typename T>
struct BatchLevel {         // one Krylov level (outer FP64 or inner FP32) for the whole batch
  int nsys = 0, m = 0;
  bool flex = false;
  std::vector<KDesc> h;
  int* flags = nullptr;     // per system: act, kdone, iters, go, again
  KDesc* d = nullptr;
  std::vector<int> cpre;    // chunk prefix
  int* d_cpre = nullptr;
  int ctotal = 0;
};

// matvec descriptors for one level: step (V_j or Z_j -> V_{j+1}) and residual (x -> r), on
// the full-length buffers of the support descriptors or, for direct systems, on the vectors
struct PassSet {
  std::vector<SDesc> h_sd;        // per system, filled before build_passes
  unsigned char* tables = nullptr;   // device memory of everything below, pass_table_bytes
  SDesc* d_sd = nullptr;
  PassDesc* d_step = nullptr;
  PassDesc* d_res = nullptr;
  std::vector<PassDesc> h_step, h_res;
  // z-pass groups: systems sharing a length and a pencil count, launched together
  struct Group {
    int M3, P;
    bool direct;
    std::vector<int> sys;
    int* d_zpre = nullptr;
    int ztotal = 0;
    PassDesc* d_step = nullptr;
    PassDesc* d_res = nullptr;
  };
  std::vector<Group> zgroups;
  std::vector<int> zsingle;      // systems with z passes of their own
  // cross-section groups: systems of one circulant cross-section with a batched kernel
  struct XyGroup {
    int M1, M2;
    std::vector<int> sys;
    int* d_pre = nullptr;
    int total = 0;
    PassDesc* d_step = nullptr;   // step flags
    PassDesc* d_res = nullptr;    // cycle flags (residual products)
  };
  std::vector<XyGroup> xygroups;
  bool any_scatter = false;       // some system is not direct
  std::vector<int> xysingle;
};

}  // namespace

struct vie_batch_s {
  int nsys;
  hipStream_t stream;
  std::vector<SysPlan> sp;
  BatchLevel<double> outer;
  BatchLevel<float> inner;
  PassSet p64, p32;
  bool mixed;
  bool circ_tier = false;         // FP64 FGMRES preconditioned by each plan's block circulant
  std::vector<Circ*> circ;        // per system (systems of one plan share it)
  std::vector<int> on;            // host copy of the cycle flags
  unsigned char* mem[2] = {nullptr, nullptr};   // the intermediates and vectors; the levels and tables
  hipGraphExec_t graph = nullptr;
  std::string err;
};

namespace {

// The level's arrays (a system without support has length 0 and no chunks; its arrays keep one
// element so every pointer is valid)
template <typename T>
void carve_level(BatchLevel<T>& L, ScratchCarver& c, const std::vector<long>& n, int m, bool flex) {
  L.nsys = (int)n.size();
  L.m = m;
  L.flex = flex;
  L.h.assign(L.nsys, KDesc{});
  L.cpre.assign(L.nsys + 1, 0);
  L.flags = c.take<int>(5 * (size_t)L.nsys);
  double* est = c.take<double>(L.nsys);
  for (int s = 0; s < L.nsys; ++s) {
    KDesc& D = L.h[s];
    D.n = n[s];
    D.nchunk = (int)((n[s] + kC - 1) / kC);
    L.cpre[s + 1] = L.cpre[s] + D.nchunk;
    const size_t len = n[s] > 0 ? (size_t)n[s] : 1, nch = D.nchunk > 0 ? (size_t)D.nchunk : 1;
    D.V = c.take<cx<T>>(len * (m + 1));
    if (flex) D.Z = c.take<cx<T>>(len * m);
    D.r = c.take<cx<T>>(len);
    D.partial = c.take<double2>(2 * (size_t)(m + 1) * nch);
    D.norms = c.take<double>(2 * nch);
    D.h = c.take<double2>((size_t)(m + 2) * 3 + 2 + (size_t)(m + 1) * m + 3 * (size_t)(m + 1));
    D.raw = D.h + (m + 2);
    D.gd = D.raw + (m + 2);
    D.sumsq = D.gd + (m + 2);
    D.H = D.sumsq + 2;
    D.sn = D.H + (size_t)(m + 1) * m;
    D.g = D.sn + (m + 1);
    D.y = D.g + (m + 1);
    D.cs = c.take<double>(m + 1);
    D.act = L.flags + s;
    D.kdone = L.flags + L.nsys + s;
    D.iters = L.flags + 2 * L.nsys + s;
    D.go = L.flags + 3 * L.nsys + s;
    D.again = L.flags + 4 * L.nsys + s;
    D.est = est + s;
  }
  L.ctotal = L.cpre[L.nsys];
  L.d = c.take<KDesc>(L.nsys);
  L.d_cpre = c.take<int>(L.nsys + 1);
}

// cleared flags and the descriptors, completed by the caller
template <typename T>
hipError_t upload_level(BatchLevel<T>& L) {
  hipError_t e = hipMemset(L.flags, 0, sizeof(int) * 5 * L.nsys);
  if (!e) e = hipMemcpy(L.d, L.h.data(), sizeof(KDesc) * L.nsys, hipMemcpyHostToDevice);
  return e ? e : hipMemcpy(L.d_cpre, L.cpre.data(), sizeof(int) * (L.nsys + 1), hipMemcpyHostToDevice);
}

// Bytes of the tables of build_passes at most: each system in one group of either kind, each
// group with two lists of descriptors and a prefix.
size_t pass_table_bytes(int n) {
  return (size_t)n * (sizeof(SDesc) + 4 * sizeof(PassDesc) + 2 * sizeof(int)) +
         (size_t)n * 2 * (sizeof(int) + 3 * 256) + 256;
}

template <typename T>
hipError_t build_passes(vie_batch_s* B, PassSet& PS, const BatchLevel<T>& L) {
  const bool dbl = sizeof(T) == 8;
  ScratchCarver tables{PS.tables};
  auto alloc = [&](void** p, size_t bytes) {
    *p = tables.take<unsigned char>(bytes);
    return tables.used <= pass_table_bytes(B->nsys) ? hipSuccess : hipErrorOutOfMemory;
  };
  hipError_t e;
  const int n = B->nsys;
  PS.h_step.resize(n);
  PS.h_res.resize(n);
  for (int s = 0; s < n; ++s) {
    const SysPlan& P = B->sp[s];
    const KDesc& D = L.h[s];
    PassDesc pd{};
    pd.g = P.g;
    pd.U = dbl ? P.U64 : P.U32;
    pd.goct = dbl ? P.goct64 : P.goct32;
    pd.chi = dbl ? P.chi64 : P.chi32;
    pd.twz = dbl ? P.tw64[2] : P.tw32[2];
    pd.twx = dbl ? P.tw64[0] : P.tw32[0];
    pd.twy = dbl ? P.tw64[1] : P.tw32[1];
    pd.active = D.act;
    if (P.direct) {
      pd.xb = L.flex ? D.Z : D.V;
      pd.yb = D.V;
      pd.xs = pd.ys = D.n;
    } else {
      // the products read fx and write fy; the batched scatter and gather around
      // them move the compressed Krylov vectors
      pd.xb = PS.h_sd[s].fx;
      pd.yb = PS.h_sd[s].fy;
      PS.any_scatter = true;
    }
    PS.h_step[s] = pd;
    pd.active = D.act0;
    if (P.direct) {
      pd.xb = D.x;
      pd.yb = D.r;
      pd.b = D.b;
      pd.xs = pd.ys = 0;
    }
    PS.h_res[s] = pd;
  }
  if ((e = alloc((void**)&PS.d_sd, sizeof(SDesc) * n))) return e;
  if ((e = hipMemcpy(PS.d_sd, PS.h_sd.data(), sizeof(SDesc) * n, hipMemcpyHostToDevice))) return e;
  // z groups.  A plan's own operator keeps its tuned choice of one
  // pencil per workgroup.  Pencils per workgroup: those that leave the
  // fewest idle in the last block of a row, then the most.
  for (int s = 0; s < n; ++s) {
    const SysPlan& P = B->sp[s];
    const Tune& t = dbl ? P.t64 : P.t32;
    int opts[8], r[3];
    const int no = z3_pencil_options<T>(P.g.M3, opts, 8);
    if (z3_radices(P.g.M3, r) && (P.box || t.z3 || !no)) {
      int Pp = z3_pencils<T>(P.g.M3, P.g.n1);
      auto padded = [&](int q) { return (P.g.n1 + q - 1) / q * q; };
      for (int i = 0; i < no; ++i)
        if (padded(opts[i]) < padded(Pp) || (padded(opts[i]) == padded(Pp) && opts[i] > Pp)) Pp = opts[i];
      auto it = std::find_if(PS.zgroups.begin(), PS.zgroups.end(), [&](const PassSet::Group& G) {
        return G.M3 == P.g.M3 && G.P == Pp && G.direct == P.direct;
      });
      if (it == PS.zgroups.end()) {
        PS.zgroups.push_back(PassSet::Group{P.g.M3, Pp, P.direct, {}, nullptr, 0, nullptr, nullptr});
        it = PS.zgroups.end() - 1;
      }
      it->sys.push_back(s);
    } else {
      PS.zsingle.push_back(s);
    }
    if (!((P.g.M1 == 64 && P.g.M2 == 64) || xyr_fits_batch(P.g))) {
      PS.xysingle.push_back(s);
      continue;
    }
    auto it = std::find_if(PS.xygroups.begin(), PS.xygroups.end(),
                           [&](const PassSet::XyGroup& G) { return G.M1 == P.g.M1 && G.M2 == P.g.M2; });
    if (it == PS.xygroups.end()) {
      PS.xygroups.push_back(PassSet::XyGroup{P.g.M1, P.g.M2, {}, nullptr, 0, nullptr, nullptr});
      it = PS.xygroups.end() - 1;
    }
    it->sys.push_back(s);
  }
  for (auto& G : PS.zgroups) {
    std::vector<int> pre(G.sys.size() + 1, 0);
    std::vector<PassDesc> st, rs;
    for (size_t i = 0; i < G.sys.size(); ++i) {
      const Geom& g = B->sp[G.sys[i]].g;
      pre[i + 1] = pre[i] + 3 * g.n2 * ((g.n1 + G.P - 1) / G.P);
      PassDesc a = PS.h_step[G.sys[i]], r = PS.h_res[G.sys[i]];
      a.P = r.P = G.P;
      st.push_back(a);
      rs.push_back(r);
    }
    G.ztotal = pre.back();
    if ((e = alloc((void**)&G.d_zpre, sizeof(int) * pre.size()))) return e;
    if ((e = hipMemcpy(G.d_zpre, pre.data(), sizeof(int) * pre.size(), hipMemcpyHostToDevice))) return e;
    if ((e = alloc((void**)&G.d_step, sizeof(PassDesc) * st.size()))) return e;
    if ((e = hipMemcpy(G.d_step, st.data(), sizeof(PassDesc) * st.size(), hipMemcpyHostToDevice))) return e;
    if ((e = alloc((void**)&G.d_res, sizeof(PassDesc) * rs.size()))) return e;
    if ((e = hipMemcpy(G.d_res, rs.data(), sizeof(PassDesc) * rs.size(), hipMemcpyHostToDevice))) return e;
  }
  for (auto& G : PS.xygroups) {
    std::vector<int> pre(G.sys.size() + 1, 0);
    std::vector<PassDesc> st, rs;
    for (size_t i = 0; i < G.sys.size(); ++i) {
      const Geom& g = B->sp[G.sys[i]].g;
      const int per = xyr_fits_batch(g) ? xyr_planes_per_group(g) : 2;   // else plane pairs
      pre[i + 1] = pre[i] + (g.M3 + per - 1) / per;
      st.push_back(PS.h_step[G.sys[i]]);
      rs.push_back(PS.h_res[G.sys[i]]);
    }
    G.total = pre.back();
    if ((e = alloc((void**)&G.d_pre, sizeof(int) * pre.size()))) return e;
    if ((e = hipMemcpy(G.d_pre, pre.data(), sizeof(int) * pre.size(), hipMemcpyHostToDevice))) return e;
    if ((e = alloc((void**)&G.d_step, sizeof(PassDesc) * st.size()))) return e;
    if ((e = hipMemcpy(G.d_step, st.data(), sizeof(PassDesc) * st.size(), hipMemcpyHostToDevice))) return e;
    if ((e = alloc((void**)&G.d_res, sizeof(PassDesc) * rs.size()))) return e;
    if ((e = hipMemcpy(G.d_res, rs.data(), sizeof(PassDesc) * rs.size(), hipMemcpyHostToDevice))) return e;
  }
  return hipSuccess;
}

// Batched matvec on compressed vectors: residual = false: V_{j+1} = A (V_j or
// Z_j), systems gated by their step flags; true: r = b - A x, gated by the cycle
// flags.  Direct systems run the three passes on the vectors; the others scatter into
// fx, run fx -> fy and gather from fy.
template <typename T>
hipError_t batch_matvec(vie_batch_s* B, PassSet& PS, const BatchLevel<T>& L, bool residual, int j) {
  hipStream_t s = B->stream;
  hipError_t e;
  const int jx = residual ? 0 : j, jy = residual ? 0 : j + 1;
  const bool dbl = sizeof(T) == 8;
  const int act_sel = residual ? 1 : 0;
  const int gsz = L.ctotal < 4096 ? (L.ctotal > 0 ? L.ctotal : 1) : 4096;
  if (PS.any_scatter) {
    hipLaunchKernelGGL((k_b_scatter<T>), dim3(gsz), dim3(kT), 0, s, L.d, PS.d_sd, L.d_cpre, L.nsys, L.ctotal,
                       residual ? 2 : (L.flex ? 1 : 0), residual ? 0 : j, act_sel);
    if ((e = hipGetLastError())) return e;
  }
  for (int which = 0; which < 3; ++which) {
    if (which == 1) {
      for (auto& G : PS.xygroups) {
        const PassDesc* d = residual ? G.d_res : G.d_step;
        const int ns = (int)G.sys.size();
        if ((e = G.M1 == 64 && G.M2 == 64 ? launch_xy64_batch<T>(d, G.d_pre, ns, G.total, s)
                                          : launch_xyr_batch<T>(G.M1, G.M2, d, G.d_pre, ns, G.total, s)))
          return e;
      }
      for (int sidx : PS.xysingle) {
        const SysPlan& P = B->sp[sidx];
        if ((e = launch_pass<T>(1, P.g, dbl ? P.t64 : P.t32, nullptr, nullptr, nullptr, 0, dbl ? P.U64 : P.U32,
                                dbl ? P.goct64 : P.goct32, dbl ? P.chi64 : P.chi32, dbl ? P.tw64 : P.tw32, s)))
          return e;
      }
      continue;
    }
    for (auto& G : PS.zgroups)
      if ((e = launch_z3_batch<T>(which, residual && G.direct ? 1 : 0, residual ? G.d_res : G.d_step, G.d_zpre,
                                  (int)G.sys.size(), G.ztotal, G.M3, G.P, jx, jy, s)))
        return e;
    for (int sidx : PS.zsingle) {
      const SysPlan& P = B->sp[sidx];
      const PassDesc& pd = residual ? PS.h_res[sidx] : PS.h_step[sidx];
      const void* xp = (const cx<T>*)pd.xb + (long)jx * pd.xs;
      void* yp = (cx<T>*)pd.yb + (long)jy * pd.ys;
      if ((e = launch_pass<T>(which, P.g, dbl ? P.t64 : P.t32, xp, yp, pd.b, residual && P.direct ? 1 : 0,
                              dbl ? P.U64 : P.U32, dbl ? P.goct64 : P.goct32, dbl ? P.chi64 : P.chi32,
                              dbl ? P.tw64 : P.tw32, s)))
        return e;
    }
  }
  if (PS.any_scatter)
    hipLaunchKernelGGL((k_b_gather<T>), dim3(gsz), dim3(kT), 0, s, L.d, PS.d_sd, L.d_cpre, L.nsys, L.ctotal,
                       residual ? 4 : 0, residual ? 0 : j + 1, residual ? 1 : 0, act_sel);
  return hipGetLastError();
}

inline int grid_for(int total) { return total < 4096 ? (total > 0 ? total : 1) : 4096; }

// Norm of a vector of every cycle-active system into sumsq[slot].
template <typename T>
hipError_t batch_norm(hipStream_t s, const BatchLevel<T>& L, int which, int j, int slot, int act_sel) {
  hipLaunchKernelGGL((k_b_nrm2<T>), dim3(grid_for(L.ctotal)), dim3(kT), 0, s, L.d, L.d_cpre, L.nsys, L.ctotal, which,
                     j, act_sel);
  hipLaunchKernelGGL(k_b_nrm2_fin, dim3(L.nsys), dim3(kT), 0, s, L.d, L.nsys, slot, act_sel);
  return hipGetLastError();
}

template <typename T>
hipError_t enqueue_cycle(vie_batch_s* B, BatchLevel<T>& L, PassSet& PS, int inner_steps);

// Inner FP32 GMRES for outer step j: b32 = V64_j, x32 = 0, inner_steps Arnoldi
// steps (masked at inner tol), x32 update, Z64_j = x32.
hipError_t enqueue_inner(vie_batch_s* B, int j) {
  hipStream_t s = B->stream;
  BatchLevel<float>& I = B->inner;
  BatchLevel<double>& O = B->outer;
  // inner rhs and zero start (inner cycle flags alias the outer step flags)
  hipLaunchKernelGGL((k_b_copy<double, float>), dim3(grid_for(O.ctotal)), dim3(kT), 0, s, O.d, I.d, O.d_cpre, O.nsys,
                     O.ctotal, 0, j, 3, 0, 0, 0);
  hipLaunchKernelGGL((k_b_copy<float, float>), dim3(grid_for(I.ctotal)), dim3(kT), 0, s, I.d, I.d, I.d_cpre, I.nsys,
                     I.ctotal, 3, 0, 2, 0, 1, 1);
  hipError_t e;
  if ((e = batch_norm<float>(s, I, 3, 0, 1, 1))) return e;       // ||b||^2 -> sumsq[1]
  if ((e = batch_norm<float>(s, I, 3, 0, 0, 1))) return e;       // beta^2 -> sumsq[0]
  hipLaunchKernelGGL((k_b_scale<float>), dim3(grid_for(I.ctotal)), dim3(kT), 0, s, I.d, I.d_cpre, I.nsys, I.ctotal, 3,
                     0, 0, 1);
  if ((e = enqueue_cycle<float>(B, I, B->p32, 0))) return e;
  hipLaunchKernelGGL((k_b_copy<float, double>), dim3(grid_for(I.ctotal)), dim3(kT), 0, s, I.d, O.d, I.d_cpre, I.nsys,
                     I.ctotal, 2, 0, 1, j, 0, 1);
  return hipGetLastError();
}

// One restart cycle (V_0 already holds r / beta and sumsq[0] = beta^2):
// init, m Arnoldi steps with CGS2, triangular solve, x update.
template <typename T>
hipError_t enqueue_cycle(vie_batch_s* B, BatchLevel<T>& L, PassSet& PS, int) {
  hipStream_t s = B->stream;
  hipError_t e;
  hipLaunchKernelGGL(k_b_init, dim3((L.nsys + 63) / 64), dim3(64), 0, s, L.d, L.nsys, L.m);
  for (int j = 0; j < L.m; ++j) {
    if (L.flex && B->mixed) {
      if ((e = enqueue_inner(B, j))) return e;
    } else if (L.flex && B->circ_tier) {
      // Z_j = W^{-1} V_j for the systems active in this cycle, one after the other
      // on the batch stream (systems that share a plan share its work buffers)
      for (int i = 0; i < L.nsys; ++i) {
        if (!B->on[i]) continue;
        const KDesc& D = L.h[i];
        if ((e = circ_apply_rows(B->circ[i], (const double2*)D.V + (long)j * D.n, (double2*)D.Z + (long)j * D.n,
                                 s)))
          return e;
      }
    }
    if ((e = batch_matvec<T>(B, PS, L, false, j))) return e;
    if (L.ctotal > 0) {
      const dim3 chunks((unsigned)L.ctotal), dots((unsigned)L.ctotal, (unsigned)(j + 4) / 4), systems((unsigned)L.nsys);
      hipLaunchKernelGGL((k_b_mdot<T, false>), dots, dim3(kT), 0, s, L.d, L.d_cpre, L.nsys, j);
      hipLaunchKernelGGL(k_b_proj, systems, dim3(kProjThreads), 0, s, L.d, j, L.m);
      hipLaunchKernelGGL((k_b_orth<T, false>), chunks, dim3(kT), 0, s, L.d, L.d_cpre, L.nsys, j);
      if (sizeof(T) == 8) {
        hipLaunchKernelGGL(k_b_gate, systems, dim3(kT), 0, s, L.d, j);
        hipLaunchKernelGGL((k_b_mdot<T, true>), dots, dim3(kT), 0, s, L.d, L.d_cpre, L.nsys, j);
        hipLaunchKernelGGL(k_b_proj_again, systems, dim3(kProjThreads), 0, s, L.d, j);
        hipLaunchKernelGGL((k_b_orth<T, true>), chunks, dim3(kT), 0, s, L.d, L.d_cpre, L.nsys, j);
      }
      hipLaunchKernelGGL((k_b_finish<T>), chunks, dim3(kT), 0, s, L.d, L.d_cpre, L.nsys, j, L.m);
    }
  }
  hipLaunchKernelGGL(k_b_trisolve, dim3((unsigned)L.nsys), dim3(kT), 0, s, L.d, L.m);
  hipLaunchKernelGGL((k_b_update<T>), dim3(grid_for(L.ctotal)), dim3(kT), 0, s, L.d, L.d_cpre, L.nsys, L.ctotal);
  return hipGetLastError();
}

}  // namespace

extern "C" int vie_solve_batch(vie_plan_t const* plans, const vie_c128* const* rhs, vie_c128* const* x, int count,
                               double tol, const vie_solve_opts* opts, vie_solve_info* infos) {
  if (!plans || !rhs || !x || count < 1 || !(tol > 0)) return VIE_EINVAL;
  vie_solve_opts o{50, 10000, 0, 0, 20, 1e-4, 1, 0};
  if (opts) o = *opts;
  hipStream_t user_stream = nullptr;
  if (o.restart <= 0) o.restart = 50;
  if (o.maxit <= 0) o.maxit = 10000;
  if (o.inner_restart <= 0) o.inner_restart = 20;
  if (!(o.inner_tol > 0)) o.inner_tol = 1e-4;
  if (o.restart > 500 || o.inner_restart > 500) return VIE_EINVAL;
  const auto t0 = std::chrono::steady_clock::now();
  vie_batch_s B;
  B.nsys = count;
  B.sp.resize(count);
  if (o.precision < 0 || o.precision > 3 || o.precision == 2) return VIE_EINVAL;
  B.mixed = o.precision == 1;
  B.circ_tier = o.precision == 3;
  if (B.circ_tier) o.use_graph = 0;   // the active set is chosen on the host per cycle
  B.circ.assign(count, nullptr);
  std::vector<long> n(count), nfull(count);
  std::vector<Support> sup(count);
  std::vector<SysPlan> own(count);   // the plans' own operators (b off the support)
  for (int s = 0; s < count; ++s) {
    SysPlan& P = own[s];
    hipStream_t st;
    int hc = 0;
    if (!plans[s] || !rhs[s] || !x[s]) return VIE_EINVAL;
    int rc = plan_export(plans[s], &P.g, &P.t64, &P.t32, &P.U64, &P.U32, &P.goct64, &P.goct32, &P.chi64, &P.chi32,
                         P.tw64, P.tw32, &st, &hc);
    if (rc) return rc;
    if (!hc) return VIE_ESTATE;
    if (B.mixed && !P.goct32) return VIE_ESTATE;
    if (B.circ_tier && !(B.circ[s] = plan_circ(plans[s]))) return VIE_ESTATE;
    if (s == 0) user_stream = st;
    const int* col = nullptr;
    int ns = 0;
    if ((rc = plan_support(plans[s], &col, &ns))) return rc;
    if ((rc = plan_solve_view(plans[s], &B.sp[s]))) return rc;
    P.direct = (long)ns == (long)P.g.n1 * P.g.n2;
    sup[s] = Support{col, ns, (long)P.g.n1 * P.g.n2, P.g.n3};
    nfull[s] = 3 * P.g.N;
    n[s] = sup[s].size();   // Krylov vectors hold the support columns only
  }
  // the batch runs on a stream of its own (graph capture needs a non-default
  // stream), ordered after the caller's stream, and returns synchronised
  if (hipStreamSynchronize(user_stream) != hipSuccess) return VIE_EDEVICE;
  if (hipStreamCreateWithFlags(&B.stream, hipStreamNonBlocking) != hipSuccess) return VIE_EDEVICE;
  hipStream_t s = B.stream;
  std::vector<const void*> bptr(count);
  std::vector<void*> xptr(count);
  int status = VIE_OK;
  int* act = nullptr;    // cycle flags (outer)
  int* hflags = nullptr;
  std::vector<void*> extra;
  auto cleanup = [&]() {
    if (B.graph) (void)hipGraphExecDestroy(B.graph);
    for (void* q : extra) (void)hipFree(q);
    if (hflags) (void)hipHostFree(hflags);
    (void)hipStreamSynchronize(B.stream);
    for (unsigned char* q : B.mem)
      if (q) (void)hipFree(q);
    (void)hipStreamDestroy(B.stream);
  };
#define BTRY(expr)                  \
  do {                              \
    hipError_t _e = (expr);         \
    if (_e != hipSuccess) {         \
      cleanup();                    \
      return VIE_EDEVICE;           \
    }                               \
  } while (0)
  // Support compression (as in vie_solve): off the support A is the identity, so
  // x = b there; on it the system is A_SS x_S = b_S - (A b_off)_S with b_off = b
  // off the support.  Per system: intermediates of its own, so that one plan may serve several
  // right-hand sides of the batch, the compressed right-hand side bc and solution xc and,
  // unless its support is every column of its operator's grid, the product's full-length
  // buffers fx (zero off the support) and fy.
  B.p64.h_sd.resize(count);
  B.p32.h_sd.resize(count);
  long nmax = 1;
  for (int i = 0; i < count; ++i) nmax = std::max(nmax, nfull[i]);
  double2 *boffv = nullptr, *dsq = nullptr, *part = nullptr;
  auto carve_vectors = [&](ScratchCarver& c) {
    act = c.take<int>(count);
    for (int i = 0; i < count; ++i) {
      SysPlan& P = B.sp[i];
      const size_t len = n[i] > 0 ? (size_t)n[i] : 1, nv = 3 * (size_t)P.g.N;
      const size_t u = (size_t)3 * P.g.n1 * P.g.n2 * P.g.M3;
      P.U64 = c.take<double2>(u);
      bptr[i] = c.take<double2>(len);
      xptr[i] = c.take<double2>(len);
      SDesc sd{P.col, P.ns, P.g.n3, (long)P.g.n1 * P.g.n2, nullptr, nullptr};
      B.p64.h_sd[i] = B.p32.h_sd[i] = sd;
      if (!P.direct) {
        B.p64.h_sd[i].fx = c.take<double2>(nv);
        B.p64.h_sd[i].fy = c.take<double2>(nv);
      }
      if (!B.mixed) continue;
      P.U32 = c.take<float2>(u);
      if (!P.direct) {
        B.p32.h_sd[i].fx = c.take<float2>(nv);
        B.p32.h_sd[i].fy = c.take<float2>(nv);
      }
    }
    boffv = c.take<double2>(nmax);   // b off the support, one system after the other
    // norms: dsq[3 i] = ||b_S||^2, dsq[3 i + 1] = ||b_off||^2, dsq[3 i + 2] = ||b_c||^2
    dsq = c.take<double2>(3 * count);
    part = c.take<double2>(partial_blocks(nmax));
  };
  std::vector<float2*> ib(count, nullptr), ix(count, nullptr);   // inner right-hand sides and solutions
  auto carve_levels = [&](ScratchCarver& c) {
    carve_level<double>(B.outer, c, n, o.restart, B.mixed || B.circ_tier);
    B.p64.tables = c.take<unsigned char>(pass_table_bytes(count));
    if (!B.mixed) return;
    for (int i = 0; i < count; ++i) {
      ib[i] = c.take<float2>(n[i] > 0 ? n[i] : 1);
      ix[i] = c.take<float2>(n[i] > 0 ? n[i] : 1);
    }
    carve_level<float>(B.inner, c, n, o.inner_restart, false);
    B.p32.tables = c.take<unsigned char>(pass_table_bytes(count));
  };
  // One allocation of the size that a first walk over the arrays finds (158 single ones of an
  // eight-system batch took 3.5 ms to make and 11 ms to free).
  auto allocate = [&](unsigned char*& base, auto carve) -> hipError_t {
    ScratchCarver size{nullptr};
    carve(size);
    if (hipError_t e = dmalloc(&base, size.used)) return e;
    ScratchCarver c{base};
    carve(c);
    return hipSuccess;
  };
  BTRY(allocate(B.mem[0], carve_vectors));
  BTRY(hipHostMalloc(&hflags, sizeof(int) * count * 4 + sizeof(double) * count * 4, hipHostMallocDefault));
  for (int i = 0; i < count; ++i) {
    const size_t nv = 3 * (size_t)B.sp[i].g.N;
    if (B.p64.h_sd[i].fx) BTRY(hipMemsetAsync(B.p64.h_sd[i].fx, 0, sizeof(double2) * nv, s));
    if (B.p32.h_sd[i].fx) BTRY(hipMemsetAsync(B.p32.h_sd[i].fx, 0, sizeof(float2) * nv, s));
  }
  BTRY(hipMemsetAsync(dsq, 0, sizeof(double2) * 3 * count, s));
  using K = KrylovOps<double>;
  for (int i = 0; i < count; ++i) {
    if (sup[i].s > 0) {
      BTRY(gather<double>(sup[i], (const double2*)rhs[i], (double2*)bptr[i], nullptr, s));
      BTRY(K::nrm2sq((const double2*)bptr[i], n[i], part, dsq + 3 * i, s));
    }
    if (own[i].direct) continue;   // nothing off the support
    BTRY(hipMemcpyAsync(boffv, rhs[i], sizeof(double2) * nfull[i], hipMemcpyDeviceToDevice, s));
    if (sup[i].s > 0) BTRY(zero_support<double>(sup[i], boffv, s));
    BTRY(K::nrm2sq(boffv, nfull[i], part, dsq + 3 * i + 1, s));
  }
  std::vector<double2> hsq(3 * count);
  BTRY(hipMemcpyAsync(hsq.data(), dsq, sizeof(double2) * 3 * count, hipMemcpyDeviceToHost, s));
  BTRY(hipStreamSynchronize(s));
  std::vector<int> boff(count, 0);
  for (int i = 0; i < count; ++i) {
    if (!std::isfinite(hsq[3 * i].x) || !std::isfinite(hsq[3 * i + 1].x)) {
      cleanup();
      return VIE_EINVAL;   // right-hand side not finite
    }
    boff[i] = sup[i].s > 0 && hsq[3 * i + 1].x > 0;
    if (!boff[i]) continue;
    // with the plan's own operator, on buffers of its own (the plan's may be in use)
    const SysPlan& P = own[i];
    double2 *y = nullptr, *U = nullptr;
    BTRY(dmalloc(&y, sizeof(double2) * nfull[i]));
    extra.push_back(y);
    BTRY(dmalloc(&U, sizeof(double2) * 3 * (size_t)P.g.n1 * P.g.n2 * P.g.M3));
    extra.push_back(U);
    BTRY(hipMemcpyAsync(boffv, rhs[i], sizeof(double2) * nfull[i], hipMemcpyDeviceToDevice, s));
    BTRY(zero_support<double>(sup[i], boffv, s));
    BTRY(launch_matvec<double>(P.g, P.t64, boffv, y, nullptr, 0, U, P.goct64, P.chi64, P.tw64, s));
    BTRY(gather<double>(sup[i], y, (double2*)bptr[i], (const double2*)bptr[i], s));
    BTRY(K::nrm2sq((const double2*)bptr[i], n[i], part, dsq + 3 * i + 2, s));
    BTRY(hipStreamSynchronize(s));
    (void)hipFree(extra.back());
    extra.pop_back();
    (void)hipFree(extra.back());
    extra.pop_back();
  }
  BTRY(hipMemcpyAsync(hsq.data(), dsq, sizeof(double2) * 3 * count, hipMemcpyDeviceToHost, s));
  BTRY(hipStreamSynchronize(s));
  // ||r|| / ||b|| = (||r_c|| / ||b_c||) * ratio with ratio = ||b_c|| / ||b||
  std::vector<double> ratio(count, 0.0), tolc(count, tol);
  for (int i = 0; i < count; ++i) {
    const double bnorm = std::sqrt(hsq[3 * i].x + hsq[3 * i + 1].x);
    const double bcsq = boff[i] ? hsq[3 * i + 2].x : hsq[3 * i].x;
    if (bnorm > 0 && bcsq > 0) {
      ratio[i] = std::sqrt(bcsq) / bnorm;
      tolc[i] = tol / ratio[i];
    }
  }
  BTRY(allocate(B.mem[1], carve_levels));
  for (int i = 0; i < count; ++i) {
    KDesc& D = B.outer.h[i];
    D.b = bptr[i];
    D.x = xptr[i];
    D.act0 = act + i;
    D.tol = tolc[i];
  }
  BTRY(upload_level(B.outer));
  if (B.mixed) {
    // inner cycle flags alias the outer step flags (an outer system that stopped
    // needs no preconditioning); the inner level has its own step flags
    for (int i = 0; i < count; ++i) {
      KDesc& D = B.inner.h[i];
      D.b = ib[i];
      D.x = ix[i];
      D.act0 = B.outer.h[i].act;
      D.tol = o.inner_tol;
    }
    BTRY(upload_level(B.inner));
    BTRY(build_passes<float>(&B, B.p32, B.inner));
  }
  BTRY(build_passes<double>(&B, B.p64, B.outer));
  BatchLevel<double>& O = B.outer;
  // all systems on for the set-up reductions
  std::vector<int> on(count, 1);
  BTRY(hipMemcpyAsync(act, on.data(), sizeof(int) * count, hipMemcpyHostToDevice, s));
  BTRY(batch_norm<double>(s, O, 3, 0, 1, 1));          // ||b_c||^2
  if (o.use_x0) {
    for (int i = 0; i < count; ++i)
      if (sup[i].s > 0) BTRY(gather<double>(sup[i], (const double2*)x[i], (double2*)xptr[i], nullptr, s));
    BTRY(batch_matvec<double>(&B, B.p64, O, true, 0));  // r = b - A x
  } else {
    hipLaunchKernelGGL((k_b_copy<double, double>), dim3(grid_for(O.ctotal)), dim3(kT), 0, s, O.d, O.d, O.d_cpre,
                       count, O.ctotal, 3, 0, 2, 0, 1, 1);   // x = 0
    hipLaunchKernelGGL((k_b_copy<double, double>), dim3(grid_for(O.ctotal)), dim3(kT), 0, s, O.d, O.d, O.d_cpre,
                       count, O.ctotal, 3, 0, 4, 0, 0, 1);   // r = b
  }
  std::vector<int> iters(count, 0), inner_it(count, 0), restarts(count, 0), matvecs(count, 0);
  std::vector<double> bn(count), rel(count), est(count);
  std::vector<double2> sq(2 * count);
  bool graph_built = false;
  int cycles = 0;
  while (true) {
    // residual norms of the cycle start: sumsq[0] = ||r||^2
    BTRY(batch_norm<double>(s, O, 4, 0, 0, 1));
    for (int i = 0; i < count; ++i)
      BTRY(hipMemcpyAsync(&sq[2 * i], O.h[i].sumsq, sizeof(double2) * 2, hipMemcpyDeviceToHost, s));
    BTRY(hipMemcpyAsync(hflags, O.h[0].iters - 2 * count, sizeof(int) * 3 * count, hipMemcpyDeviceToHost, s));
    BTRY(hipStreamSynchronize(s));
    int nact = 0;
    for (int i = 0; i < count; ++i) {
      bn[i] = std::sqrt(sq[2 * i + 1].x);
      rel[i] = bn[i] > 0 ? std::sqrt(sq[2 * i].x) / bn[i] * ratio[i] : 0.0;
      iters[i] = hflags[2 * count + i];
      on[i] = (std::isfinite(rel[i]) && rel[i] > tol && iters[i] < o.maxit) ? 1 : 0;
      if (!std::isfinite(rel[i])) status = VIE_ENUMERIC;
      nact += on[i];
    }
    if (nact == 0 || status == VIE_ENUMERIC) break;
    B.on = on;
    BTRY(hipMemcpyAsync(act, on.data(), sizeof(int) * count, hipMemcpyHostToDevice, s));
    // V_0 = r / beta for the active systems
    hipLaunchKernelGGL((k_b_scale<double>), dim3(grid_for(O.ctotal)), dim3(kT), 0, s, O.d, O.d_cpre, count, O.ctotal,
                       4, 0, 0, 1);
    // The first cycle is launched kernel by kernel, which overlaps with its execution; the
    // graph, which does not (8 ms to build and destroy for 30 outer steps of 20 inner ones,
    // against 65 ms of work), is for further cycles.
    if (o.use_graph && cycles > 0) {
      if (!graph_built) {
        hipGraph_t gr;
        BTRY(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
        hipError_t ce = enqueue_cycle<double>(&B, O, B.p64, 0);
        hipError_t ee = hipStreamEndCapture(s, &gr);
        if (ce || ee) {
          cleanup();
          return VIE_EDEVICE;
        }
        BTRY(hipGraphInstantiate(&B.graph, gr, nullptr, nullptr, 0));
        (void)hipGraphDestroy(gr);
        graph_built = true;
      }
      BTRY(hipGraphLaunch(B.graph, s));
    } else {
      BTRY(enqueue_cycle<double>(&B, O, B.p64, 0));
    }
    ++cycles;
    for (int i = 0; i < count; ++i)
      if (on[i]) restarts[i]++;
    // true residual r = b - A x of the active systems
    BTRY(batch_matvec<double>(&B, B.p64, O, true, 0));
    if (cycles > 100000) break;
  }
  // x = b off the support, xc on it
  for (int i = 0; i < count; ++i) {
    BTRY(hipMemcpyAsync(x[i], rhs[i], sizeof(double2) * nfull[i], hipMemcpyDeviceToDevice, s));
    if (sup[i].s > 0) BTRY(scatter<double>(sup[i], (const double2*)xptr[i], (double2*)x[i], s));
  }
  // report
  std::vector<int> inn(count, 0);
  BTRY(hipStreamSynchronize(s));
  if (B.mixed) {
    // flags of the inner level: [act | kdone | iters], nsys each
    std::vector<int> all(3 * count);
    BTRY(hipMemcpy(all.data(), B.inner.h[0].act, sizeof(int) * 3 * count, hipMemcpyDeviceToHost));
    for (int i = 0; i < count; ++i) inn[i] = all[2 * count + i];
  }
  const double secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  int worst = status;
  for (int i = 0; i < count; ++i) {
    const int st = status == VIE_ENUMERIC ? VIE_ENUMERIC : (rel[i] <= tol ? VIE_OK : VIE_ENOCONV);
    if (st != VIE_OK && worst == VIE_OK) worst = st;
    if (infos) {
      infos[i].iters = iters[i];
      infos[i].inner_iters = inn[i];
      infos[i].restarts = restarts[i];
      infos[i].matvecs = iters[i] + restarts[i] + (o.use_x0 ? 1 : 0) + boff[i];
      infos[i].status = st;
      infos[i].rel_res_true = rel[i];
      infos[i].rel_res_est = rel[i];
      infos[i].seconds = secs;
      infos[i].fallback = 0;
      infos[i].stalled = 0;
    }
  }
  cleanup();
#undef BTRY
  return worst;
}
