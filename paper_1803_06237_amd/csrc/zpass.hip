// Passes 1 and 3 of the matvec (zero-padded z FFT / inverse z FFT with crop and
// contrast) as transforms of two or three stages held in registers, for circulant
// lengths M3 >= 64.
//
// From 512 on M3 = R1 R2 R3 with radices of 8 to 16 (z3_radices).  With n = u + R3 s + R2 R3 j
// and k = k1 + R1 k2 + R1 R2 k3 (u, k3 < R3; s, k2 < R2; j, k1 < R1):
//   A: per t = u + R3 s: R1 points over j, times W_M3^(t k1);
//   B: per (u, k1): R2 points over s, times W_(R2 R3)^(u k2);
//   C: per q = k1 + R1 k2: R3 points over u, giving X[q + R1 R2 k3].
// The inverse runs C, B, A with conjugate twiddles.  The zero padding (x[n] = 0 for
// n >= n3) and the crop (only n < n3 kept) are half of A's R1 values.  Up to 256 points
// M3 = R1 R2 (R3 = 1 below): A and then, in C's place, R2 points over t for each k1.
//
// A workgroup handles P pencils of consecutive i1 at fixed (component, i2), one
// task of each stage per thread.  A's threads run along z, the contiguous axis of
// x, y and chi; C's run over the pencils first, so that the kz-plane-major
// intermediate U[kz][c][i2][i1] is read and written in runs of P elements straight
// from and to registers.  Between the stages the values pass through LDS, in 8-byte
// elements (FP64: real parts, then imaginary parts; FP32: whole values), with row
// pitches that spread the 32 lanes of an access over the banks (Z3Map).
//
// Bound by memory latency and HBM; 16 values per thread keep FP64 within 128
// registers, four waves per SIMD.  Against the two-stage form it replaces, which held
// 32 values per thread at M3 = 1024 and 64 at 2048 and 4096 (one wave per SIMD in FP64)
// and staged U through LDS a third time, and against the generic LDS passes, the better
// of them for long FP64 pencils, forward + inverse in us: FP64 30 x 12 pencils of 4096
// 131 -> 85, 32 x 32 of 4096 422 -> 227 (floor at the copy rate 64 + 92), of 1024
// 52 -> 45; FP32 67 -> 57, 129 -> 105, 36 -> 31.  Two stages against the generic passes:
// 8 x 8 pencils of 64 15.5 -> 13, 16 x 16 of 128 26 -> 15, 32 x 32 of 256 33 -> 26; FP32
// 32 x 32 of 256 36 -> 22.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "block_maps.hpp"
#include "dft_codelets.hpp"
#include "vie_internal.hpp"

namespace vie {

namespace {

// The lists below give the inverse's radices; the forward pass takes them in reverse where
// that leaves an even first one, so that both run the small radix, with every thread busy,
// on their loads and the large one on their stores (FP64 32 x 32 pencils of 1024, us: forward
// 20.6 as 8, 8, 16 and 25.9 as 16, 8, 8, inverse 27.3 and 25.0).
constexpr bool z3_reverse(int R3) { return R3 != 1 && R3 % 2 == 0; }
constexpr int z3_first(int R1, int R3) { return z3_reverse(R3) ? R3 : R1; }
constexpr int z3_last(int R1, int R3) { return z3_reverse(R3) ? R1 : R3; }

template <typename T> struct Z3Elem { using type = cx<T>; };
template <> struct Z3Elem<double> { using type = double; };

// LDS element of (pencil p, ...): between A and B at row(k1) + t, between B and C at
// u * Qp + q.  Pitches modulo 32 elements: consecutive lanes (u, k1) of B read rows k1
// as one run of R3 k1 + u, and write q = k1 + ... in steps of 32 / R3 per u; pencils
// follow 32 / P apart for the (p, q) lanes of C.
template <int R1, int R2, int R3>
struct Z3Map {
  static constexpr bool two = R3 == 1;   // C: Q tasks of RC points
  static constexpr int M = R1 * R2 * R3, N1 = R2 * R3, TB = R1 * R3, Q = two ? R1 : R1 * R2, RC = two ? R2 : R3;
  static constexpr int TM = N1 > TB ? (N1 > Q ? N1 : Q) : (TB > Q ? TB : Q);   // threads of a pencil
  static constexpr int mod_up(int v, int r) { return v + ((r - v) % 32 + 32) % 32; }   // least >= v, = r mod 32
  static constexpr int N1p = two ? N1 | 1 : mod_up(N1, R3), Qp = mod_up(Q, (32 + R3 / 2) / R3);
  static constexpr int S = two || R1 * N1p > R3 * Qp ? R1 * N1p : R3 * Qp;
  __host__ __device__ static constexpr int pencil(int P) { return two ? mod_up(S, R2 % 32) : mod_up(S, 32 / P); }
};

// v[k] of this thread to slot wa(k), k < NW; then w[j] from slot ra(j), j < NR.  S is
// free on entry; the caller synchronises before reusing it.
template <int NW, int NR, typename WA, typename RA>
__device__ __forceinline__ void z3_exchange(const double2* v, double2* w, double* S, bool won, bool ron, WA wa,
                                            RA ra) {
  if (won) {
#pragma unroll
    for (int k = 0; k < NW; ++k) S[wa(k)] = v[k].x;
  }
  __syncthreads();
  if (ron) {
#pragma unroll
    for (int j = 0; j < NR; ++j) w[j].x = S[ra(j)];
  }
  __syncthreads();
  if (won) {
#pragma unroll
    for (int k = 0; k < NW; ++k) S[wa(k)] = v[k].y;
  }
  __syncthreads();
  if (ron) {
#pragma unroll
    for (int j = 0; j < NR; ++j) w[j].y = S[ra(j)];
  }
}
template <int NW, int NR, typename WA, typename RA>
__device__ __forceinline__ void z3_exchange(const float2* v, float2* w, float2* S, bool won, bool ron, WA wa, RA ra) {
  if (won) {
#pragma unroll
    for (int k = 0; k < NW; ++k) S[wa(k)] = v[k];
  }
  __syncthreads();
  if (ron) {
#pragma unroll
    for (int j = 0; j < NR; ++j) w[j] = S[ra(j)];
  }
}

// Forward stages from A's inputs v[0, R1) (LINE: all of them, else the lower half) of
// the tasks (p, t) to C's outputs z[k3] of the tasks (p3, q).  tw: the plan's tables,
// W_M3 in natural order, then for the forward radices W_M3^(t k1) at M3 + N1 k1 + t and
// W_(R2 R3)^(u k2) at 2 M3 + R3 k2 + u, then the same for the inverse's.
template <typename T, int R1, int R2, int R3, bool LINE>
__device__ __forceinline__ void z3_forward(cx<T>* v, cx<T>* z, int np, int P, gptr<const cx<T>> tw,
                                           typename Z3Elem<T>::type* S, int tid) {
  using L = Z3Map<R1, R2, R3>;
  const int PS = L::pencil(P);
  const int pa = tid / L::N1, t = tid % L::N1;
  if (pa < np) {
    if constexpr (LINE) dft_codelet<T, false, R1>(v);
    else dft_half<T, R1>(v);
#pragma unroll
    for (int k = 1; k < R1; ++k) v[k] = cmul(v[k], tw[L::M + k * L::N1 + t]);
  }
  const int pc = tid & (P - 1), q = tid >> (31 - __clz(P));
  const bool on = pc < np && q < L::Q;
  if constexpr (L::two) {
    z3_exchange<R1, R2>(
        v, z, S, pa < np, on, [&](int k) { return pa * PS + k * L::N1p + t; },
        [&](int j) { return pc * PS + q * L::N1p + j; });
    if (on) dft_codelet<T, false, R2>(z);
  } else {
    const int pb = tid / L::TB, rb = tid % L::TB, u = rb % R3, k1 = rb / R3;
    cx<T> w[R2];
    z3_exchange<R1, R2>(
        v, w, S, pa < np, pb < np, [&](int k) { return pa * PS + k * L::N1p + t; },
        [&](int s) { return pb * PS + k1 * L::N1p + u + R3 * s; });
    if (pb < np) {
      dft_codelet<T, false, R2>(w);
#pragma unroll
      for (int k = 1; k < R2; ++k) w[k] = cmul(w[k], tw[2 * L::M + k * R3 + u]);
    }
    __syncthreads();
    z3_exchange<R2, R3>(
        w, z, S, pb < np, on, [&](int k) { return pb * PS + u * L::Qp + k1 + R1 * k; },
        [&](int j) { return pc * PS + j * L::Qp + q; });
    if (on) dft_codelet<T, false, R3>(z);
  }
}

template <typename T, int R1, int R2, int R3>
__device__ __forceinline__ void zfwd3_body(gptr<const cx<T>> __restrict__ x, gptr<cx<T>> __restrict__ U,
                                           const Geom& g, int P, gptr<const cx<T>> __restrict__ tw, int blk,
                                           typename Z3Elem<T>::type* S, int tid) {
  using L = Z3Map<R1, R2, R3>;
  const PencilBlock pb = pencil_block(blk, g.n1, g.n2, P);
  const int i2 = pb.i2, c = pb.c, i1_0 = pb.i1_0, np = pb.np;
  cx<T> v[R1];
  {
    const int p = tid / L::N1, t = tid % L::N1;
    if (p < np) {
      gptr<const cx<T>> src = x + (((long)c * g.n1 + i1_0 + p) * g.n2 + i2) * g.n3;
#pragma unroll
      for (int j = 0; j < R1 / 2; ++j) {   // n >= M3 / 2 >= n3 is padding
        const int n = t + L::N1 * j;
        const cx<T> in = src[n < g.n3 ? n : g.n3 - 1];
        v[j] = cx<T>{n < g.n3 ? in.x : (T)0, n < g.n3 ? in.y : (T)0};
      }
    }
  }
  cx<T> z[L::RC];
  z3_forward<T, R1, R2, R3, false>(v, z, np, P, tw, S, tid);
  const int p = tid & (P - 1), q = tid >> (31 - __clz(P));
  if (p < np && q < L::Q) {
    const long plane = 3L * g.n1 * g.n2;
    gptr<cx<T>> dst = U + ((long)c * g.n2 + i2) * g.n1 + i1_0 + p;
#pragma unroll
    for (int k = 0; k < L::RC; ++k) dst[(long)(q + L::Q * k) * plane] = z[k];
  }
}

template <typename T, int R1, int R2, int R3, int MODE>
__device__ __forceinline__ void zinv3_body(gptr<const cx<T>> __restrict__ U, gptr<const cx<T>> __restrict__ x,
                                           gptr<cx<T>> __restrict__ y, gptr<const cx<T>> __restrict__ bvec,
                                           gptr<const cx<T>> __restrict__ chi, const Geom& g, int P,
                                           gptr<const cx<T>> __restrict__ tw, int blk,
                                           typename Z3Elem<T>::type* S, int tid) {
  using L = Z3Map<R1, R2, R3>;
  const int PS = L::pencil(P);
  tw += L::M + R2 * z3_last(R1, R3);   // past the forward tables
  const PencilBlock pk = pencil_block(blk, g.n1, g.n2, P);
  const int i2 = pk.i2, c = pk.c, i1_0 = pk.i1_0, np = pk.np;
  const int pc = tid & (P - 1), q = tid >> (31 - __clz(P));
  const bool on = pc < np && q < L::Q;
  cx<T> z[L::RC];
  if (on) {
    const long plane = 3L * g.n1 * g.n2;
    gptr<const cx<T>> src = U + ((long)c * g.n2 + i2) * g.n1 + i1_0 + pc;
#pragma unroll
    for (int k = 0; k < L::RC; ++k) z[k] = src[(long)(q + L::Q * k) * plane];
    dft_codelet<T, true, L::RC>(z);
    const int row = L::two ? L::M + q * R2 : 2 * L::M + q / R1 * R3;
#pragma unroll
    for (int j = 1; j < L::RC; ++j) z[j] = cmulc(z[j], tw[row + j]);
  }
  const int pa = tid / L::N1, t = tid % L::N1;
  cx<T> v[R1];
  if constexpr (L::two) {
    z3_exchange<R2, R1>(
        z, v, S, on, pa < np, [&](int j) { return pc * PS + q * L::N1p + j; },
        [&](int k) { return pa * PS + k * L::N1p + t; });
  } else {
    const int pb = tid / L::TB, rb = tid % L::TB, u = rb % R3, k1 = rb / R3;
    cx<T> w[R2];
    z3_exchange<R3, R2>(
        z, w, S, on, pb < np, [&](int j) { return pc * PS + j * L::Qp + q; },
        [&](int k) { return pb * PS + u * L::Qp + k1 + R1 * k; });
    if (pb < np) {
      dft_codelet<T, true, R2>(w);
#pragma unroll
      for (int s = 0; s < R2; ++s) w[s] = cmulc(w[s], tw[L::M + k1 * L::N1 + u + R3 * s]);
    }
    __syncthreads();
    z3_exchange<R2, R1>(
        w, v, S, pb < np, pa < np, [&](int s) { return pb * PS + k1 * L::N1p + u + R3 * s; },
        [&](int k) { return pa * PS + k * L::N1p + t; });
  }
  if (pa < np) {
    dft_codelet<T, true, R1>(v);
    // the kept outputs, in registers here (else their arithmetic sinks into the conditional
    // stores with the transform's intermediates live across all of them)
#pragma unroll
    for (int j = 0; j < R1 / 2; ++j) asm volatile("" : "+v"(v[j].x), "+v"(v[j].y));
    const long vox = ((long)(i1_0 + pa) * g.n2 + i2) * g.n3;
    const long off = (long)c * g.N + vox;
#pragma unroll
    for (int j = 0; j < R1 / 2; ++j) {   // n >= M3 / 2 >= n3 is cropped
      const int n = t + L::N1 * j, m = n < g.n3 ? n : g.n3 - 1;
      cx<T> r = csub(x[off + m], cmul(chi[vox + m], v[j]));
      if (MODE == 1) r = csub(bvec[off + m], r);
      if (n < g.n3) y[off + n] = r;
    }
  }
}

template <typename T, int R1, int R2, int R3>
__global__ __launch_bounds__(1024) void k_zfwd3(const cx<T>* __restrict__ x, cx<T>* __restrict__ U, Geom g, int P,
                                                const cx<T>* __restrict__ tw) {
  extern __shared__ unsigned char smem_raw[];
  zfwd3_body<T, R1, R2, R3>((gptr<const cx<T>>)x, (gptr<cx<T>>)U, g, P, (gptr<const cx<T>>)tw,
                            xcd_group(blockIdx.x, gridDim.x, P, (int)sizeof(cx<T>)),
                            reinterpret_cast<typename Z3Elem<T>::type*>(smem_raw), threadIdx.x);
}

template <typename T, int R1, int R2, int R3, int MODE>
__global__ __launch_bounds__(1024) void k_zinv3(const cx<T>* __restrict__ U, const cx<T>* __restrict__ x,
                                                cx<T>* __restrict__ y, const cx<T>* __restrict__ bvec,
                                                const cx<T>* __restrict__ chi, Geom g, int P,
                                                const cx<T>* __restrict__ tw) {
  extern __shared__ unsigned char smem_raw[];
  zinv3_body<T, R1, R2, R3, MODE>((gptr<const cx<T>>)U, (gptr<const cx<T>>)x, (gptr<cx<T>>)y, (gptr<const cx<T>>)bvec,
                                  (gptr<const cx<T>>)chi, g, P, (gptr<const cx<T>>)tw,
                                  xcd_group(blockIdx.x, gridDim.x, P, (int)sizeof(cx<T>)),
                                  reinterpret_cast<typename Z3Elem<T>::type*>(smem_raw), threadIdx.x);
}

// In-place transforms of contiguous lines of M3 values, one workgroup each (the spectra
// of the tables at plan time).
template <int R1, int R2, int R3>
__global__ __launch_bounds__(1024) void k_z3_lines(double2* __restrict__ F, const double2* __restrict__ tw) {
  extern __shared__ unsigned char smem_raw[];
  using L = Z3Map<R1, R2, R3>;
  double2* line = F + (long)blockIdx.x * L::M;
  const int tid = threadIdx.x;
  double2 v[R1], z[L::RC];
  if (tid < L::N1) {
#pragma unroll
    for (int j = 0; j < R1; ++j) v[j] = line[tid + L::N1 * j];
  }
  z3_forward<double, R1, R2, R3, true>(v, z, 1, 1, (gptr<const double2>)tw, reinterpret_cast<double*>(smem_raw), tid);
  if (tid < L::Q) {
#pragma unroll
    for (int k = 0; k < L::RC; ++k) line[tid + L::Q * k] = z[k];
  }
}

__device__ __forceinline__ int find_sys(const int* prefix, int nsys, int item) {
  int lo = 0, hi = nsys - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= item) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Persistent batched z passes: each workgroup walks the (system, pencil block)
// items of the batch with a grid stride.
template <typename T, int R1, int R2, int R3>
__global__ __launch_bounds__(1024) void k_zfwd3_batch(const PassDesc* __restrict__ d, const int* __restrict__ prefix,
                                                      int nsys, int total, int jx, int jy) {
  extern __shared__ unsigned char smem_raw[];
  auto* S = reinterpret_cast<typename Z3Elem<T>::type*>(smem_raw);
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int s = find_sys(prefix, nsys, item);
    const PassDesc& D = d[s];
    if (D.active && *D.active == 0) continue;
    zfwd3_body<T, R1, R2, R3>((gptr<const cx<T>>)(const cx<T>*)D.xb + (long)jx * D.xs, (gptr<cx<T>>)(cx<T>*)D.U, D.g,
                              D.P, (gptr<const cx<T>>)(const cx<T>*)D.twz, item - prefix[s], S, opaque_tid());
    __syncthreads();
  }
}

template <typename T, int R1, int R2, int R3, int MODE>
__global__ __launch_bounds__(1024) void k_zinv3_batch(const PassDesc* __restrict__ d, const int* __restrict__ prefix,
                                                      int nsys, int total, int jx, int jy) {
  extern __shared__ unsigned char smem_raw[];
  auto* S = reinterpret_cast<typename Z3Elem<T>::type*>(smem_raw);
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int s = find_sys(prefix, nsys, item);
    const PassDesc& D = d[s];
    if (D.active && *D.active == 0) continue;
    zinv3_body<T, R1, R2, R3, MODE>(
        (gptr<const cx<T>>)(const cx<T>*)D.U, (gptr<const cx<T>>)(const cx<T>*)D.xb + (long)jx * D.xs,
        (gptr<cx<T>>)(cx<T>*)D.yb + (long)jy * D.ys, (gptr<const cx<T>>)(const cx<T>*)D.b,
        (gptr<const cx<T>>)(const cx<T>*)D.chi, D.g, D.P, (gptr<const cx<T>>)(const cx<T>*)D.twz, item - prefix[s], S,
        opaque_tid());
    __syncthreads();
  }
}

// Every length with the inverse's radices: the first even (half of its inputs are padding), all near each
// other (a pencil has as many threads as its stage of smallest radix has tasks), the length a
// multiple of 16, which the plane order of the cross-section passes wants.  Each is at most 1.25
// times the one before but for 128 after 96 (16 x 7 would need a radix of 7) and 512 after 256
// (two radices of up to 16 end there, three of 8 and more begin at 512).
#define VIE_Z3_LENGTHS(X) \
  X(8, 8, 1)              \
  X(10, 8, 1)             \
  X(12, 8, 1)             \
  X(16, 8, 1)             \
  X(12, 12, 1)            \
  X(16, 10, 1)            \
  X(16, 12, 1)            \
  X(16, 15, 1)            \
  X(16, 16, 1)            \
  X(8, 8, 8)              \
  X(8, 8, 10)             \
  X(8, 8, 12)             \
  X(10, 10, 8)            \
  X(12, 10, 8)            \
  X(16, 8, 8)             \
  X(12, 12, 8)            \
  X(16, 10, 8)            \
  X(12, 12, 10)           \
  X(16, 10, 10)           \
  X(16, 12, 10)           \
  X(16, 16, 8)            \
  X(16, 12, 12)           \
  X(16, 16, 10)           \
  X(16, 15, 12)           \
  X(16, 16, 12)           \
  X(16, 15, 15)           \
  X(16, 16, 16)

struct Z3Shape {
  int threads;   // of a pencil
  int pencil;    // LDS elements of a pencil of P
};
bool z3_shape(int M3, int P, Z3Shape* s) {
#define VIE_Z3(A, B, C)                                                    \
  if (M3 == A * B * C) {                                                   \
    using F = Z3Map<z3_first(A, C), B, z3_last(A, C)>;                      \
    *s = {F::TM, std::max(F::pencil(P), Z3Map<A, B, C>::pencil(P))};        \
    return true;                                                           \
  }
  VIE_Z3_LENGTHS(VIE_Z3)
#undef VIE_Z3
  return false;
}
int z3_threads(int M3, int P) {
  Z3Shape s;
  return z3_shape(M3, P, &s) ? (P * s.threads + 63) / 64 * 64 : 0;
}

}  // namespace

bool z3_radices(int M3, int r[3], bool inverse) {
#define VIE_Z3(A, B, C)                     \
  if (M3 == A * B * C) {                    \
    r[0] = inverse ? A : z3_first(A, C);    \
    r[1] = B;                               \
    r[2] = inverse ? C : z3_last(A, C);     \
    return true;                            \
  }
  VIE_Z3_LENGTHS(VIE_Z3)
#undef VIE_Z3
  return false;
}

int z3_length(int need) {
  int m = 0;
#define VIE_Z3(A, B, C) \
  if (A * B * C >= need && (m == 0 || A * B * C < m)) m = A * B * C;
  VIE_Z3_LENGTHS(VIE_Z3)
#undef VIE_Z3
  return m;
}

// Pencil counts P tried by the plan-time tuner, default first, by the power of two the
// length belongs to; each keeps the workgroup within 1024 threads and its LDS within
// 160 KiB.  None below 512 points, where P is the power of two that holds a row of pencils,
// up to 128 bytes of the intermediate (z3_pencils): a workgroup has few waves anyway.
template <typename T>
int z3_pencil_options(int M3, int* out, int cap) {
  const bool dbl = sizeof(T) == 8;
  int r[3];
  if (M3 < 512 || !z3_radices(M3, r)) return 0;
  int opts[6] = {0, 0, 0, 0, 0, 0}, n = 0;
  if (M3 <= 512) {
    if (dbl) { opts[0] = 8; opts[1] = 4; opts[2] = 16; opts[3] = 2; n = 4; }
    else { opts[0] = 16; opts[1] = 8; opts[2] = 4; opts[3] = 2; n = 4; }
  } else if (M3 <= 1024) {
    if (dbl) { opts[0] = 4; opts[1] = 2; opts[2] = 8; n = 3; }
    else { opts[0] = 8; opts[1] = 4; opts[2] = 2; n = 3; }
  } else if (M3 <= 2048) {
    if (dbl) { opts[0] = 2; opts[1] = 4; opts[2] = 1; n = 3; }
    else { opts[0] = 4; opts[1] = 2; n = 2; }
  } else {
    if (dbl) { opts[0] = 2; opts[1] = 1; n = 2; }
    else { opts[0] = 2; opts[1] = 4; opts[2] = 1; n = 3; }
  }
  for (int i = 0; i < n && i < cap; ++i) out[i] = opts[i];
  return n;
}

template <typename T>
int z3_pencils(int M3, int n1) {
  int opts[8];
  if (z3_pencil_options<T>(M3, opts, 8)) return opts[0];
  int P = 1;
  while (P < n1 && P < (sizeof(T) == 8 ? 8 : 16)) P *= 2;
  return P;
}

size_t z3_lds_bytes(int M3, int P) {
  Z3Shape s;
  return z3_shape(M3, P, &s) ? (size_t)P * s.pencil * 8 : 0;
}

template <typename T>
hipError_t launch_z3(int which, const Geom& g, int P, const void* x, void* y, const void* b, int mode, void* U,
                     const void* chi, const void* twz, hipStream_t st) {
  using C = cx<T>;
  if (P == 0) P = z3_pencils<T>(g.M3, g.n1);
  if (P < 1 || P > 16 || (P & (P - 1)) || z3_threads(g.M3, P) > 1024) return hipErrorNotSupported;
  const dim3 grid(pencil_blocks(g.n1, g.n2, P)), block(z3_threads(g.M3, P));
  const size_t lds = z3_lds_bytes(g.M3, P);
#define VIE_Z3(A, B, D)                                                                                        \
  if (g.M3 == A * B * D) {                                                                                     \
    if (which == 0)                                                                                            \
      hipLaunchKernelGGL((k_zfwd3<T, z3_first(A, D), B, z3_last(A, D)>), grid, block, lds, st, (const C*)x, (C*)U,    \
                         g, P, (const C*)twz);                                                                   \
    else if (mode == 0)                                                                                        \
      hipLaunchKernelGGL((k_zinv3<T, A, B, D, 0>), grid, block, lds, st, (const C*)U, (const C*)x, (C*)y,        \
                         (const C*)nullptr, (const C*)chi, g, P, (const C*)twz);                                \
    else                                                                                                       \
      hipLaunchKernelGGL((k_zinv3<T, A, B, D, 1>), grid, block, lds, st, (const C*)U, (const C*)x, (C*)y,        \
                         (const C*)b, (const C*)chi, g, P, (const C*)twz);                                      \
    return hipGetLastError();                                                                                  \
  }
  VIE_Z3_LENGTHS(VIE_Z3)
#undef VIE_Z3
  return hipErrorNotSupported;
}

hipError_t launch_z3_lines(int M3, long lines, double2* F, const double2* twz, hipStream_t st) {
  const size_t lds = z3_lds_bytes(M3, 1);
#define VIE_Z3(A, B, D)                                                                                       \
  if (M3 == A * B * D) {                                                                                      \
    hipLaunchKernelGGL((k_z3_lines<z3_first(A, D), B, z3_last(A, D)>), dim3((unsigned)lines),                  \
                       dim3(z3_threads(M3, 1)), lds, st, F, twz);                                             \
    return hipGetLastError();                                                                                 \
  }
  VIE_Z3_LENGTHS(VIE_Z3)
#undef VIE_Z3
  return hipErrorNotSupported;
}

template <typename T>
hipError_t launch_z3_batch(int which, int mode, const PassDesc* d, const int* prefix, int nsys, int total, int M3,
                           int P, int jx, int jy, hipStream_t st) {
  const size_t lds = z3_lds_bytes(M3, P);
  const dim3 grid(total < 4096 ? total : 4096), block(z3_threads(M3, P));
#define VIE_Z3(A, B, D)                                                                                          \
  if (M3 == A * B * D) {                                                                                         \
    if (which == 0)                                                                                              \
      hipLaunchKernelGGL((k_zfwd3_batch<T, z3_first(A, D), B, z3_last(A, D)>), grid, block, lds, st, d, prefix,   \
                         nsys, total, jx, jy);                                                                   \
    else if (mode == 0)                                                                                          \
      hipLaunchKernelGGL((k_zinv3_batch<T, A, B, D, 0>), grid, block, lds, st, d, prefix, nsys, total, jx, jy);    \
    else                                                                                                         \
      hipLaunchKernelGGL((k_zinv3_batch<T, A, B, D, 1>), grid, block, lds, st, d, prefix, nsys, total, jx, jy);    \
    return hipGetLastError();                                                                                    \
  }
  VIE_Z3_LENGTHS(VIE_Z3)
#undef VIE_Z3
  return hipErrorNotSupported;
}

// large LDS for the passes of length M3
template <typename T>
hipError_t allow_lds_z3(int M3) {
  const int big = 160 * 1024;
  hipError_t e = hipSuccess;
  auto allow = [&](const void* k) {
    if (!e) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, big);
  };
#define VIE_Z3(A, B, D)                              \
  if (M3 == A * B * D) {                             \
    allow((const void*)k_zfwd3<T, z3_first(A, D), B, z3_last(A, D)>);       \
    allow((const void*)k_zinv3<T, A, B, D, 0>);       \
    allow((const void*)k_zinv3<T, A, B, D, 1>);       \
    allow((const void*)k_zfwd3_batch<T, z3_first(A, D), B, z3_last(A, D)>); \
    allow((const void*)k_zinv3_batch<T, A, B, D, 0>); \
    allow((const void*)k_zinv3_batch<T, A, B, D, 1>); \
  }
  VIE_Z3_LENGTHS(VIE_Z3)
#undef VIE_Z3
  return e;
}

template hipError_t launch_z3<double>(int, const Geom&, int, const void*, void*, const void*, int, void*,
                                      const void*, const void*, hipStream_t);
template hipError_t launch_z3<float>(int, const Geom&, int, const void*, void*, const void*, int, void*,
                                     const void*, const void*, hipStream_t);
template int z3_pencil_options<double>(int, int*, int);
template int z3_pencil_options<float>(int, int*, int);
template int z3_pencils<double>(int, int);
template int z3_pencils<float>(int, int);
template hipError_t allow_lds_z3<double>(int);
template hipError_t allow_lds_z3<float>(int);
template hipError_t launch_z3_batch<double>(int, int, const PassDesc*, const int*, int, int, int, int, int, int,
                                            hipStream_t);
template hipError_t launch_z3_batch<float>(int, int, const PassDesc*, const int*, int, int, int, int, int, int,
                                           hipStream_t);

}  // namespace vie
