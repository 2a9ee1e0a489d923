// Learned preconditioner: a 4-level 3-D U-Net (channels 16/32/48/64, 3x3x3
// convolutions, bias-free ReLU) that maps a normalised residual r (and the
// contrast chi) to the correction A^{-1} r - r; the preconditioner is
// z = r + net(r).  It is used as the right
// preconditioner of flexible GMRES and as an initial guess, with plain GMRES as
// the fallback.  This part is this library's addition, not the paper's method.
//
// Activations are channels-last bfloat16 [V][C] (V = D H W voxels, W fastest,
// C a multiple of 16, channel stride / offset per view so concatenations are
// written in place).  Convolutions are implicit GEMMs on the matrix cores:
// v_mfma_f32_16x16x32_bf16, FP32 accumulation.  Forward: output channels x voxels,
// K = 27 Cin; a tile's input with its halo and the weights of 16 input channels are
// staged in LDS and read as fragments (k_conv2).  Input
// gradient: the same kernel with taps flipped and channels swapped, the ReLU
// mask of the forward input fused into the epilogue.  Weight gradient: a GEMM over
// voxels with every tap in registers, split over voxel tiles with a fixed-order
// reduction (k_wgrad).  Master weights, gradients and
// Adam moments are FP32.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "../../include/vie.h"
#include "krylov.hpp"
#include "vie_internal.hpp"

namespace vie {

typedef unsigned short bf16_t;
typedef short s4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef unsigned int u4v __attribute__((ext_vector_type(4)));
typedef unsigned int u2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16_t f2bf(float f) {   // round to nearest, ties to even
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float(((unsigned)h) << 16); }

// B volumes of D x H x W voxels one after the other (B > 1: the samples of a training group).
// Levels that are pooled or upsampled have even D, so those passes take the stack as one
// volume; the convolutions keep their halos inside a sample.
struct Vol {
  int D, H, W, B = 1;
  __host__ __device__ long V() const { return (long)D * H * W; }
  __host__ __device__ long all() const { return B * V(); }
  Vol stack() const { return Vol{B * D, H, W}; }
};

// ------------------------------------------------------------------ convolution
// Y[v, o] = act(sum_t sum_i W[t][o][i] X[v + t][i]); tap t = (dz+1)*9 + (dy+1)*3 + (dx+1).
// LDS-staged implicit GEMM on v_mfma_f32_16x16x32_bf16.  A workgroup of four waves
// computes a tile of TZ (D) x 4 (H) x 16 MT (W) output voxels for up to 64 output
// channels (grid.y picks the group of NT 16-channel N-tiles).  Wave w takes the
// TZ rows (z0 + (TZ == 2 ? w / 2 : 0), y0 + ...) assigned to it, i.e. TZ * MT / ...
// 16-voxel M-tiles: with TZ = 2, MT = 2 (the 2 x 4 x 32 tile of the large levels)
// four M-tiles per wave; with TZ = 1, MT = 1 (the 1 x 4 x 16 tile that keeps the
// small levels' launches wide) one.  The input is consumed in chunks of 16
// channels: the chunk's halo tile and its weights for all taps and the group's
// output channels are staged in LDS once and read by every K-step.  One MFMA
// K-step covers two taps of the chunk (K = 2 x 16): lanes 0-31 take tap t, lanes
// 32-63 tap t + 1 (the 28th tap is zero).  Halo layout [half][voxel][8 channels]
// (half = channels 0-7 or 8-15), so the 16 lanes of one fragment row read 256
// contiguous bytes; weight layout [tap pair][N-tile][lane] of 16-byte B fragments,
// so a wave reads 1 KiB contiguous.
constexpr int kCty = 4;                                  // output tile height (H)
constexpr int kPairs = 14;                               // tap pairs of a 3 x 3 x 3 kernel
template <int TZ, int MT> struct ConvTile {
  static constexpr int tx = 16 * MT, ty = kCty, tz = TZ;
  static constexpr int hx = tx + 2, hy = ty + 2, hz = tz + 2;
  static constexpr int hvox = hx * hy * hz;
  static constexpr int rows = TZ;                        // rows (z, y pairs) per wave: TZ
};

// dynamic LDS bytes of k_conv2 for nt N-tiles
template <int TZ, int MT>
static inline size_t conv2_lds(int taps, int nt) {
  return (size_t)2 * ConvTile<TZ, MT>::hvox * 8 * 2 + (size_t)(taps == 1 ? 1 : kPairs) * nt * 64 * 16;
}

// Inference folds its neighbours into the convolutions (each was a launch of 5 to 8 us of a
// 215 us apply at 32 x 32 x 256, 192 so): the first `chunks` 16-channel chunks of
// the input read their parents in a volume of half the size (nearest upsampling), and the
// last layer's output goes straight into the result.
struct ConvUp {
  const bf16_t* X = nullptr;
  int cs = 0, chunks = 0;
};
// z_c = base_c + (out[2c] + i out[2c + 1]) / s, s = sqrt(3 N / sumsq): the network predicts the
// correction A^{-1} r - base, so an untrained (small) network leaves the base preconditioner
// (or the identity)
struct NetOut {
  const double2* base = nullptr;
  const double2* sumsq = nullptr;
  double2* z = nullptr;
};

template <int TAPS, int NT, int TZ, int MT>
__global__ __launch_bounds__(256) void k_conv2(const bf16_t* __restrict__ X, int xcs, int xco, int Cin,
                                               const bf16_t* __restrict__ Wt, int Cout, bf16_t* __restrict__ Y,
                                               int ycs, int yco, float* __restrict__ Yf, Vol vol, int relu,
                                               const bf16_t* __restrict__ mask, int mcs, int mco, int n0,
                                               ConvUp up, NetOut res) {
  using Tl = ConvTile<TZ, MT>;
  constexpr int kHx = Tl::hx, kHy = Tl::hy, kHvox = Tl::hvox;
  constexpr int MI = TZ * MT;                  // M-tiles per wave
  extern __shared__ __attribute__((aligned(16))) unsigned char conv_smem[];
  bf16_t* tile = reinterpret_cast<bf16_t*>(conv_smem);
  u4v* wfrag = reinterpret_cast<u4v*>(conv_smem + (size_t)2 * kHvox * 8 * 2);
  constexpr int NPAIR = TAPS == 1 ? 1 : kPairs;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ntx = (vol.W + Tl::tx - 1) / Tl::tx, nty = (vol.H + Tl::ty - 1) / Tl::ty;
  int b = blockIdx.x;
  const int tx = b % ntx;
  b /= ntx;
  const int ty = b % nty;
  b /= nty;
  const int ntz = (vol.D + Tl::tz - 1) / Tl::tz;
  const int tz = b % ntz;
  const long v0 = (b / ntz) * vol.V();         // first voxel of the sample
  const int x0 = tx * Tl::tx, y0 = ty * Tl::ty, z0 = tz * Tl::tz;
  X += v0 * xcs;
  const int nt0 = n0 + blockIdx.y * NT;        // first N-tile of this workgroup's group
  const int m = lane & 15, kq = lane >> 4;     // fragment row / K-quarter
  const int half = kq & 1, second = kq >> 1;   // channel half, which tap of the pair
  // wave rows: TZ = 2: (wave / 2, 2 (wave % 2) + {0, 1}); TZ = 1: (0, wave)
  const int wz = TZ == 2 ? wave >> 1 : 0, wy = TZ == 2 ? 2 * (wave & 1) : wave;
  // this lane's halo row for tap offset 0 (the halo corner) of its first M-tile
  const int lds_lane = (half * kHvox + (wz * kHy + wy) * kHx + m) * 8;
  // piece e of the chunk's halo tile: channels 8 (e & 1) .. + 7 of halo voxel e / 2
  auto halo_voxel = [&](int e) {               // -1 outside the volume
    const int hv = e >> 1;
    const int xx = x0 + hv % kHx - 1, yy = y0 + (hv / kHx) % kHy - 1, zz = z0 + hv / (kHx * kHy) - 1;
    const bool in = xx >= 0 && xx < vol.W && yy >= 0 && yy < vol.H && zz >= 0 && zz < vol.D;
    return in ? (zz * vol.H + yy) * vol.W + xx : -1;
  };
  auto halo_parent = [&](int e) {              // the same of the coarse volume
    const int hv = e >> 1;
    const int xx = x0 + hv % kHx - 1, yy = y0 + (hv / kHx) % kHy - 1, zz = z0 + hv / (kHx * kHy) - 1;
    const bool in = xx >= 0 && xx < vol.W && yy >= 0 && yy < vol.H && zz >= 0 && zz < vol.D;
    return in ? ((zz >> 1) * (vol.H / 2) + (yy >> 1)) * (vol.W / 2) + (xx >> 1) : -1;
  };
  // v: the halo voxel, or its parent for an upsampled chunk
  auto halo_load = [&](int e, int v, int ch) {
    const bf16_t* p = ch < up.chunks ? up.X + (long)v * up.cs : X + (long)v * xcs + xco;
    return v >= 0 ? *reinterpret_cast<const u4v*>(p + ch * 16 + (e & 1) * 8) : u4v{0u, 0u, 0u, 0u};
  };
  auto halo_store = [&](int e, u4v v) {
    *reinterpret_cast<u4v*>(tile + ((e & 1) * kHvox + (e >> 1)) * 8) = v;
  };
  // B fragment e = (pair, N-tile, lane) of the chunk: W[tap][co][ci .. ci + 7]
  auto frag_load = [&](int e, int ch) {
    const int l = e & 63, t = (e >> 6) % NT, tp = (e >> 6) / NT;
    const int lm = l & 15, lq = l >> 4;
    const int tap = TAPS == 1 ? 0 : 2 * tp + (lq >> 1);
    u4v val = u4v{0u, 0u, 0u, 0u};
    if (TAPS == 1 ? (lq >> 1) == 0 : tap < 27)
      val = *reinterpret_cast<const u4v*>(Wt + ((long)tap * Cout + (nt0 + t) * 16 + lm) * Cin + ch * 16 + (lq & 1) * 8);
    return val;
  };
  // The next chunk's halo pieces and B fragments wait in registers while this chunk's MFMAs
  // run: a chunk then costs its compute, not its memory latency.  Not for the large tile with
  // one N-tile: its layers have one chunk (48 -> 16: three) and four workgroups per CU to
  // overlap, which the registers would not leave room for (25 us a layer at 32 x 32 x 256).
  constexpr bool kAhead = TZ == 1 || NT > 1;
  constexpr int kHalo = 2 * kHvox, kFrag = NPAIR * NT * 64;
  constexpr int NH = kAhead ? (kHalo + 255) / 256 : 1, NW = kAhead ? (kFrag + 255) / 256 : 1;
  u4v hreg[NH], wreg[NW];
  int hvox[NH], pvox[NH];
  auto load_chunk = [&](int ch) {
#pragma unroll
    for (int q = 0; q < NH; ++q) hreg[q] = halo_load(threadIdx.x, ch < up.chunks ? pvox[q] : hvox[q], ch);
#pragma unroll
    for (int q = 0; q < NW; ++q)
      if ((int)threadIdx.x + 256 * q < kFrag) wreg[q] = frag_load(threadIdx.x + 256 * q, ch);
  };
  f4v acc[MI][NT];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[i][t] = f4v{0.f, 0.f, 0.f, 0.f};
  const int nchunk = Cin / 16;
  if constexpr (kAhead) {
#pragma unroll
    for (int q = 0; q < NH; ++q) {
      const int e = threadIdx.x + 256 * q;
      hvox[q] = e < kHalo ? halo_voxel(e) : -1;
      pvox[q] = up.chunks && e < kHalo ? halo_parent(e) : -1;
    }
    load_chunk(0);
  }
  for (int ch = 0; ch < nchunk; ++ch) {
    __syncthreads();
    if constexpr (kAhead) {
#pragma unroll
      for (int q = 0; q < NH; ++q)
        if ((int)threadIdx.x + 256 * q < kHalo) halo_store(threadIdx.x + 256 * q, hreg[q]);
#pragma unroll
      for (int q = 0; q < NW; ++q)
        if ((int)threadIdx.x + 256 * q < kFrag) wfrag[threadIdx.x + 256 * q] = wreg[q];
    } else {
      if (ch < up.chunks)
        for (int e = threadIdx.x; e < kHalo; e += 256) halo_store(e, halo_load(e, halo_parent(e), ch));
      else
        for (int e = threadIdx.x; e < kHalo; e += 256) halo_store(e, halo_load(e, halo_voxel(e), ch));
      for (int e = threadIdx.x; e < kFrag; e += 256) wfrag[e] = frag_load(e, ch);
    }
    __syncthreads();
    if (kAhead && ch + 1 < nchunk) load_chunk(ch + 1);
#pragma unroll
    for (int tp = 0; tp < NPAIR; ++tp) {
      constexpr int kStep = kHx * kHy;
      const int t0 = 2 * tp, t1 = 2 * tp + 1;
      const int off0 = TAPS == 1 ? kStep + kHx + 1 : (t0 / 9) * kStep + ((t0 / 3) % 3) * kHx + t0 % 3;
      // the 28th tap (t1 = 27) does not exist: it reads tap t0's (finite) halo values,
      // and its B fragment is zero
      const int off1 = (TAPS == 1 || t1 >= 27) ? off0 : (t1 / 9) * kStep + ((t1 / 3) % 3) * kHx + t1 % 3;
      const int off = second ? off1 : off0;
      bf8v bfr[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) bfr[t] = __builtin_bit_cast(bf8v, wfrag[(tp * NT + t) * 64 + lane]);
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        // M-tile i: row (i / MT) of the wave, voxels 16 (i % MT) .. + 15
        const int ao = lds_lane + (off + (i / MT) * kHx + 16 * (i % MT)) * 8;
        const bf8v a = __builtin_bit_cast(bf8v, *reinterpret_cast<const u4v*>(tile + ao));
        // weights as the first operand: a lane then holds four consecutive output
        // channels of one voxel, stored as one 8-byte (FP32: 16-byte) value
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[t], a, acc[i][t], 0, 0, 0);
      }
    }
  }
  // D[row = 4 kq + r][col = m]: channel 4 kq + r, voxel 16 (i % MT) + m of wave row i / MT
  const int zz = z0 + wz;
  if (zz >= vol.D) return;
  const long N = vol.V();
  double is = 0.0;
  if (res.z) {
    const double s = res.sumsq->x > 0 ? sqrt(3.0 * (double)N / res.sumsq->x) : 0.0;
    is = s > 0 ? 1.0 / s : 0.0;
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int yy = y0 + wy + i / MT, xx = x0 + 16 * (i % MT) + m;
    if (yy >= vol.H || xx >= vol.W) continue;
    const long vo = v0 + ((long)zz * vol.H + yy) * vol.W + xx;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int n = (nt0 + t) * 16 + 4 * kq;
      f4v val = acc[i][t];
      if (relu)
#pragma unroll
        for (int r = 0; r < 4; ++r) val[r] = fmaxf(val[r], 0.f);
      if (mask) {
        const u2v mk = *reinterpret_cast<const u2v*>(mask + vo * mcs + mco + n);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          val[r] = __uint_as_float(r & 1 ? mk[r / 2] & 0xFFFF0000u : mk[r / 2] << 16) > 0.f ? val[r] : 0.f;
      }
      if (Y) {
        u2v o;
#pragma unroll
        for (int r = 0; r < 2; ++r) o[r] = (unsigned)f2bf(val[2 * r]) | ((unsigned)f2bf(val[2 * r + 1]) << 16);
        *reinterpret_cast<u2v*>(Y + vo * ycs + yco + n) = o;
      }
      if (Yf) *reinterpret_cast<f4v*>(Yf + vo * Cout + n) = val;
      if (res.z)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int c = n / 2 + h;   // component of channels n + 2 h, n + 2 h + 1
          if (c < 3) {
            const double2 rv = res.base[c * N + vo];
            res.z[c * N + vo] = double2{rv.x + val[2 * h] * is, rv.y + val[2 * h + 1] * is};
          }
        }
    }
  }
}

// partial[blk][tap][o][i] = sum over the block's voxels v of dY[v, o] X[v + tap, i]
//
// An implicit GEMM with K = voxels: M = 16 output channels, N = 16 input channels, one
// accumulator per tap, so a wave keeps all 27 taps of one (o, i) tile pair in registers
// (108 values per lane) and every dY fragment serves 27 MFMAs.  A workgroup takes one
// 16-channel chunk of X and NO output tiles; it stages a 2 x 4 x TX voxel tile of dY and
// the tile's X halo (4 x 6 x (TX + 2) voxels) in LDS, channels last, and walks tiles with a
// grid stride.  A K-step is 32 voxels; both operands need voxels along the lane's registers
// while memory holds channels there, so fragments come from the transposing LDS read
// (ds_read_b64_tr_b16: the 16 lanes of a group address four rows of 16 channels, lane c gets
// channel c of the four rows).  A tap is then a row offset, with no unaligned access.  With
// NO < 4 the waves split the K-steps and add their accumulators through LDS at the end.
// Voxels outside the volume are staged as zeros in both tiles.
// Bound: LDS reads (56 of 8 bytes a lane per 27 MFMAs), at a fraction of the matrix rate;
// the element-by-element loads of the earlier kernel (two bytes a lane, nothing reused
// between taps) took 422 us a layer at 32 x 32 x 128 on average; a training step on two
// samples of 32 x 32 x 128 went from 14.3 to 3.5 ms.
template <int TAPS, int NO, int TX>
struct WgradTile {
  static constexpr int waves = NO == 3 ? 3 : 4;
  static constexpr int ks = waves / NO;                  // waves sharing an output tile
  static constexpr int hx = TX + 2, hvox = 4 * 6 * hx, vox = 2 * 4 * TX;
  static constexpr int stage = (hvox + NO * vox) * 16 * 2;
  static constexpr int red = ks > 1 ? NO * TAPS * 256 * 4 : 0;
  static constexpr int bytes = stage > red ? stage : red;
};

typedef __attribute__((address_space(3))) s4v* lds_s4v;
__device__ __forceinline__ bf8v read_rows8(bf16_t* p) {   // rows 0-3 and 4-7 of 16 channels
  const s4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v)p);
  const s4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v)(p + 64));
  return __builtin_bit_cast(bf8v, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int TAPS, int NO, int TX>
__global__ __launch_bounds__((64 * WgradTile<TAPS, NO, TX>::waves)) void k_wgrad(
    const bf16_t* __restrict__ X, int xcs, int xco, int Cin, const bf16_t* __restrict__ dY, int ycs, int yco, int Cout,
    float* __restrict__ partial, Vol vol, int o0) {
  using Tl = WgradTile<TAPS, NO, TX>;
  __shared__ __attribute__((aligned(16))) unsigned char smem[Tl::bytes];
  bf16_t* xt = reinterpret_cast<bf16_t*>(smem);           // [halo voxel][16]
  bf16_t* yt = xt + Tl::hvox * 16;                        // [output tile][voxel][16]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m = lane & 15, kq = lane >> 4;
  const int ot = wave % NO, part = wave / NO;
  const int rowoff = (m >> 2) * 16 + (m & 3) * 4;         // this lane's share of a transposing read
  const int ntx = (vol.W + TX - 1) / TX, nty = (vol.H + 3) / 4, ntz = (vol.D + 1) / 2;
  const int ntiles = ntx * nty * ntz * vol.B;
  const int ci = blockIdx.y * 16;
  f4v acc[TAPS];
#pragma unroll
  for (int t = 0; t < TAPS; ++t) acc[t] = f4v{0.f, 0.f, 0.f, 0.f};
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int x0 = (tile % ntx) * TX, y0 = ((tile / ntx) % nty) * 4, z0 = (tile / (ntx * nty)) % ntz * 2;
    const long v0 = tile / (ntx * nty * ntz) * vol.V();   // first voxel of the sample
    __syncthreads();
    for (int e = threadIdx.x; e < 2 * Tl::hvox; e += 64 * Tl::waves) {
      const int hv = e >> 1, hf = e & 1;
      const int xx = x0 + hv % Tl::hx - 1, yy = y0 + (hv / Tl::hx) % 6 - 1, zz = z0 + hv / (Tl::hx * 6) - 1;
      u4v val = u4v{0u, 0u, 0u, 0u};
      if (xx >= 0 && xx < vol.W && yy >= 0 && yy < vol.H && zz >= 0 && zz < vol.D)
        val = *reinterpret_cast<const u4v*>(X + (v0 + ((long)zz * vol.H + yy) * vol.W + xx) * xcs + xco + ci + hf * 8);
      *reinterpret_cast<u4v*>(xt + hv * 16 + hf * 8) = val;
    }
    for (int e = threadIdx.x; e < 2 * NO * Tl::vox; e += 64 * Tl::waves) {
      const int hf = e & 1, o = (e >> 1) % NO, v = (e >> 1) / NO;
      const int xx = x0 + v % TX, yy = y0 + (v / TX) % 4, zz = z0 + v / (TX * 4);
      u4v val = u4v{0u, 0u, 0u, 0u};
      if (xx < vol.W && yy < vol.H && zz < vol.D)
        val = *reinterpret_cast<const u4v*>(dY + (v0 + ((long)zz * vol.H + yy) * vol.W + xx) * ycs + yco +
                                            (o0 + o) * 16 + hf * 8);
      *reinterpret_cast<u4v*>(yt + (o * Tl::vox + v) * 16 + hf * 8) = val;
    }
    __syncthreads();
#pragma unroll 1
    for (int k = part; k < Tl::vox / 32; k += Tl::ks) {
      const int v = 32 * k + 8 * kq;                       // this lane group's eight voxels
      const int row = v / TX, x = v % TX;
      const bf8v a = read_rows8(yt + (ot * Tl::vox + v) * 16 + rowoff);
      bf16_t* xb = xt + (((row >> 2) * 6 + (row & 3)) * Tl::hx + x) * 16 + rowoff;
#pragma unroll
      for (int t = 0; t < TAPS; ++t) {
        const int off = TAPS == 1 ? (6 + 1) * Tl::hx + 1 : ((t / 9) * 6 + (t / 3) % 3) * Tl::hx + t % 3;
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, read_rows8(xb + off * 16), acc[t], 0, 0, 0);
      }
    }
  }
  if constexpr (Tl::ks > 1) {
    float* red = reinterpret_cast<float*>(smem) + ot * TAPS * 256;
#pragma unroll 1
    for (int p = 1; p < Tl::ks; ++p) {
      __syncthreads();
      if (part == p)
#pragma unroll
        for (int t = 0; t < TAPS; ++t) *reinterpret_cast<f4v*>(red + (t * 64 + lane) * 4) = acc[t];
      __syncthreads();
      if (part == 0)
#pragma unroll
        for (int t = 0; t < TAPS; ++t) acc[t] += *reinterpret_cast<const f4v*>(red + (t * 64 + lane) * 4);
    }
    if (part != 0) return;
  }
#pragma unroll
  for (int t = 0; t < TAPS; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      partial[(((long)blockIdx.x * TAPS + t) * Cout + (o0 + ot) * 16 + 4 * kq + r) * Cin + ci + m] = acc[t][r];
}

// g (+)= sum over chunks of partial, in a fixed order.  A block sums 64 entries with 16
// threads each (every 16th chunk, four loads in flight), then adds the 16 through LDS: with
// one thread per entry the up to 1000 partials of a layer were one chain of loads (43 us a
// layer on average at 32 x 32 x 128).
constexpr int kWrSplit = 16;
__global__ __launch_bounds__(64 * kWrSplit) void k_wreduce(const float* __restrict__ partial, int nchunk, long per,
                                                           float* __restrict__ g, int accumulate) {
  __shared__ float red[kWrSplit][64];
  const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
  for (long i0 = (long)blockIdx.x * 64; i0 < per; i0 += (long)gridDim.x * 64) {
    const long i = i0 + lane;
    float s = 0.f;
    if (i < per) {
      int c = part;
      for (; c + 3 * kWrSplit < nchunk; c += 4 * kWrSplit) {
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = partial[(long)(c + k * kWrSplit) * per + i];
#pragma unroll
        for (int k = 0; k < 4; ++k) s += v[k];
      }
      for (; c < nchunk; c += kWrSplit) s += partial[(long)c * per + i];
    }
    red[part][lane] = s;
    __syncthreads();
    if (part == 0 && i < per) {
      float t = 0.f;
#pragma unroll
      for (int k = 0; k < kWrSplit; ++k) t += red[k][lane];
      g[i] = accumulate ? g[i] + t : t;
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ pooling, upsampling
// Y (coarse) = mean of the 8 children of X (fine); one thread per 8 channels of a
// coarse voxel (C, strides and offsets are multiples of 8: 16-byte accesses)
__global__ void k_pool(const bf16_t* __restrict__ X, int xcs, int xco, bf16_t* __restrict__ Y, int ycs, int yco, int C,
                       Vol fine) {
  const Vol c{fine.D / 2, fine.H / 2, fine.W / 2};
  const int C8 = C / 8;
  const long n = c.V() * C8;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const int ch = (int)(i % C8) * 8;
    const long v = i / C8;
    const int x = (int)(v % c.W), y = (int)((v / c.W) % c.H), z = (int)(v / ((long)c.W * c.H));
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int q = 0; q < 8; ++q) {
      const long fv = (((long)(2 * z + (q >> 2)) * fine.H + 2 * y + ((q >> 1) & 1)) * fine.W + 2 * x + (q & 1));
      const u4v raw = *reinterpret_cast<const u4v*>(X + fv * xcs + xco + ch);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        s[2 * k] += __uint_as_float(raw[k] << 16);
        s[2 * k + 1] += __uint_as_float(raw[k] & 0xFFFF0000u);
      }
    }
    u4v o;
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = (unsigned)f2bf(s[2 * k] * 0.125f) | ((unsigned)f2bf(s[2 * k + 1] * 0.125f) << 16);
    *reinterpret_cast<u4v*>(Y + v * ycs + yco + ch) = o;
  }
}

// dX (fine) (+)= dY[parent] / 8, masked by mask > 0 (the ReLU before the pooling)
__global__ void k_pool_grad(const bf16_t* __restrict__ dY, int ycs, int yco, bf16_t* __restrict__ dX, int xcs, int xco,
                            int C, Vol fine, const bf16_t* __restrict__ mask, int mcs, int mco, int accumulate) {
  const long n = fine.V() * C;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const int ch = (int)(i % C);
    const long v = i / C;
    const int x = (int)(v % fine.W), y = (int)((v / fine.W) % fine.H), z = (int)(v / ((long)fine.W * fine.H));
    const long pv = ((long)(z / 2) * (fine.H / 2) + y / 2) * (fine.W / 2) + x / 2;
    float g = bf2f(dY[pv * ycs + yco + ch]) * 0.125f;
    if (mask && !(bf2f(mask[v * mcs + mco + ch]) > 0.f)) g = 0.f;
    const long o = v * xcs + xco + ch;
    dX[o] = f2bf(accumulate ? bf2f(dX[o]) + g : g);
  }
}

// Y (fine) = X[parent] (nearest neighbour); one thread per 8 channels of a fine voxel
__global__ void k_up(const bf16_t* __restrict__ X, int xcs, int xco, bf16_t* __restrict__ Y, int ycs, int yco, int C,
                     Vol fine) {
  const int C8 = C / 8;
  const long n = fine.V() * C8;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const int ch = (int)(i % C8) * 8;
    const long v = i / C8;
    const int x = (int)(v % fine.W), y = (int)((v / fine.W) % fine.H), z = (int)(v / ((long)fine.W * fine.H));
    const long pv = ((long)(z / 2) * (fine.H / 2) + y / 2) * (fine.W / 2) + x / 2;
    *reinterpret_cast<u4v*>(Y + v * ycs + yco + ch) = *reinterpret_cast<const u4v*>(X + pv * xcs + xco + ch);
  }
}

// dX (coarse) = sum of dY over the 8 children
__global__ void k_up_grad(const bf16_t* __restrict__ dY, int ycs, int yco, bf16_t* __restrict__ dX, int xcs, int xco,
                          int C, Vol fine) {
  const Vol c{fine.D / 2, fine.H / 2, fine.W / 2};
  const long n = c.V() * C;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const int ch = (int)(i % C);
    const long v = i / C;
    const int x = (int)(v % c.W), y = (int)((v / c.W) % c.H), z = (int)(v / ((long)c.W * c.H));
    float s = 0.f;
    for (int q = 0; q < 8; ++q) {
      const long fv = (((long)(2 * z + (q >> 2)) * fine.H + 2 * y + ((q >> 1) & 1)) * fine.W + 2 * x + (q & 1));
      s += bf2f(dY[fv * ycs + yco + ch]);
    }
    dX[v * xcs + xco + ch] = f2bf(s);
  }
}

// ------------------------------------------------------------------ data in / out, loss, Adam
// X0[v][0..15] = (Re/Im r_x, r_y, r_z) * s, Re/Im chi, (Re/Im w_x, w_y, w_z) * s or zeros
// when w is null, zeros;  s = sqrt(3N / ||r||^2)
__global__ void k_pack(const double2* __restrict__ r, const double2* __restrict__ w, const double2* __restrict__ chi,
                       const double2* __restrict__ sumsq, long N, bf16_t* __restrict__ X0) {
  const double s = sumsq->x > 0 ? sqrt(3.0 * (double)N / sumsq->x) : 0.0;
  for (long v = blockIdx.x * (long)blockDim.x + threadIdx.x; v < N; v += (long)gridDim.x * blockDim.x) {
    bf16_t* o = X0 + v * 16;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double2 a = r[(long)c * N + v];
      o[2 * c] = f2bf((float)(a.x * s));
      o[2 * c + 1] = f2bf((float)(a.y * s));
    }
    const double2 k = chi[v];
    o[6] = f2bf((float)k.x);
    o[7] = f2bf((float)k.y);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double2 a = w ? w[(long)c * N + v] : double2{0.0, 0.0};
      o[8 + 2 * c] = f2bf((float)(a.x * s));
      o[9 + 2 * c] = f2bf((float)(a.y * s));
    }
    o[14] = 0;
    o[15] = 0;
  }
}

// mean squared error of out against (target - base) * s over 6 channels; dOut = d(loss)/d(out)
__global__ __launch_bounds__(256) void k_loss(const float* __restrict__ out, const double2* __restrict__ target,
                                              const double2* __restrict__ base, const double2* __restrict__ sumsq,
                                              long N, bf16_t* __restrict__ dOut, float gscale,
                                              double* __restrict__ partial) {
  __shared__ double red[256];
  const double s = sumsq->x > 0 ? sqrt(3.0 * (double)N / sumsq->x) : 0.0;
  double acc = 0.0;
  for (long v = blockIdx.x * (long)blockDim.x + threadIdx.x; v < N; v += (long)gridDim.x * blockDim.x) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double2 t = target[(long)c * N + v], rv = base[(long)c * N + v];
      const float d0 = out[v * 16 + 2 * c] - (float)((t.x - rv.x) * s);
      const float d1 = out[v * 16 + 2 * c + 1] - (float)((t.y - rv.y) * s);
      acc += (double)d0 * d0 + (double)d1 * d1;
      dOut[v * 16 + 2 * c] = f2bf(gscale * d0);
      dOut[v * 16 + 2 * c + 1] = f2bf(gscale * d1);
    }
#pragma unroll
    for (int c = 6; c < 16; ++c) dOut[v * 16 + c] = 0;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// The constants come from the host, formed in FP64 and rounded once: k.omb1 = 1 - beta1,
// k.omb2 = 1 - beta2 and the bias corrections c1 = 1 - beta1^t, c2 = 1 - beta2^t
// (1 - 0.999f in FP32 would carry a relative error of 1.3e-5).
struct AdamK {
  float lr, b1, omb1, b2, omb2, eps, c1, c2;
};

// weight i of n of a layer: Adam step (update), bf16 copy for the forward pass and the
// tap-reversed transposed copy for the input gradient
__device__ __forceinline__ void adam_weight(float* w, float* mo, float* ve, const float* g, long i, const AdamK& k,
                                            int taps, int Cout, int Cin, bf16_t* wbf, bf16_t* wtbf, int update) {
  float wi = w[i];
  if (update) {
    const float gi = g[i];
    const float m1 = k.b1 * mo[i] + k.omb1 * gi;
    const float v1 = k.b2 * ve[i] + k.omb2 * gi * gi;
    mo[i] = m1;
    ve[i] = v1;
    wi -= k.lr * (m1 / k.c1) / (sqrtf(v1 / k.c2) + k.eps);
    w[i] = wi;
  }
  const int ci = (int)(i % Cin);
  const int co = (int)((i / Cin) % Cout);
  const int t = (int)(i / ((long)Cin * Cout));
  const bf16_t h = f2bf(wi);
  wbf[i] = h;
  wtbf[((long)(taps - 1 - t) * Cin + ci) * Cout + co] = h;
}

__global__ void k_adam(float* __restrict__ w, float* __restrict__ mo, float* __restrict__ ve,
                       const float* __restrict__ g, long n, AdamK k, int taps, int Cout, int Cin,
                       bf16_t* __restrict__ wbf, bf16_t* __restrict__ wtbf, int update) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    adam_weight(w, mo, ve, g, i, k, taps, Cout, Cin, wbf, wtbf, update);
}

// every layer of the network in one launch; its weights lie one layer after the other
constexpr int kLayers = 15;
struct LayerTable {
  int first[kLayers + 1];   // multiples of 256
  short taps[kLayers], cout[kLayers], cin[kLayers];
};
__global__ __launch_bounds__(256) void k_adam_net(float* __restrict__ w, float* __restrict__ mo,
                                                  float* __restrict__ ve, const float* __restrict__ g, AdamK k,
                                                  LayerTable lt, bf16_t* __restrict__ wbf, bf16_t* __restrict__ wtbf,
                                                  int update) {
  const int i0 = blockIdx.x * 256;
  int l = 0;
  while (i0 >= lt.first[l + 1]) ++l;   // one layer per block
  const int f = lt.first[l];
  adam_weight(w + f, mo + f, ve + f, g + f, i0 + (int)threadIdx.x - f, k, lt.taps[l], lt.cout[l], lt.cin[l], wbf + f,
              wtbf + f, update);
}

__global__ void k_f2bf(const float* a, bf16_t* b, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) b[i] = f2bf(a[i]);
}

__global__ void k_bf2f(const bf16_t* a, float* b, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) b[i] = bf2f(a[i]);
}

__global__ void k_fill_bf(bf16_t* p, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) p[i] = 0;
}

// Adam (Kingma & Ba) constants of step t and learning rate lr
static inline AdamK adam_constants(int t, float lr) {
  const double b1 = 0.9, b2 = 0.999;
  AdamK k;
  k.lr = lr;
  k.b1 = (float)b1;
  k.omb1 = (float)(1.0 - b1);
  k.b2 = (float)b2;
  k.omb2 = (float)(1.0 - b2);
  k.eps = 1e-8f;
  k.c1 = (float)(1.0 - std::pow(b1, (double)t));
  k.c2 = (float)(1.0 - std::pow(b2, (double)t));
  return k;
}

static inline int gblocks(long n) { return (int)std::min<long>(4096, (n + 255) / 256); }

// k_conv2 may use more than 64 KiB of dynamic LDS (83.5 KiB with four N-tiles); to be allowed on
// the current device before conv_launch
template <int TAPS>
static hipError_t allow_conv_lds_taps() {
  const auto a = hipFuncAttributeMaxDynamicSharedMemorySize;
  hipError_t e;
  if ((e = hipFuncSetAttribute((const void*)k_conv2<TAPS, 1, 2, 2>, a, (int)conv2_lds<2, 2>(TAPS, 1)))) return e;
  if ((e = hipFuncSetAttribute((const void*)k_conv2<TAPS, 2, 2, 2>, a, (int)conv2_lds<2, 2>(TAPS, 2)))) return e;
  if ((e = hipFuncSetAttribute((const void*)k_conv2<TAPS, 3, 2, 2>, a, (int)conv2_lds<2, 2>(TAPS, 3)))) return e;
  if ((e = hipFuncSetAttribute((const void*)k_conv2<TAPS, 4, 2, 2>, a, (int)conv2_lds<2, 2>(TAPS, 4)))) return e;
  return hipFuncSetAttribute((const void*)k_conv2<TAPS, 1, 1, 1>, a, (int)conv2_lds<1, 1>(TAPS, 1));
}
static hipError_t allow_conv_lds() {
  const hipError_t e = allow_conv_lds_taps<27>();
  return e ? e : allow_conv_lds_taps<1>();
}

template <int TAPS>
static void conv2_launch_nt(bool big, int nt, dim3 grid, int n0, hipStream_t s, const bf16_t* X, int xcs, int xco,
                            int Cin, const bf16_t* W, int Cout, bf16_t* Y, int ycs, int yco, float* Yf, Vol vol,
                            int relu, const bf16_t* mask, int mcs, int mco, const ConvUp& up, const NetOut& res) {
#define VIE_CONV2(NTV, TZ, MT)                                                                                   \
  if (nt == NTV && big == (TZ == 2))                                                                             \
    hipLaunchKernelGGL((k_conv2<TAPS, NTV, TZ, MT>), grid, dim3(256), (conv2_lds<TZ, MT>(TAPS, NTV)), s, X, xcs,  \
                       xco, Cin, W, Cout, Y, ycs, yco, Yf, vol, relu, mask, mcs, mco, n0, up, res);
  VIE_CONV2(1, 2, 2)
  VIE_CONV2(2, 2, 2)
  VIE_CONV2(3, 2, 2)
  VIE_CONV2(4, 2, 2)
  VIE_CONV2(1, 1, 1)
#undef VIE_CONV2
}

// The 2 x 4 x 32 voxel tile where it gives at least 512 workgroups, with output-channel
// groups of four N-tiles in one launch and a smaller last group in a second; else the
// 1 x 4 x 16 tile (the small levels of the network) with one N-tile per workgroup: at
// level 2 of 32 x 32 x 256 three N-tiles leave 64 workgroups for 256 CUs, one gives 192
// with a third of the weights to stage each.
hipError_t conv_launch(int taps, const bf16_t* X, int xcs, int xco, int Cin, const bf16_t* W, int Cout, bf16_t* Y,
                       int ycs, int yco, float* Yf, Vol vol, int relu, const bf16_t* mask, int mcs, int mco,
                       hipStream_t s, const ConvUp& up = {}, const NetOut& res = {}) {
  const long big = (long)vol.B * ((vol.D + 1) / 2) * ((vol.H + kCty - 1) / kCty) * ((vol.W + 31) / 32);
  const long small = (long)vol.B * vol.D * ((vol.H + kCty - 1) / kCty) * ((vol.W + 15) / 16);
  const bool use_big = big >= 512;
  const int ntiles = Cout / 16, per = use_big ? 4 : 1, full = ntiles / per, rest = ntiles % per;
  auto go = [&](int nt, int groups, int n0) {
    const dim3 grid((unsigned)(use_big ? big : small), (unsigned)groups);
    if (taps == 27)
      conv2_launch_nt<27>(use_big, nt, grid, n0, s, X, xcs, xco, Cin, W, Cout, Y, ycs, yco, Yf, vol, relu, mask, mcs,
                          mco, up, res);
    else
      conv2_launch_nt<1>(use_big, nt, grid, n0, s, X, xcs, xco, Cin, W, Cout, Y, ycs, yco, Yf, vol, relu, mask, mcs,
                         mco, up, res);
  };
  if (full) go(per, full, 0);
  if (rest) go(rest, 1, full * per);
  return hipGetLastError();
}

// Voxel tiles are spread over enough workgroups to give every CU four (counting the
// chunks of 16 input channels), as far as the partials fit; output tiles go in groups of
// four, a smaller last group in a second launch.  Rows of 16 voxels where the volume is
// no wider (the deep levels), else 32.
template <int TAPS, int TX>
static void wgrad_launch_no(int no, dim3 grid, int o0, hipStream_t s, const bf16_t* X, int xcs, int xco, int Cin,
                            const bf16_t* dY, int ycs, int yco, int Cout, float* partial, Vol vol) {
#define VIE_WGRAD(NOV)                                                                                             \
  if (no == NOV)                                                                                                   \
    hipLaunchKernelGGL((k_wgrad<TAPS, NOV, TX>), grid, dim3(64 * WgradTile<TAPS, NOV, TX>::waves), 0, s, X, xcs,   \
                       xco, Cin, dY, ycs, yco, Cout, partial, vol, o0);
  VIE_WGRAD(1)
  VIE_WGRAD(2)
  VIE_WGRAD(3)
  VIE_WGRAD(4)
#undef VIE_WGRAD
}

hipError_t wgrad_launch(int taps, const bf16_t* X, int xcs, int xco, int Cin, const bf16_t* dY, int ycs, int yco,
                        int Cout, float* partial, long partial_cap, float* g, int accumulate, Vol vol, hipStream_t s) {
  const long per = (long)taps * Cout * Cin;
  const bool narrow = vol.W <= 16;
  const int tx = narrow ? 16 : 32;
  const long tiles = (long)vol.B * ((vol.D + 1) / 2) * ((vol.H + 3) / 4) * ((vol.W + tx - 1) / tx);
  const int ichunks = Cin / 16, otiles = Cout / 16;
  long nblk = std::max(1, 1024 / (ichunks * ((otiles + 3) / 4)));
  nblk = std::max(1L, std::min(std::min(nblk, tiles), partial_cap / per));
  if (nblk * per > partial_cap) return hipErrorInvalidValue;
  for (int o0 = 0; o0 < otiles; o0 += 4) {
    const int no = std::min(4, otiles - o0);
    const dim3 grid((unsigned)nblk, (unsigned)ichunks);
    if (taps == 27 && narrow)
      wgrad_launch_no<27, 16>(no, grid, o0, s, X, xcs, xco, Cin, dY, ycs, yco, Cout, partial, vol);
    else if (taps == 27)
      wgrad_launch_no<27, 32>(no, grid, o0, s, X, xcs, xco, Cin, dY, ycs, yco, Cout, partial, vol);
    else if (narrow)
      wgrad_launch_no<1, 16>(no, grid, o0, s, X, xcs, xco, Cin, dY, ycs, yco, Cout, partial, vol);
    else
      wgrad_launch_no<1, 32>(no, grid, o0, s, X, xcs, xco, Cin, dY, ycs, yco, Cout, partial, vol);
  }
  hipLaunchKernelGGL(k_wreduce, dim3((unsigned)std::min<long>(4096, (per + 63) / 64)), dim3(64 * kWrSplit), 0, s,
                     partial, (int)nblk, per, g, accumulate);
  return hipGetLastError();
}

}  // namespace vie

// =============================================================================
// the network object
// =============================================================================
using namespace vie;

namespace {

struct Conv {
  int taps, cin, cout;       // padded channel counts (multiples of 16)
  int cin_real;
  float *w, *g;              // parts of the network's arrays
  bf16_t *wbf, *wtbf;
  long n() const { return (long)taps * cin * cout; }
};

}  // namespace

struct vie_net_s {
  int n[3];
  Vol lv[4];
  hipStream_t stream;
  Conv L[kLayers];
  float *w, *m, *v, *g;      // all layers' weights, moments, gradients, one layer after the other
  bf16_t *wbf, *wtbf;
  LayerTable lt;
  size_t params;
  // activation buffers, each `batch` samples of elems values, and out, in one allocation (37
  // single ones made the first step of a small network twice as long as the next)
  struct Act {
    bf16_t** p;
    long elems;
  };
  std::vector<Act> acts;
  void* act_mem = nullptr;
  int batch = 0;
  // activations and their gradients
  bf16_t *X0, *E1a, *D1cat, *Dd1a, *Dd1b, *P1, *E2a, *D2cat, *Dd2a, *Dd2b, *P2, *E3a, *D3cat, *Dd3a, *Dd3b, *P3, *E4a,
      *E4b;
  bf16_t *gE1a, *gD1cat, *gDd1a, *gDd1b, *gP1, *gE2a, *gD2cat, *gDd2a, *gDd2b, *gP2, *gE3a, *gD3cat, *gDd3a, *gDd3b,
      *gP3, *gE4a, *gE4b, *gOut;
  float* out;          // [V1][16] FP32 network output
  float* partial;      // wgrad split-K partials
  long partial_cap;
  double2* sumsq;      // ||r||^2 of the current input
  double2* red;        // reduction scratch
  double* lpart;       // loss partials
  double* lpart_h;
  int step = 0;
  std::vector<void*> allocs;
  std::string err;
};

namespace {

hipError_t nalloc(vie_net_s* n, void** p, size_t bytes) {
  hipError_t e = dmalloc(p, bytes);
  if (!e) n->allocs.push_back(*p);
  return e;
}

constexpr int kGroup = 4;      // most samples of a training group
constexpr int kLossParts = 4096;

// the levels' volumes with B samples
struct Levels {
  Vol v[4];
  Levels(const vie_net_s* N, int B) {
    for (int i = 0; i < 4; ++i) v[i] = Vol{N->lv[i].D, N->lv[i].H, N->lv[i].W, B};
  }
  const Vol& operator[](int i) const { return v[i]; }
};

// room for B samples in the activation buffers; false, with the buffers as they were, when
// there is not enough memory
bool net_room(vie_net_s* N, int B) {
  if (B <= N->batch) return true;
  void* fresh = nullptr;
  ScratchCarver c{nullptr};
  for (auto& a : N->acts) c.take<bf16_t>((size_t)a.elems * B);
  const size_t acts = c.used;
  c.take<float>((size_t)N->lv[0].V() * 16 * B);
  if (dmalloc(&fresh, c.used) || hipStreamSynchronize(N->stream)) {
    if (fresh) (void)hipFree(fresh);
    (void)hipGetLastError();
    return false;
  }
  if (N->act_mem) (void)hipFree(N->act_mem);
  N->act_mem = fresh;
  N->batch = B;
  c = ScratchCarver{static_cast<unsigned char*>(fresh)};
  for (auto& a : N->acts) *a.p = c.take<bf16_t>((size_t)a.elems * B);
  N->out = c.take<float>((size_t)N->lv[0].V() * 16 * B);
  const long fill = (long)(acts / sizeof(bf16_t));
  hipLaunchKernelGGL(k_fill_bf, dim3(gblocks(fill)), dim3(256), 0, N->stream, static_cast<bf16_t*>(fresh), fill);
  return true;
}

// forward pass of B samples from X0 to out; all activations kept for the backward pass.  With
// a result (one sample, inference) the upsampled halves of the concatenations are not formed,
// nor is out.
hipError_t net_forward(vie_net_s* N, int B, const NetOut& res = {}) {
  const bool infer = res.z != nullptr;
  hipStream_t s = N->stream;
  const Levels l(N, B);
  hipError_t e;
#define CONV_UP(i, X, xcs, src, Y, ycs, yco, lev, relu)                                                            \
  if ((e = conv_launch(N->L[i].taps, X, xcs, 0, N->L[i].cin, N->L[i].wbf, N->L[i].cout, Y, ycs, yco, nullptr,      \
                       l[lev], relu, nullptr, 0, 0, s, infer ? src : ConvUp{})))                                    \
    return e;
#define CONV(i, X, xcs, xco, Y, ycs, yco, lev, relu)                                                           \
  if ((e = conv_launch(N->L[i].taps, X, xcs, xco, N->L[i].cin, N->L[i].wbf, N->L[i].cout, Y, ycs, yco, nullptr, \
                       l[lev], relu, nullptr, 0, 0, s)))                                                          \
    return e;
  CONV(0, N->X0, 16, 0, N->E1a, 16, 0, 0, 1)
  CONV(1, N->E1a, 16, 0, N->D1cat, 48, 32, 0, 1)
  hipLaunchKernelGGL(k_pool, dim3(gblocks(l[1].all() * 16)), dim3(256), 0, s, N->D1cat, 48, 32, N->P1, 16, 0, 16,
                     l[0].stack());
  CONV(2, N->P1, 16, 0, N->E2a, 32, 0, 1, 1)
  CONV(3, N->E2a, 32, 0, N->D2cat, 80, 48, 1, 1)
  hipLaunchKernelGGL(k_pool, dim3(gblocks(l[2].all() * 32)), dim3(256), 0, s, N->D2cat, 80, 48, N->P2, 32, 0, 32,
                     l[1].stack());
  CONV(4, N->P2, 32, 0, N->E3a, 48, 0, 2, 1)
  CONV(5, N->E3a, 48, 0, N->D3cat, 112, 64, 2, 1)
  hipLaunchKernelGGL(k_pool, dim3(gblocks(l[3].all() * 48)), dim3(256), 0, s, N->D3cat, 112, 64, N->P3, 48, 0, 48,
                     l[2].stack());
  CONV(6, N->P3, 48, 0, N->E4a, 64, 0, 3, 1)
  CONV(7, N->E4a, 64, 0, N->E4b, 64, 0, 3, 1)
  if (!infer)
    hipLaunchKernelGGL(k_up, dim3(gblocks(l[2].all() * 64)), dim3(256), 0, s, N->E4b, 64, 0, N->D3cat, 112, 0, 64,
                     l[2].stack());
  CONV_UP(8, N->D3cat, 112, (ConvUp{N->E4b, 64, 4}), N->Dd3a, 48, 0, 2, 1)
  CONV(9, N->Dd3a, 48, 0, N->Dd3b, 48, 0, 2, 1)
  if (!infer)
    hipLaunchKernelGGL(k_up, dim3(gblocks(l[1].all() * 48)), dim3(256), 0, s, N->Dd3b, 48, 0, N->D2cat, 80, 0, 48,
                     l[1].stack());
  CONV_UP(10, N->D2cat, 80, (ConvUp{N->Dd3b, 48, 3}), N->Dd2a, 32, 0, 1, 1)
  CONV(11, N->Dd2a, 32, 0, N->Dd2b, 32, 0, 1, 1)
  if (!infer)
    hipLaunchKernelGGL(k_up, dim3(gblocks(l[0].all() * 32)), dim3(256), 0, s, N->Dd2b, 32, 0, N->D1cat, 48, 0, 32,
                     l[0].stack());
  CONV_UP(12, N->D1cat, 48, (ConvUp{N->Dd2b, 32, 2}), N->Dd1a, 16, 0, 0, 1)
  CONV(13, N->Dd1a, 16, 0, N->Dd1b, 16, 0, 0, 1)
#undef CONV
#undef CONV_UP
  return conv_launch(1, N->Dd1b, 16, 0, 16, N->L[14].wbf, 16, nullptr, 0, 0, infer ? nullptr : N->out, l[0],
                     0, nullptr, 0, 0, s, {}, res);
}

// backward pass of B samples from gOut; (+)= their weight gradients into L[i].g
hipError_t net_backward(vie_net_s* N, int accumulate, int B) {
  hipStream_t s = N->stream;
  const Levels l(N, B);
  hipError_t e;
  const long cap = N->partial_cap;
  // dgrad of layer i: input gradient (cin channels) from output gradient dY (cout channels)
#define DGRAD(i, dY, ycs, yco, dX, xcs, xco, lev, mask, mcs, mco)                                                 \
  if ((e = conv_launch(N->L[i].taps, dY, ycs, yco, N->L[i].cout, N->L[i].wtbf, N->L[i].cin, dX, xcs, xco, nullptr, \
                       l[lev], 0, mask, mcs, mco, s)))                                                               \
    return e;
#define WGRAD(i, X, xcs, xco, dY, ycs, yco, lev)                                                                   \
  if ((e = wgrad_launch(N->L[i].taps, X, xcs, xco, N->L[i].cin, dY, ycs, yco, N->L[i].cout, N->partial, cap,      \
                        N->L[i].g, accumulate, l[lev], s)))                                                          \
    return e;
  // level 1 decoder
  WGRAD(14, N->Dd1b, 16, 0, N->gOut, 16, 0, 0)
  DGRAD(14, N->gOut, 16, 0, N->gDd1b, 16, 0, 0, N->Dd1b, 16, 0)
  WGRAD(13, N->Dd1a, 16, 0, N->gDd1b, 16, 0, 0)
  DGRAD(13, N->gDd1b, 16, 0, N->gDd1a, 16, 0, 0, N->Dd1a, 16, 0)
  WGRAD(12, N->D1cat, 48, 0, N->gDd1a, 16, 0, 0)
  DGRAD(12, N->gDd1a, 16, 0, N->gD1cat, 48, 0, 0, N->D1cat, 48, 0)
  hipLaunchKernelGGL(k_up_grad, dim3(gblocks(l[1].all() * 32)), dim3(256), 0, s, N->gD1cat, 48, 0, N->gDd2b, 32, 0, 32,
                     l[0].stack());
  // level 2 decoder
  WGRAD(11, N->Dd2a, 32, 0, N->gDd2b, 32, 0, 1)
  DGRAD(11, N->gDd2b, 32, 0, N->gDd2a, 32, 0, 1, N->Dd2a, 32, 0)
  WGRAD(10, N->D2cat, 80, 0, N->gDd2a, 32, 0, 1)
  DGRAD(10, N->gDd2a, 32, 0, N->gD2cat, 80, 0, 1, N->D2cat, 80, 0)
  hipLaunchKernelGGL(k_up_grad, dim3(gblocks(l[2].all() * 48)), dim3(256), 0, s, N->gD2cat, 80, 0, N->gDd3b, 48, 0, 48,
                     l[1].stack());
  // level 3 decoder
  WGRAD(9, N->Dd3a, 48, 0, N->gDd3b, 48, 0, 2)
  DGRAD(9, N->gDd3b, 48, 0, N->gDd3a, 48, 0, 2, N->Dd3a, 48, 0)
  WGRAD(8, N->D3cat, 112, 0, N->gDd3a, 48, 0, 2)
  DGRAD(8, N->gDd3a, 48, 0, N->gD3cat, 112, 0, 2, N->D3cat, 112, 0)
  hipLaunchKernelGGL(k_up_grad, dim3(gblocks(l[3].all() * 64)), dim3(256), 0, s, N->gD3cat, 112, 0, N->gE4b, 64, 0, 64,
                     l[2].stack());
  // bottom
  WGRAD(7, N->E4a, 64, 0, N->gE4b, 64, 0, 3)
  DGRAD(7, N->gE4b, 64, 0, N->gE4a, 64, 0, 3, N->E4a, 64, 0)
  WGRAD(6, N->P3, 48, 0, N->gE4a, 64, 0, 3)
  DGRAD(6, N->gE4a, 64, 0, N->gP3, 48, 0, 3, nullptr, 0, 0)
  // skip E3b = D3cat[64:112]: its gradient already holds the skip path; add the pooling path
  hipLaunchKernelGGL(k_pool_grad, dim3(gblocks(l[2].all() * 48)), dim3(256), 0, s, N->gP3, 48, 0, N->gD3cat, 112, 64, 48,
                     l[2].stack(), N->D3cat, 112, 64, 1);
  WGRAD(5, N->E3a, 48, 0, N->gD3cat, 112, 64, 2)
  DGRAD(5, N->gD3cat, 112, 64, N->gE3a, 48, 0, 2, N->E3a, 48, 0)
  WGRAD(4, N->P2, 32, 0, N->gE3a, 48, 0, 2)
  DGRAD(4, N->gE3a, 48, 0, N->gP2, 32, 0, 2, nullptr, 0, 0)
  hipLaunchKernelGGL(k_pool_grad, dim3(gblocks(l[1].all() * 32)), dim3(256), 0, s, N->gP2, 32, 0, N->gD2cat, 80, 48, 32,
                     l[1].stack(), N->D2cat, 80, 48, 1);
  WGRAD(3, N->E2a, 32, 0, N->gD2cat, 80, 48, 1)
  DGRAD(3, N->gD2cat, 80, 48, N->gE2a, 32, 0, 1, N->E2a, 32, 0)
  WGRAD(2, N->P1, 16, 0, N->gE2a, 32, 0, 1)
  DGRAD(2, N->gE2a, 32, 0, N->gP1, 16, 0, 1, nullptr, 0, 0)
  hipLaunchKernelGGL(k_pool_grad, dim3(gblocks(l[0].all() * 16)), dim3(256), 0, s, N->gP1, 16, 0, N->gD1cat, 48, 32, 16,
                     l[0].stack(), N->D1cat, 48, 32, 1);
  WGRAD(1, N->E1a, 16, 0, N->gD1cat, 48, 32, 0)
  DGRAD(1, N->gD1cat, 48, 32, N->gE1a, 16, 0, 0, N->E1a, 16, 0)
  WGRAD(0, N->X0, 16, 0, N->gE1a, 16, 0, 0)
#undef DGRAD
#undef WGRAD
  return hipGetLastError();
}

hipError_t refresh_weights(vie_net_s* N, int update, float lr) {
  if (update) N->step++;
  const AdamK k = adam_constants(std::max(1, N->step), lr);
  hipLaunchKernelGGL(k_adam_net, dim3((unsigned)(N->params / 256)), dim3(256), 0, N->stream, N->w, N->m, N->v, N->g, k,
                     N->lt, N->wbf, N->wtbf, update);
  return hipGetLastError();
}

int nfail(vie_net_s* n, int code, const std::string& m) {
  if (n) n->err = m;
  return code;
}

}  // namespace

namespace vie {
// used by the solver (vie_api.cpp): z = ||r|| net(r / ||r||, chi)
hipError_t net_apply(vie_net_s* N, const double2* r, const double2* w, const double2* chi, double2* z) {
  const long V = N->lv[0].V();
  hipError_t e;
  if ((e = KrylovOps<double>::nrm2sq(r, 3 * V, N->red, N->sumsq, N->stream))) return e;
  hipLaunchKernelGGL(k_pack, dim3(gblocks(V)), dim3(256), 0, N->stream, r, w, chi, N->sumsq, V, N->X0);
  return net_forward(N, 1, NetOut{w ? w : r, N->sumsq, z});
}
const int* net_grid(vie_net_s* N) { return N->n; }
void net_set_stream(vie_net_s* N, hipStream_t s) { N->stream = s; }
}  // namespace vie

extern "C" {

int vie_net_create(vie_net_t* out, const int grid[3], unsigned seed, void* hip_stream) {
  if (!out || !grid) return VIE_EINVAL;
  *out = nullptr;
  for (int d = 0; d < 3; ++d)
    if (grid[d] < 8 || grid[d] % 8 != 0 || grid[d] > 4096) return VIE_EINVAL;
  auto* N = new vie_net_s();
  std::memcpy(N->n, grid, sizeof(int) * 3);
  N->stream = reinterpret_cast<hipStream_t>(hip_stream);
  for (int l = 0; l < 4; ++l) N->lv[l] = Vol{grid[0] >> l, grid[1] >> l, grid[2] >> l};
  // (taps, cin, cout, cin_real): 16/32/48/64 U-Net, input 8 real channels, output 6
  const int spec[15][4] = {{27, 16, 16, 14},  {27, 16, 16, 16},  {27, 16, 32, 16},  {27, 32, 32, 32},
                           {27, 32, 48, 32},  {27, 48, 48, 48},  {27, 48, 64, 48},  {27, 64, 64, 64},
                           {27, 112, 48, 112}, {27, 48, 48, 48}, {27, 80, 32, 80},  {27, 32, 32, 32},
                           {27, 48, 16, 48},  {27, 16, 16, 16},  {1, 16, 16, 16}};
  auto bail = [&](int code) {
    vie_net_destroy(N);
    return code;
  };
  if (allow_conv_lds()) return bail(VIE_EDEVICE);
  size_t total = 0;
  for (int i = 0; i < kLayers; ++i) {
    Conv& C = N->L[i];
    C.taps = spec[i][0];
    C.cin = spec[i][1];
    C.cout = spec[i][2];
    C.cin_real = spec[i][3];
    N->lt.first[i] = (int)total;
    N->lt.taps[i] = (short)C.taps;
    N->lt.cout[i] = (short)C.cout;
    N->lt.cin[i] = (short)C.cin;
    total += C.n();
  }
  N->lt.first[kLayers] = (int)total;
  N->params = total;
  for (float** p : {&N->w, &N->m, &N->v, &N->g})
    if (nalloc(N, (void**)p, sizeof(float) * total)) return bail(VIE_ENOMEM);
  if (nalloc(N, (void**)&N->wbf, sizeof(bf16_t) * total) || nalloc(N, (void**)&N->wtbf, sizeof(bf16_t) * total))
    return bail(VIE_ENOMEM);
  for (float* q : {N->m, N->v, N->g})
    if (hipMemset(q, 0, sizeof(float) * total)) return bail(VIE_EDEVICE);
  std::mt19937_64 rng(seed);
  for (int i = 0; i < kLayers; ++i) {
    Conv& C = N->L[i];
    const long n = C.n(), f = N->lt.first[i];
    C.w = N->w + f;
    C.g = N->g + f;
    C.wbf = N->wbf + f;
    C.wtbf = N->wtbf + f;
    // He initialisation over the real fan-in; padded input channels and the
    // padded outputs of the last layer stay zero
    std::vector<float> w(n, 0.f);
    std::normal_distribution<double> nd(0.0, std::sqrt(2.0 / (C.taps * C.cin_real)) * (i == 14 ? 0.1 : 1.0));
    const int cout_real = i == 14 ? 6 : C.cout;
    for (int t = 0; t < C.taps; ++t)
      for (int o = 0; o < cout_real; ++o)
        for (int ci = 0; ci < C.cin_real; ++ci) w[((long)t * C.cout + o) * C.cin + ci] = (float)nd(rng);
    if (hipMemcpy(C.w, w.data(), sizeof(float) * n, hipMemcpyHostToDevice)) return bail(VIE_EDEVICE);
  }
  const long V[4] = {N->lv[0].V(), N->lv[1].V(), N->lv[2].V(), N->lv[3].V()};
  struct B {
    bf16_t** p;
    long v;
    int c;
  } bufs[] = {{&N->X0, V[0], 16},    {&N->E1a, V[0], 16},   {&N->D1cat, V[0], 48}, {&N->Dd1a, V[0], 16},
              {&N->Dd1b, V[0], 16},  {&N->P1, V[1], 16},    {&N->E2a, V[1], 32},   {&N->D2cat, V[1], 80},
              {&N->Dd2a, V[1], 32},  {&N->Dd2b, V[1], 32},  {&N->P2, V[2], 32},    {&N->E3a, V[2], 48},
              {&N->D3cat, V[2], 112}, {&N->Dd3a, V[2], 48}, {&N->Dd3b, V[2], 48},  {&N->P3, V[3], 48},
              {&N->E4a, V[3], 64},   {&N->E4b, V[3], 64},   {&N->gE1a, V[0], 16},  {&N->gD1cat, V[0], 48},
              {&N->gDd1a, V[0], 16}, {&N->gDd1b, V[0], 16}, {&N->gP1, V[1], 16},   {&N->gE2a, V[1], 32},
              {&N->gD2cat, V[1], 80}, {&N->gDd2a, V[1], 32}, {&N->gDd2b, V[1], 32}, {&N->gP2, V[2], 32},
              {&N->gE3a, V[2], 48},  {&N->gD3cat, V[2], 112}, {&N->gDd3a, V[2], 48}, {&N->gDd3b, V[2], 48},
              {&N->gP3, V[3], 48},   {&N->gE4a, V[3], 64},  {&N->gE4b, V[3], 64},  {&N->gOut, V[0], 16}};
  for (auto& b : bufs) N->acts.push_back({b.p, b.v * b.c});
  if (!net_room(N, 1)) return bail(VIE_ENOMEM);
  N->partial_cap = 8L << 20;   // floats
  if (nalloc(N, (void**)&N->partial, sizeof(float) * N->partial_cap)) return bail(VIE_ENOMEM);
  if (nalloc(N, (void**)&N->sumsq, sizeof(double2) * 2 * kGroup)) return bail(VIE_ENOMEM);
  // partials of KrylovOps::nrm2sq over the 3V residual values
  if (nalloc(N, (void**)&N->red, sizeof(double2) * (partial_blocks(3 * V[0]) + 1))) return bail(VIE_ENOMEM);
  if (nalloc(N, (void**)&N->lpart, sizeof(double) * kLossParts * kGroup)) return bail(VIE_ENOMEM);
  if (hipHostMalloc(&N->lpart_h, sizeof(double) * kLossParts * kGroup, hipHostMallocDefault)) return bail(VIE_ENOMEM);
  if (refresh_weights(N, 0, 0.f) || hipStreamSynchronize(N->stream)) return bail(VIE_EDEVICE);
  *out = N;
  return VIE_OK;
}

void vie_net_destroy(vie_net_t N) {
  if (!N) return;
  for (void* p : N->allocs) (void)hipFree(p);
  if (N->act_mem) (void)hipFree(N->act_mem);
  if (N->lpart_h) (void)hipHostFree(N->lpart_h);
  delete N;
}

int vie_net_num_params(vie_net_t N, size_t* count) {
  if (!N || !count) return VIE_EINVAL;
  *count = N->params;
  return VIE_OK;
}

int vie_net_get_params(vie_net_t N, float* host, size_t count) {
  size_t c = 0;
  if (!N || !host || vie_net_num_params(N, &c) || c != count) return VIE_EINVAL;
  return hipMemcpy(host, N->w, sizeof(float) * c, hipMemcpyDeviceToHost) ? VIE_EDEVICE : VIE_OK;
}

int vie_net_set_params(vie_net_t N, const float* host, size_t count) {
  size_t c = 0;
  if (!N || !host || vie_net_num_params(N, &c) || c != count) return VIE_EINVAL;
  for (size_t i = 0; i < count; ++i)
    if (!std::isfinite(host[i])) return nfail(N, VIE_EINVAL, "weight " + std::to_string(i) + " is not finite");
  if (hipMemcpy(N->w, host, sizeof(float) * c, hipMemcpyHostToDevice)) return VIE_EDEVICE;
  if (refresh_weights(N, 0, 0.f) || hipStreamSynchronize(N->stream)) return VIE_EDEVICE;
  return VIE_OK;
}

int vie_net_get_state(vie_net_t N, float* host, size_t count, int* step) {
  size_t c = 0;
  if (!N || !host || !step || vie_net_num_params(N, &c) || c != count) return VIE_EINVAL;
  const size_t b = sizeof(float) * count;
  if (hipMemcpy(host, N->w, b, hipMemcpyDeviceToHost) || hipMemcpy(host + count, N->m, b, hipMemcpyDeviceToHost) ||
      hipMemcpy(host + 2 * count, N->v, b, hipMemcpyDeviceToHost))
    return VIE_EDEVICE;
  *step = N->step;
  return VIE_OK;
}

int vie_net_set_state(vie_net_t N, const float* host, size_t count, int step) {
  size_t c = 0;
  if (!N || !host || vie_net_num_params(N, &c) || c != count) return VIE_EINVAL;
  if (step < 0) return nfail(N, VIE_EINVAL, "negative Adam step");
  for (size_t i = 0; i < 3 * count; ++i)
    if (!std::isfinite(host[i])) return nfail(N, VIE_EINVAL, "state value " + std::to_string(i) + " is not finite");
  for (size_t i = 2 * count; i < 3 * count; ++i)
    if (host[i] < 0.f) return nfail(N, VIE_EINVAL, "negative second moment " + std::to_string(i - 2 * count));
  const size_t b = sizeof(float) * count;
  if (hipMemcpy(N->w, host, b, hipMemcpyHostToDevice) || hipMemcpy(N->m, host + count, b, hipMemcpyHostToDevice) ||
      hipMemcpy(N->v, host + 2 * count, b, hipMemcpyHostToDevice))
    return VIE_EDEVICE;
  N->step = step;
  if (refresh_weights(N, 0, 0.f) || hipStreamSynchronize(N->stream)) return VIE_EDEVICE;
  return VIE_OK;
}

int vie_net_apply(vie_net_t N, const vie_c128* r, const vie_c128* chi, vie_c128* z) {
  return vie_net_apply_base(N, r, nullptr, chi, z);
}

int vie_net_apply_base(vie_net_t N, const vie_c128* r, const vie_c128* w, const vie_c128* chi, vie_c128* z) {
  if (!N || !r || !chi || !z) return VIE_EINVAL;
  if (net_apply(N, reinterpret_cast<const double2*>(r), reinterpret_cast<const double2*>(w),
                reinterpret_cast<const double2*>(chi), reinterpret_cast<double2*>(z)))
    return VIE_EDEVICE;
  return VIE_OK;
}

int vie_net_train_step(vie_net_t N, int count, const vie_c128* const* r, const vie_c128* const* chi,
                       const vie_c128* const* target, float lr, double* loss) {
  return vie_net_train_step_base(N, count, r, nullptr, chi, target, lr, loss);
}

int vie_net_train_step_base(vie_net_t N, int count, const vie_c128* const* r, const vie_c128* const* w,
                            const vie_c128* const* chi, const vie_c128* const* target, float lr, double* loss) {
  if (!N || count < 1 || !r || !chi || !target || !(lr >= 0)) return VIE_EINVAL;
  for (int i = 0; i < count; ++i)
    if (!r[i] || !chi[i] || !target[i]) return VIE_EINVAL;
  const long V = N->lv[0].V();
  double total = 0.0;
  const int nb = gblocks(V);
  // The samples run in groups through the same launches: the deep levels, a few dozen
  // workgroups each, take the time of one sample, and every weight gradient is reduced once
  // per group.  A step on 32 x 32 x 128 with two samples and its weights and gradients copied
  // out: 1.86 ms one by one, with the layers' weights updated and copied singly, 1.18 now.
  int group = std::min(count, kGroup);
  while (group > 1 && !net_room(N, group)) --group;
  for (int i0 = 0; i0 < count; i0 += group) {
    const int B = std::min(group, count - i0);
    const float gscale = 2.0f / (6.0f * (float)V * (float)count);
    auto base = [&](int i) { return reinterpret_cast<const double2*>(w && w[i] ? w[i] : r[i]); };
    for (int q = 0; q < B; ++q) {
      const double2* ri = reinterpret_cast<const double2*>(r[i0 + q]);
      double2* sumsq = N->sumsq + 2 * q;
      if (KrylovOps<double>::nrm2sq(ri, 3 * V, N->red, sumsq, N->stream)) return VIE_EDEVICE;
      hipLaunchKernelGGL(k_pack, dim3(gblocks(V)), dim3(256), 0, N->stream, ri,
                         w ? reinterpret_cast<const double2*>(w[i0 + q]) : nullptr,
                         reinterpret_cast<const double2*>(chi[i0 + q]), sumsq, V, N->X0 + q * V * 16);
    }
    if (net_forward(N, B)) return VIE_EDEVICE;
    for (int q = 0; q < B; ++q)
      hipLaunchKernelGGL(k_loss, dim3(nb), dim3(256), 0, N->stream, N->out + q * V * 16,
                         reinterpret_cast<const double2*>(target[i0 + q]), base(i0 + q), N->sumsq + 2 * q, V,
                         N->gOut + q * V * 16, gscale, N->lpart + q * nb);
    if (net_backward(N, i0 > 0 ? 1 : 0, B)) return VIE_EDEVICE;
    if (hipMemcpyAsync(N->lpart_h, N->lpart, sizeof(double) * nb * B, hipMemcpyDeviceToHost, N->stream) ||
        hipStreamSynchronize(N->stream))
      return VIE_EDEVICE;
    for (int q = 0; q < B; ++q) {
      double s = 0.0;
      for (int b = 0; b < nb; ++b) s += N->lpart_h[q * nb + b];
      total += s / (6.0 * (double)V);
    }
  }
  if (refresh_weights(N, 1, lr) || hipStreamSynchronize(N->stream)) return VIE_EDEVICE;
  if (loss) *loss = total / count;
  return VIE_OK;
}

// Diagnostic single-layer operations on FP32 device buffers (converted to BF16
// on the way in, FP32 out) for parity tests: mode 0 forward (relu optional),
// 1 input gradient, 2 weight gradient.
int vie_nn_conv_test(int mode, const int dims[3], int taps, int cin, int cout, const float* x, const float* w,
                     float* out, int relu, void* hip_stream) {
  if (!dims || !x || !out || (taps != 1 && taps != 27) || cin % 16 || cout % 16 || cin < 16 || cout < 16)
    return VIE_EINVAL;
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  const Vol vol{dims[0], dims[1], dims[2]};
  const long V = vol.V();
  const long nw = (long)taps * cin * cout;
  std::vector<void*> tmp;
  auto al = [&](size_t b) {
    void* p = nullptr;
    if (dmalloc(&p, b)) return (void*)nullptr;
    tmp.push_back(p);
    return p;
  };
  auto fin = [&](int c) {
    (void)hipStreamSynchronize(s);
    for (void* p : tmp) (void)hipFree(p);
    return c;
  };
  // convert inputs: x has (mode 0, 2: cin; mode 1: cout) channels per voxel
  const int xc = mode == 1 ? cout : cin;
  if (allow_conv_lds()) return fin(VIE_EDEVICE);
  bf16_t* xb = (bf16_t*)al(sizeof(bf16_t) * V * xc);
  if (!xb) return fin(VIE_ENOMEM);
  hipLaunchKernelGGL(k_f2bf, dim3(gblocks(V * xc)), dim3(256), 0, s, x, xb, V * xc);
  if (mode == 2) {
    // w holds dY (cout channels per voxel)
    bf16_t* yb = (bf16_t*)al(sizeof(bf16_t) * V * cout);
    float* part = (float*)al(sizeof(float) * (8L << 20));
    if (!yb || !part) return fin(VIE_ENOMEM);
    hipLaunchKernelGGL(k_f2bf, dim3(gblocks(V * cout)), dim3(256), 0, s, w, yb, V * cout);
    if (wgrad_launch(taps, xb, cin, 0, cin, yb, cout, 0, cout, part, 8L << 20, out, 0, vol, s)) return fin(VIE_EDEVICE);
    return fin(VIE_OK);
  }
  // weights [taps][cout][cin] FP32 -> BF16 forward copy and flipped-transposed copy
  float* w32 = (float*)al(sizeof(float) * nw);
  float* dummy = (float*)al(sizeof(float) * nw);
  bf16_t* wbf = (bf16_t*)al(sizeof(bf16_t) * nw);
  bf16_t* wtbf = (bf16_t*)al(sizeof(bf16_t) * nw);
  if (!w32 || !dummy || !wbf || !wtbf) return fin(VIE_ENOMEM);
  if (hipMemcpyAsync(w32, w, sizeof(float) * nw, hipMemcpyDeviceToDevice, s)) return fin(VIE_EDEVICE);
  hipLaunchKernelGGL(k_adam, dim3(gblocks(nw)), dim3(256), 0, s, w32, dummy, dummy, dummy, nw, adam_constants(1, 0.f),
                     taps, cout, cin, wbf, wtbf, 0);
  hipError_t e;
  if (mode == 0)
    e = conv_launch(taps, xb, cin, 0, cin, wbf, cout, nullptr, 0, 0, out, vol, relu, nullptr, 0, 0, s);
  else
    e = conv_launch(taps, xb, cout, 0, cout, wtbf, cin, nullptr, 0, 0, out, vol, 0, nullptr, 0, 0, s);
  return fin(e ? VIE_EDEVICE : VIE_OK);
}

int vie_net_get_grads(vie_net_t N, float* host, size_t count) {
  size_t c = 0;
  if (!N || !host || vie_net_num_params(N, &c) || c != count) return VIE_EINVAL;
  if (hipStreamSynchronize(N->stream)) return VIE_EDEVICE;
  return hipMemcpy(host, N->g, sizeof(float) * c, hipMemcpyDeviceToHost) ? VIE_EDEVICE : VIE_OK;
}

// Diagnostic pooling / upsampling on FP32 device buffers (rounded to bfloat16 on
// entry, bfloat16 results widened to FP32), C channels per voxel, fine grid dims:
// op 0 pool x[fine] -> out[coarse]; 1 pool gradient x = dY[coarse] -> out[fine],
// masked by mask[fine] > 0 when mask != NULL and added to acc[fine] when acc != NULL;
// 2 upsampling x[coarse] -> out[fine]; 3 its gradient x = dY[fine] -> out[coarse].
int vie_nn_op_test(int op, const int dims[3], int C, const float* x, const float* mask, const float* acc,
                   float* out, void* hip_stream) {
  if (!dims || !x || !out || C < 8 || C % 8 || op < 0 || op > 3) return VIE_EINVAL;
  for (int d = 0; d < 3; ++d)
    if (dims[d] < 2 || dims[d] % 2) return VIE_EINVAL;
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  const Vol fine{dims[0], dims[1], dims[2]};
  const long Vf = fine.V(), Vc = Vf / 8;
  const long nin = (op == 0 || op == 3) ? Vf * C : Vc * C;
  const long nout = (op == 0 || op == 3) ? Vc * C : Vf * C;
  std::vector<void*> tmp;
  auto al = [&](size_t b) {
    void* p = nullptr;
    if (dmalloc(&p, b)) return (void*)nullptr;
    tmp.push_back(p);
    return p;
  };
  auto fin = [&](int c) {
    (void)hipStreamSynchronize(s);
    for (void* p : tmp) (void)hipFree(p);
    return c;
  };
  bf16_t* xb = (bf16_t*)al(sizeof(bf16_t) * nin);
  bf16_t* ob = (bf16_t*)al(sizeof(bf16_t) * nout);
  if (!xb || !ob) return fin(VIE_ENOMEM);
  hipLaunchKernelGGL(k_f2bf, dim3(gblocks(nin)), dim3(256), 0, s, x, xb, nin);
  bf16_t* mb = nullptr;
  if (op == 1 && mask) {
    if (!(mb = (bf16_t*)al(sizeof(bf16_t) * nout))) return fin(VIE_ENOMEM);
    hipLaunchKernelGGL(k_f2bf, dim3(gblocks(nout)), dim3(256), 0, s, mask, mb, nout);
  }
  if (op == 1 && acc) hipLaunchKernelGGL(k_f2bf, dim3(gblocks(nout)), dim3(256), 0, s, acc, ob, nout);
  if (op == 0)
    hipLaunchKernelGGL(k_pool, dim3(gblocks(nout)), dim3(256), 0, s, xb, C, 0, ob, C, 0, C, fine);
  else if (op == 1)
    hipLaunchKernelGGL(k_pool_grad, dim3(gblocks(nout)), dim3(256), 0, s, xb, C, 0, ob, C, 0, C, fine, mb, C, 0,
                       acc ? 1 : 0);
  else if (op == 2)
    hipLaunchKernelGGL(k_up, dim3(gblocks(nout)), dim3(256), 0, s, xb, C, 0, ob, C, 0, C, fine);
  else
    hipLaunchKernelGGL(k_up_grad, dim3(gblocks(nout)), dim3(256), 0, s, xb, C, 0, ob, C, 0, C, fine);
  hipLaunchKernelGGL(k_bf2f, dim3(gblocks(nout)), dim3(256), 0, s, ob, out, nout);
  return fin(hipGetLastError() ? VIE_EDEVICE : VIE_OK);
}

// Diagnostic Adam step t (t >= 1) on n FP32 device values in place: w, m, v updated
// with gradient g as the training step does.
int vie_nn_adam_test(long n, float* w, float* m, float* v, const float* g, int t, float lr, void* hip_stream) {
  if (n < 1 || !w || !m || !v || !g || t < 1 || !(lr >= 0)) return VIE_EINVAL;
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  bf16_t *wb = nullptr, *wtb = nullptr;
  if (dmalloc(&wb, sizeof(bf16_t) * n)) return VIE_ENOMEM;
  if (dmalloc(&wtb, sizeof(bf16_t) * n)) {
    (void)hipFree(wb);
    return VIE_ENOMEM;
  }
  hipLaunchKernelGGL(k_adam, dim3(gblocks(n)), dim3(256), 0, s, w, m, v, g, n, adam_constants(t, lr), 1, 1, (int)n,
                     wb, wtb, 1);
  const hipError_t e = hipGetLastError();
  (void)hipStreamSynchronize(s);
  (void)hipFree(wb);
  (void)hipFree(wtb);
  return e ? VIE_EDEVICE : VIE_OK;
}

const char* vie_net_last_error(vie_net_t N) { return N ? N->err.c_str() : ""; }

}  // extern "C"
