// Learned coarse correction: a small 3-D U-Net on the coarse vertex grid,
// with its own forward, backward and Adam kernels, the transfers between
// unknowns and the coarse grid, and training data taken from the solver.
//
// Network (4 levels, widths c0..c3, in_ch input channels): 'same' 3x3x3
// convolutions with zero padding, ReLU, average pooling over the existing
// children, nearest upsampling, additive skips:
//   enc_l: h = relu(conv_b(relu(conv_a(x))))   (l = 0..2, pool after)
//   bottom: relu(conv_b(relu(conv_a(.))))
//   dec_l: h = relu(conv_a(up(h))) + s_l; h = relu(conv_b(h))  (l = 2,1,0)
//   head:  conv(c0 -> 1)
// Parameters: one flat FP32 master vector (per convolution W[co][ci][27]
// then b[co]; tap = dz*9 + dy*3 + dx), a BF16 copy used by every
// convolution, FP32 activations and FP32 accumulation.
//
// Convolution kernels: implicit GEMMs on the BF16 matrix cores (MFMA) with
// FP32 accumulation.  A workgroup stages a 4x4x4 brick of its input with a
// one-voxel halo in LDS, split into BF16 terms (three for the forward and
// data-gradient passes, which keeps FP32 accuracy with BF16 weights; two
// for the weight gradient), and runs the 27 taps from there.  The data
// gradient is the forward kernel on weights packed transposed with the taps
// mirrored.  Pooling, upsampling, skips and ReLU masks, and their gradients, are
// part of the convolution before or after them (ConvMode): one launch per
// convolution.  The weight gradients of all layers are one launch at the end of
// the backward pass: brick ranges summed into partials that a second launch adds
// in a fixed order (no atomics).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <vector>

#include "dev_common.h"
#include "learned.h"
#include "wgrad_dev.h"

namespace fc {


__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// ---------------------------------------------------------- MFMA convolutions
// Every convolution is an implicit GEMM on the 16x16x32 BF16 matrix cores
// with FP32 accumulation.  Operand layouts of v_mfma_f32_16x16x32_bf16 (one
// wave): lane l supplies A[l % 16][8 (l / 16) + j] and B[8 (l / 16) + j]
// [l % 16], j = 0..7, and holds D[4 (l / 16) + j][l % 16], j = 0..3.
//
// A workgroup owns a brick of 4x4x4 voxels; its input, with a one-voxel
// halo (6x6x6), is staged once in LDS, already split into BF16 terms, and
// every tap of the stencil reads it there.  A 16-voxel row tile of the GEMM
// is one 4x4 (y, x) plane of the brick.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // in a row of a grid

__device__ __forceinline__ f32x4 mfma32(uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr int kHaloVox = 216;   // 6^3 halo voxels of a 4^3 brick

// two BF16 numbers (nearest even) in one word, the first in the low half
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
}

// v = h0 + h1 + h2 in BF16 with |v - (h0 + h1 + h2)| <= 2^-24 |v| (each
// term the BF16 rounding of what the earlier ones leave; the remainders are
// exact in FP32).  Products of BF16 numbers are exact in FP32, so three
// MFMAs over the three terms give the FP32-accurate product with a BF16
// weight.  Two terms leave 2^-16 |v|.  Two numbers at a time.
template <int kTerms>
__device__ __forceinline__ void split_bf16(float a, float b, uint32_t (&h)[kTerms]) {
#pragma unroll
  for (int s = 0; s < kTerms; ++s) {
    h[s] = pack_bf16(a, b);
    a -= __uint_as_float(h[s] << 16);
    b -= __uint_as_float(h[s] & 0xffff0000u);
  }
}

// offset of tap t = dz*9 + dy*3 + dx in a 6x6x6 halo (taps past 26 are
// padding with zero weight and read the corner)
__device__ __forceinline__ int halo_tap_offset(int t) {
  if (t >= 27) return 0;
  const int dz = t / 9, r = t - 9 * dz, dy = r / 3;
  return dz * 36 + dy * 6 + (r - 3 * dy);
}

// Reduction layout of a convolution with cin input channels: chunks of cc
// channels (4, 8 or 16), each chunk a run of ksteps * 32 reduction indices
// k = tap * cc + c (c the channel within the chunk), zero weights past
// 27 * cc.
struct ConvK {
  int cc, nchunk, ksteps, krow;
};

inline ConvK conv_k(int cin) {
  ConvK g;
  g.cc = cin <= 4 ? 4 : cin <= 8 ? 8 : 16;
  g.nchunk = (cin + g.cc - 1) / g.cc;
  g.ksteps = (27 * g.cc + 31) / 32;
  g.krow = g.nchunk * g.ksteps * 32;
  return g;
}

// What a convolution does with its result val (bias added), on top of the layer
// itself: every elementwise, pooling or upsampling pass next to it.
enum ConvMode {
  kConvPlain,     // y = val
  kConvRelu,      // y = relu(val)
  kConvReluPool,  // y = relu(val), y2 = its average over the existing children
  kConvReluAdd,   // y = relu(val), y2 = y + e1
  kConvMask,      // y = val where e1 > 0, else 0
  kConvMaskTwo,   // y = val, y2 = val where e1 > 0, else 0
  kConvSumMask,   // y2 = sum over the existing children where e1 > 0, else 0
  kConvExpand,    // y on the finer grid N2: gradient of the average, plus e2,
                  // where e1 > 0, else 0
};

struct ConvArgs {
  const float* x;
  const uint16_t* W;
  const float* bias;     // may be null
  float *y, *y2;
  const float *e1, *e2;
  int Ci, nchunk, krow, Co, N, nb;
  int up;                // 1: x is on the grid of (N + 1) / 2, nearest upsampling
  int mode, N2;          // ConvMode; grid of y2 (pooling) or y (expanding)
  FastDiv dnb;           // division by nb
};

// sum_{i,t} w(o,i,t) x[b][i][v + off_t] with the weights packed by k_pack_conv
// (rows o of krow BF16 values, chunks of kCc input channels) and the input split
// into three BF16 terms.  Workgroup: brick blockIdx.x (nb^3 per sample), output
// channels 16 blockIdx.y .. + 15 (one column tile), sample blockIdx.z; wave w
// computes plane z = w % 4 of the brick.  Per chunk, the halo input and the
// tile's weights are staged in LDS, the next chunk's loads in flight during the
// products.  kKs = 4: sixteen waves, the reduction steps of a plane dealt to four
// of them and added at the end, and the loads of two chunks in flight; for grids
// that leave the chip idle, where a step is a chain of latencies.
// Bound by latencies and instruction issue: a workgroup is one pass of load,
// split, 27 taps and store.  Against the layer alone, with pooling, upsampling,
// skip and mask passes between: 25 launches and 152 us -> 15 and 98 us for one
// 33^3 grid; the network's gradient on eight 25^3 grids 1,150 us in 95 launches ->
// 494 us in 33.
template <int kCc, int kKs>
__global__ __launch_bounds__(256 * kKs) void k_conv3d(const ConvArgs A) {
  constexpr int kT = 256 * kKs;
  constexpr int kRs = kCc == 16 ? 24 : kCc;      // LDS row of a halo voxel (pad: banks)
  constexpr int kSteps = (27 * kCc + 31) / 32;
  constexpr int kWRow = kSteps * 32 + 8;         // LDS row of one output channel
  constexpr int kIter = kCc / 4 > kKs ? kCc / 4 / kKs : 1;   // runs of 4 channels per thread
  constexpr int kWItems = 16 * kSteps * 4;       // 8 weights per item
  constexpr int kWIter = (kWItems + kT - 1) / kT;
  constexpr int kXs = kHaloVox * kRs;
  constexpr int kRed = kKs > 1 ? 3 * 4 * 64 * 8 : 0;   // in 16-bit words
  constexpr int kLds = 3 * kXs + 16 * kWRow > kRed ? 3 * kXs + 16 * kWRow : kRed;
  __shared__ __align__(16) uint16_t lds[kLds];   // [term][voxel][channel], [column][k]
  __shared__ float2 pool[2][64];
  uint16_t* wl = lds + 3 * kXs;
  const int N = A.N, V = N * N * N, nb = A.nb, Ci = A.Ci, Co = A.Co;
  const int Ns = A.up ? (N + 1) / 2 : N, Vs = Ns * Ns * Ns;
  const int b = blockIdx.z, o0 = blockIdx.y * 16;
  const int line = (int)fdiv(blockIdx.x, A.dnb), bx = blockIdx.x - line * nb;
  const int bz = (int)fdiv(line, A.dnb), by = line - bz * nb;
  const int x0 = 4 * bx - 1, y0 = 4 * by - 1, z0 = 4 * bz - 1;   // halo corner
  const int tid = threadIdx.x, w = (tid >> 6) & 3, l = tid & 63, r16 = l & 15, kg = l >> 4;
  const int ks = kKs > 1 ? __builtin_amdgcn_readfirstlane(tid >> 8) : 0;
  const int hv0 = (w * 6 + (r16 >> 2)) * 6 + (r16 & 3);   // this lane's A row, tap 0
  // one accumulator per input term (independent MFMA chains), added
  // smallest term first at the end
  f32x4 acc[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the halo voxel of this thread; a run of 256 threads takes the channels 4 q ..
  // of the chunk, q = ks, ks + kKs, .. (wave-uniform)
  const int hv = tid & 255;
  const int hz = hv / 36, hr = hv - 36 * hz, hy = hr / 6, hx = hr - 6 * hy;
  const int vz = z0 + hz, vy = y0 + hy, vx = x0 + hx;
  const bool inside = hv < kHaloVox && vz >= 0 && vz < N && vy >= 0 && vy < N && vx >= 0 && vx < N;
  const int vox = inside ? ((vz >> A.up) * Ns + (vy >> A.up)) * Ns + (vx >> A.up) : 0;
  const float* xb = A.x + (int64_t)b * Ci * Vs;
  struct Chunk {
    float v[kIter][4];
    uint4 wv[kWIter];
  };
  auto load = [&](int ch, Chunk& c) {
#pragma unroll
    for (int it = 0; it < kIter; ++it)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = ch * kCc + 4 * (ks + kKs * it) + j;
        c.v[it][j] = xb[(int64_t)min(i, Ci - 1) * Vs + vox];
      }
#pragma unroll
    for (int it = 0; it < kWIter; ++it) {
      const int e = tid + kT * it;
      const int r = e / (4 * kSteps), q = e - r * 4 * kSteps;
      c.wv[it] = uint4{0u, 0u, 0u, 0u};
      if (e < kWItems && o0 + r < Co)
        c.wv[it] = *reinterpret_cast<const uint4*>(A.W + (int64_t)(o0 + r) * A.krow +
                                                   (int64_t)ch * kSteps * 32 + 8 * q);
    }
  };
  auto stage = [&](int ch, const Chunk& c) {
#pragma unroll
    for (int it = 0; it < kIter; ++it) {
      const int q = ks + kKs * it, i = ch * kCc + 4 * q;
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = inside && i + j < Ci ? c.v[it][j] : 0.f;
      uint32_t h0[3], h1[3];
      split_bf16(v[0], v[1], h0);
      split_bf16(v[2], v[3], h1);
      if (hv < kHaloVox && 4 * q < kCc)
#pragma unroll
        for (int s = 0; s < 3; ++s)
          *reinterpret_cast<uint2*>(&lds[s * kXs + hv * kRs + 4 * q]) = uint2{h0[s], h1[s]};
    }
#pragma unroll
    for (int it = 0; it < kWIter; ++it) {
      const int e = tid + kT * it;
      if (e >= kWItems) continue;
      const int r = e / (4 * kSteps), q = e - r * 4 * kSteps;
      *reinterpret_cast<uint4*>(&wl[r * kWRow + 8 * q]) = c.wv[it];
    }
  };
  struct Operands {
    uint4 a[3], b;
  };
  auto fetch = [&](int s, Operands& p) {
    const int k = 32 * s + 8 * kg;   // this lane's eight reduction indices
    p.b = *reinterpret_cast<const uint4*>(&wl[r16 * kWRow + k]);
    const int t = k / kCc, c = k - t * kCc;
    const int a0 = (hv0 + halo_tap_offset(t)) * kRs + c;
    const int a1 = kCc == 4 ? (hv0 + halo_tap_offset(t + 1)) * kRs : 0;
#pragma unroll
    for (int h = 0; h < 3; ++h) {
      if constexpr (kCc == 4) {
        const uint2 p0 = *reinterpret_cast<const uint2*>(&lds[h * kXs + a0]);
        const uint2 p1 = *reinterpret_cast<const uint2*>(&lds[h * kXs + a1]);
        p.a[h] = uint4{p0.x, p0.y, p1.x, p1.y};
      } else {
        p.a[h] = *reinterpret_cast<const uint4*>(&lds[h * kXs + a0]);
      }
    }
  };
  auto multiply = [&](const Operands& p) {
#pragma unroll
    for (int h = 0; h < 3; ++h) acc[h] = mfma32(p.a[h], p.b, acc[h]);
  };
  // the reads of a step one step ahead of its products
  auto compute = [&] {
    constexpr int kMine = (kSteps + kKs - 1) / kKs;
    Operands p[2];
    fetch(min(ks, kSteps - 1), p[0]);
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      // a step past the last repeats it and is not multiplied
      if (i + 1 < kMine) fetch(min(ks + kKs * (i + 1), kSteps - 1), p[(i + 1) & 1]);
      if (kSteps % kKs == 0 || i < kMine - 1 || ks + kKs * i < kSteps) multiply(p[i & 1]);
    }
  };
  if constexpr (kKs == 1) {
    Chunk c;
    load(0, c);
    for (int ch = 0; ch < A.nchunk; ++ch) {
      if (ch > 0) __syncthreads();   // the previous chunk's reads are done
      stage(ch, c);
      __syncthreads();
      if (ch + 1 < A.nchunk) load(ch + 1, c);
      compute();
    }
  } else {
    Chunk c0, c1;
    load(0, c0);
    if (A.nchunk > 1) load(1, c1);
    for (int ch = 0; ch < A.nchunk; ch += 2) {
      if (ch > 0) __syncthreads();
      stage(ch, c0);
      __syncthreads();
      if (ch + 2 < A.nchunk) load(ch + 2, c0);
      compute();
      if (ch + 1 >= A.nchunk) break;
      __syncthreads();
      stage(ch + 1, c1);
      __syncthreads();
      if (ch + 3 < A.nchunk) load(ch + 3, c1);
      compute();
    }
  }
  f32x4 sum = (acc[2] + acc[1]) + acc[0];
  if constexpr (kKs > 1) {
    f32x4* red = reinterpret_cast<f32x4*>(lds);
    __syncthreads();
    if (ks > 0) red[((ks - 1) * 4 + w) * 64 + l] = sum;
    __syncthreads();
    if (ks == 0)
#pragma unroll
      for (int k = 1; k < kKs; ++k) sum += red[((k - 1) * 4 + w) * 64 + l];
  }
  // D[4 kg + j][r16]: voxel (y = kg, x = j) of plane w, channel o0 + r16
  const int gz = z0 + 1 + w, gy = y0 + 1 + kg, gx0 = x0 + 1, o = o0 + r16;
  const bool in = ks == 0 && gz < N && gy < N && o < Co;
  const int64_t bo = (int64_t)b * Co + o;
  const float bias = A.bias && o < Co ? A.bias[o] : 0.f;
  const int mode = A.mode;
  const bool relu = mode >= kConvRelu && mode <= kConvReluAdd;
  f32x4 val;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    val[j] = sum[j] + bias;
    if (relu) val[j] = fmaxf(val[j], 0.f);
  }
  // a lane's four voxels are one row of the brick: 16-byte accesses unless the
  // grid ends in it (every 4-byte store is a request of its own: 64 per
  // instruction)
  auto put = [&](float* p, const f32x4 v, int n) {
    if (n >= 4)
      *reinterpret_cast<f32x4u*>(p) = v;
    else
#pragma unroll
      for (int j = 0; j < 3; ++j)
        if (j < n) p[j] = v[j];
  };
  auto get = [&](const float* p, int n) {
    f32x4 v{0.f, 0.f, 0.f, 0.f};
    if (n >= 4)
      v = *reinterpret_cast<const f32x4u*>(p);
    else
#pragma unroll
      for (int j = 0; j < 3; ++j)
        if (j < n) v[j] = p[j];
    return v;
  };
  auto masked = [&](const f32x4 e, const f32x4 v) {
    f32x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = e[j] > 0.f ? v[j] : 0.f;
    return r;
  };
  const int nrow = N - gx0;   // voxels of the row in the grid (four at most count)
  if (mode == kConvExpand) {
    if (in) {
      const int F = A.N2;
      const int nz = 2 * gz + 1 < F ? 2 : 1, ny = 2 * gy + 1 < F ? 2 : 1;
#pragma unroll
      for (int h = 0; h < 2; ++h) {   // two coarse voxels, four fine ones
        const int fx = 2 * gx0 + 4 * h;
        if (fx >= F) break;
        f32x4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v[j] = val[2 * h + j / 2] /
                 (float)(nz * ny * (2 * (gx0 + 2 * h + j / 2) + 1 < F ? 2 : 1));
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int dz = c >> 1, dy = c & 1;
          if (dz >= nz || dy >= ny) continue;
          const int64_t f = ((bo * F + 2 * gz + dz) * F + 2 * gy + dy) * F + fx;
          put(A.y + f, masked(get(A.e1 + f, F - fx), v + get(A.e2 + f, F - fx)), F - fx);
        }
      }
    }
  } else if (in && mode != kConvSumMask) {
    const int64_t at = bo * V + (gz * N + gy) * N + gx0;
    if (mode == kConvMask) {
      put(A.y + at, masked(get(A.e1 + at, nrow), val), nrow);
    } else {
      put(A.y + at, val, nrow);
      if (mode == kConvReluAdd) put(A.y2 + at, val + get(A.e1 + at, nrow), nrow);
      if (mode == kConvMaskTwo) put(A.y2 + at, masked(get(A.e1 + at, nrow), val), nrow);
    }
  }
  if (mode != kConvReluPool && mode != kConvSumMask) return;
  // 2x2x2 children: x within the lane, y one 16-lane group on, z one wave on
  float2 c;
  c.x = (in && gx0 < N ? val[0] : 0.f) + (in && gx0 + 1 < N ? val[1] : 0.f);
  c.y = (in && gx0 + 2 < N ? val[2] : 0.f) + (in && gx0 + 3 < N ? val[3] : 0.f);
  c.x += __shfl_xor(c.x, 16, 64);
  c.y += __shfl_xor(c.y, 16, 64);
  if (ks == 0 && (w & 1)) pool[w >> 1][l] = c;
  __syncthreads();
  if (ks != 0 || (w & 1) || (kg & 1)) return;
  const float2 up = pool[w >> 1][l];
  const int H = A.N2, Z = 2 * bz + (w >> 1), Y = 2 * by + (kg >> 1);
  if (Z >= H || Y >= H || o >= Co) return;
  const float s2[2] = {c.x + up.x, c.y + up.y};
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int X = 2 * bx + j;
    if (X >= H) break;
    const int64_t at = ((bo * H + Z) * H + Y) * H + X;
    if (mode == kConvSumMask) {
      A.y2[at] = A.e1[at] > 0.f ? s2[j] : 0.f;
    } else {
      const int cnt = (2 * Z + 1 < N ? 2 : 1) * (2 * Y + 1 < N ? 2 : 1) * (2 * X + 1 < N ? 2 : 1);
      A.y2[at] = s2[j] / (float)cnt;
    }
  }
}

// Packed BF16 weights of one layer for k_conv3d.  Forward (trans = 0): row
// o of Co rows, reduction over the Ci input channels, value W[o][i][t].
// Data gradient (trans = 1): row i of Ci rows, reduction over the Co output
// channels with the taps mirrored, value W[o][i][26 - t] (the adjoint of a
// 'same' convolution is the convolution with the mirrored stencil).
__global__ void k_pack_conv(const float* __restrict__ w, int Co, int Ci, int trans, int cc,
                            int ksteps, int krow, uint16_t* __restrict__ out) {
  const int rows = trans ? Ci : Co, cin = trans ? Co : Ci;
  const int64_t total = (int64_t)rows * krow;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int r = (int)(e / krow), k = (int)(e - (int64_t)r * krow);
    const int chunk = k / (ksteps * 32), kk = k - chunk * ksteps * 32;
    const int t = kk / cc, c = chunk * cc + kk % cc;
    float v = 0.f;
    if (t < 27 && c < cin)
      v = trans ? w[((int64_t)c * Ci + r) * 27 + 26 - t] : w[((int64_t)r * Ci + c) * 27 + t];
    out[e] = f2bf(v);
  }
}

// Weight gradients gw[o][i][t] = sum_{b,v} g[b][o][v] x[b][i][v + off_t] and
// gb[o] = sum g[b][o][v] of every layer, on the matrix cores: rows o, columns
// the 16 input channels i of one tile per tap, reduction over the voxels of a
// brick (32 per step: two 4x4 planes), both operands split into two BF16 terms
// and the three products above 2^-16 summed.  A workgroup takes 16 input
// channels, 16 output channels and a range of bricks (over samples and space) of
// one layer; wave w the taps of five of the nine (dz, dy), on planes 2 (w % 2) and
// next.  A lane reads the rows of its channel and shifts them for the three dx.  The sums go to
// part[range][t][o][i] (slot t = 27 of i = 0: bias); k_wgrad_reduce adds the
// ranges in order (deterministic, no atomics).
// Bound by instruction issue (340 vector instructions a wave and brick).  Eight
// 25^3 grids: 88 us for all layers, 465 us in 15 launches of 16x16x16 products
// with three shifted copies of x in LDS.
struct WgradJob {
  const float *x, *g;
  int64_t nbricks, per, part;   // bricks, bricks per range, offset of the partials
  int Ci, Co, N, nb, up;        // up: x is on the grid of (N + 1) / 2
  int nic, nop, nrange;
  int wg0, red0;                // first workgroup of the sums and of the reduction
  int64_t woff, boff;           // of the gradient
};
struct WgradJobs {
  WgradJob j[15];
};

__global__ __launch_bounds__(kWgradThreads, 3) void k_conv3d_wgrad(const WgradJobs jobs,
                                                                float* __restrict__ part) {
  constexpr int kXRow = 148;                      // dwords per channel: 36 rows of 4, pad
  constexpr int kGRow = 36;                       // dwords per channel: 64 voxels, pad
  constexpr int kXIter = kWgradXIter;
  constexpr int kGIter = kWgradGIter;
  constexpr int kXs = 16 * kXRow, kGs = 16 * kGRow;
  __shared__ __align__(16) uint32_t lds[2][2 * (kXs + kGs)];   // [buffer][x terms, g terms]
  int id = 0;
  while (id < 14 && (int)blockIdx.x >= jobs.j[id + 1].wg0) ++id;
  const WgradJob& J = jobs.j[id];
  const int local = blockIdx.x - J.wg0;
  const int ic = local % J.nic, oc = (local / J.nic) % J.nop, range = local / (J.nic * J.nop);
  const int i0 = ic * 16, o0 = oc * 16, N = J.N, nb = J.nb, Ci = J.Ci, Co = J.Co;
  const int Ns = J.up ? (N + 1) / 2 : N, V = N * N * N, Vs = Ns * Ns * Ns;
  const int nx = min(16, Ci - i0), ng = min(16, Co - o0);
  const int tid = threadIdx.x, l = tid & 63, r16 = l & 15, kg = l >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = w & 1, zy0 = 4 * (w >> 1);   // (dz, dy) pairs zy0 .. zy0 + 4
  f32x4 acc[16];   // fifteen taps, bias
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int64_t lo = range * J.per, hi = min(lo + J.per, J.nbricks);
  const int up = J.up;
  const WgradX X = wgrad_x(tid, Ns, up);
  const WgradG G = wgrad_g(tid, N);
  const int64_t xci = (int64_t)X.c * Vs, gco = (int64_t)G.c * V;
  const int xat = X.c * kXRow + X.row * 4 + X.col;
  const int gat = G.c * kGRow + G.pair;
  float2 xv[kXIter], gv[kGIter];
  bool x0in, x1in, g0in, g1in;
  // brick of the next load, stepped (a division per brick costs as much as its
  // products)
  int b, bx, by, bz;
  {
    const int64_t nb3 = (int64_t)nb * nb * nb;
    b = (int)(lo / nb3);
    const int brick = (int)(lo - b * nb3);
    bx = brick % nb;
    by = (brick / nb) % nb;
    bz = brick / (nb * nb);
  }
  auto load = [&] {
    const uint32_t in = wgrad_inside(bx, by, bz, N);
    x0in = (in & X.need0) == X.need0;
    x1in = (in & X.need1) == X.need1;
    g0in = (in & G.need0) == G.need0;
    g1in = (in & G.need1) == G.need1;
    const int64_t corner = wgrad_corner(bx, by, bz, Ns, up);
    const float* xb = J.x + ((int64_t)b * Ci + i0) * Vs + corner;
    // a pair's second channel past the last one repeats the first
    const float* p0 = xb + (x0in ? X.off0 : X.own);
    const float* p1 = xb + (x1in ? X.off1 : X.own);
#pragma unroll
    for (int it = 0; it < kXIter; ++it) {
      if (2 * it >= nx) break;
      const int64_t ci = 2 * it + 1 < nx ? xci : 0;
      xv[it].x = p0[ci];
      xv[it].y = p1[ci];
      p0 += 2 * (int64_t)Vs;
      p1 += 2 * (int64_t)Vs;
    }
    const float* gb = J.g + ((int64_t)b * Co + o0) * V + ((int64_t)4 * bz * N + 4 * by) * N + 4 * bx;
    const float* q0 = gb + gco + (g0in ? G.off : 0);
    const float* q1 = gb + gco + (g1in ? G.off + 1 : 0);
#pragma unroll
    for (int it = 0; it < kGIter; ++it) {
      if (8 * it >= ng) break;
      const int64_t co = (int64_t)8 * it * V - (8 * it + G.c < ng ? 0 : gco);
      gv[it].x = q0[co];
      gv[it].y = q1[co];
    }
    if (++bx == nb) {
      bx = 0;
      if (++by == nb) {
        by = 0;
        if (++bz == nb) {
          bz = 0;
          ++b;
        }
      }
    }
  };
  auto put = [&](uint32_t* p0, uint32_t* p1, float a, float b) {
    uint32_t h[2];
    split_bf16(a, b, h);
    *p0 = h[0];
    *p1 = h[1];
  };
  if (lo < hi) load();
  for (int64_t bi = lo; bi < hi; ++bi) {
    uint32_t* xs = lds[(bi - lo) & 1];
    uint32_t* gs = xs + 2 * kXs;
#pragma unroll
    for (int it = 0; it < kXIter; ++it) {
      if (2 * it >= nx) break;
      const int at = xat + 2 * it * kXRow;
      if (X.act && 2 * it + X.c < nx)
        put(&xs[at], &xs[kXs + at], x0in ? xv[it].x : 0.f, x1in ? xv[it].y : 0.f);
    }
#pragma unroll
    for (int it = 0; it < kGIter; ++it) {
      if (8 * it >= ng) break;
      const int at = gat + 8 * it * kGRow;
      if (8 * it + G.c < ng)
        put(&gs[at], &gs[kGs + at], g0in ? gv[it].x : 0.f, g1in ? gv[it].y : 0.f);
    }
    // one barrier per brick: the next brick goes to the other buffer, whose
    // readers passed this barrier's predecessor
    __syncthreads();
    if (bi + 1 < hi) load();   // in flight during the products below
    // A: g[o][voxels 32 half + 8 kg ..]: plane 2 half + kg / 2, rows 2 (kg % 2)
    // and next; B: the same voxels of x, shifted by the tap
    const int ga = r16 * kGRow + 16 * half + 4 * kg;
    const int xa = r16 * kXRow + ((2 * half + (kg >> 1)) * 6 + 2 * (kg & 1)) * 4;
    const uint4 g0 = *reinterpret_cast<const uint4*>(&gs[ga]);
    const uint4 g1 = *reinterpret_cast<const uint4*>(&gs[kGs + ga]);
    const uint4 ones{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};   // BF16 1.0
    acc[15] = mfma32(g1, ones, acc[15]);
    acc[15] = mfma32(g0, ones, acc[15]);
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const int dz = (zy0 + i) / 3, dy = zy0 + i - 3 * dz;   // wave-uniform
      const uint32_t* p = &xs[xa + (dz * 6 + dy) * 4];
      uint4 xt[2][3];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint4 a = *reinterpret_cast<const uint4*>(p + h * kXs);
        const uint4 b = *reinterpret_cast<const uint4*>(p + h * kXs + 4);
        xt[h][0] = uint4{a.x, a.y, b.x, b.y};
        xt[h][1] = uint4{__builtin_amdgcn_alignbit(a.y, a.x, 16),
                         __builtin_amdgcn_alignbit(a.z, a.y, 16),
                         __builtin_amdgcn_alignbit(b.y, b.x, 16),
                         __builtin_amdgcn_alignbit(b.z, b.y, 16)};
        xt[h][2] = uint4{a.y, a.z, b.y, b.z};
      }
      // the three products of a tap go to the same sums: three taps interleaved
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
          acc[3 * i + dx] = mfma32(k == 0 ? g1 : g0, xt[k == 1][dx], acc[3 * i + dx]);
      __builtin_amdgcn_sched_barrier(0);   // reads hoisted further spill registers
    }
  }
  // the two plane pairs added
  f32x4* red = reinterpret_cast<f32x4*>(&lds[0][0]);
  static_assert(2 * 16 * 64 * sizeof(f32x4) <= sizeof(lds), "sums of two waves");
  __syncthreads();
  if (half == 1)
#pragma unroll
    for (int q = 0; q < 16; ++q) red[((w >> 1) * 16 + q) * 64 + l] = acc[q];
  __syncthreads();
  if (half != 0) return;
  // D[4 kg + j][r16]: output channel o0 + 4 kg + j, input channel i0 + r16; the
  // second pair of waves leaves out the taps it shares with the first
  float* out = part + J.part + (int64_t)range * 28 * Co * Ci;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const f32x4 v = acc[q] + red[((w >> 1) * 16 + q) * 64 + l];
    const int t = q < 15 ? 3 * zy0 + q : 27;
    if (q < 3 && zy0 != 0) continue;
    if (q == 15 && (zy0 != 0 || ic != 0 || r16 != 0)) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int o = o0 + 4 * kg + j;
      if (o < Co && i0 + r16 < Ci) out[((int64_t)t * Co + o) * Ci + i0 + r16] = v[j];
    }
  }
}

// gw[o][i][t] and gb[o] of every layer from the per-range sums: 32 outputs per
// workgroup of 256 threads, thread (slice, output) adds ranges slice, slice + 8,
// .. in order, then the 8 slice sums are added in order (deterministic).
__global__ __launch_bounds__(256) void k_wgrad_reduce(const WgradJobs jobs,
                                                      const float* __restrict__ part,
                                                      float* __restrict__ g) {
  __shared__ float sums[8][33];
  int id = 0;
  while (id < 14 && (int)blockIdx.x >= jobs.j[id + 1].red0) ++id;
  const WgradJob& J = jobs.j[id];
  const int lane = threadIdx.x & 31, slice = threadIdx.x >> 5;
  const int64_t e = (int64_t)(blockIdx.x - J.red0) * 32 + lane;
  const int64_t per = (int64_t)J.Co * J.Ci, nout = 28 * per;
  const int t = (int)(e / per), oi = (int)(e - t * per), o = oi / J.Ci, i = oi - o * J.Ci;
  const bool on = e < nout && (t < 27 || i == 0);
  float s = 0.f;
  if (on) {
    const float* p = part + J.part + e;
#pragma unroll 4
    for (int c = slice; c < J.nrange; c += 8) s += p[c * nout];
  }
  sums[slice][lane] = s;
  __syncthreads();
  if (slice != 0 || !on) return;
  float tot = 0.f;
  for (int k = 0; k < 8; ++k) tot += sums[k][lane];
  if (t < 27) g[J.woff + (int64_t)oi * 27 + t] = tot;
  else g[J.boff + o] = tot;
}

// mean squared error: per-workgroup partial sums and g = 2 (y - t) / n
__global__ __launch_bounds__(256) void k_mse(const float* __restrict__ y,
                                             const float* __restrict__ t, float* __restrict__ g,
                                             int64_t n, double* __restrict__ partial) {
  __shared__ double red[16];
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float d = y[i] - t[i];
    s += (double)d * d;
    g[i] = 2.f * d / (float)n;
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// omb1 = 1 - beta1, omb2 = 1 - beta2, c1 = 1 - beta1^t, c2 = 1 - beta2^t are
// formed in FP64 by the host: in FP32 the differences from 1 lose about
// 1e-5 of their value to cancellation (1 - 0.999f is off by 1.3e-5
// relative), which would bias every update by that much.
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, int64_t n, float lr, float b1, float b2, float omb1,
                       float omb2, float eps, float c1, float c2) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + omb1 * gi;
    const float vi = b2 * v[i] + omb2 * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

static inline dim3 grid1(int64_t n) {
  return dim3((unsigned)std::min<int64_t>((n + 255) / 256, 8192));
}

// ------------------------------------------------------------ network
static const int kLayerIO[15][2] = {{-1, 0}, {0, 0}, {0, 1}, {1, 1}, {1, 2}, {2, 2}, {2, 3},
                                    {3, 3}, {3, 2}, {2, 2}, {2, 1}, {1, 1}, {1, 0}, {0, 0},
                                    {0, -2}};

void Net::init(const int32_t* c, int32_t in_channels) {
  for (int i = 0; i < 4; ++i) ch[i] = c[i];
  in_ch = in_channels;
  int64_t off = 0;
  for (int l = 0; l < 15; ++l) {
    ci[l] = kLayerIO[l][0] == -1 ? in_ch : ch[kLayerIO[l][0]];
    co[l] = kLayerIO[l][1] == -2 ? 1 : ch[kLayerIO[l][1]];
    woff[l] = off;
    off += (int64_t)ci[l] * co[l] * 27;
    boff[l] = off;
    off += co[l];
  }
  nparam = off;
  int64_t e = 0;
  for (int l = 0; l < 15; ++l) {
    wfoff[l] = e;
    e += (int64_t)co[l] * conv_k(ci[l]).krow;
    wtoff[l] = e;
    e += (int64_t)ci[l] * conv_k(co[l]).krow;
  }
  nwpk = e;
}

int64_t net_param_count(const int32_t* c, int32_t in_channels) {
  Net n;
  n.init(c, in_channels);
  return n.nparam;
}

// One workgroup per 4^3 brick and 16 output channels, of 16 waves where there are
// fewer than kSplitBelow of them: 27 bricks of 32 channels take 7 us instead of
// 10.5, while 512 bricks of eight 13^3 grids take 15 instead of 12.5 (two
// workgroups of 16 waves fit a compute unit, three to four of four waves).
constexpr int64_t kSplitBelow = 512;

static hipError_t launch_conv(ConvArgs a, int B, hipStream_t s) {
  const ConvK k = conv_k(a.Ci);
  a.nchunk = k.nchunk;
  a.krow = k.krow;
  a.nb = (a.N + 3) / 4;
  a.dnb = make_fastdiv((uint32_t)a.nb);
  const dim3 g((unsigned)(a.nb * a.nb * a.nb), (unsigned)((a.Co + 15) / 16), (unsigned)B);
  const bool split = (int64_t)g.x * g.y * g.z < kSplitBelow;
#define FC_CONV(CC)                                                       \
  if (split)                                                              \
    hipLaunchKernelGGL((k_conv3d<CC, 4>), g, dim3(1024), 0, s, a);        \
  else                                                                    \
    hipLaunchKernelGGL((k_conv3d<CC, 1>), g, dim3(256), 0, s, a);
  if (k.cc == 4) {
    FC_CONV(4)
  } else if (k.cc == 8) {
    FC_CONV(8)
  } else {
    FC_CONV(16)
  }
#undef FC_CONV
  return hipGetLastError();
}

// layer l on x, or with trans the gradient of its input from that of its output
static ConvArgs conv_args(const Net& net, int l, bool trans, const float* x, float* y, int N,
                          int mode) {
  ConvArgs a{};
  a.x = x;
  a.W = net.wpk + (trans ? net.wtoff[l] : net.wfoff[l]);
  a.bias = trans ? nullptr : net.p + net.boff[l];
  a.y = y;
  a.Ci = trans ? net.co[l] : net.ci[l];
  a.Co = trans ? net.ci[l] : net.co[l];
  a.N = N;
  a.mode = mode;
  return a;
}

// Partials of the weight gradients for batch B: sizes and first workgroups of
// every layer's ranges.  About kWgradWgs workgroups in all, each with the same
// number of bricks, so the last one to start is as short as the others.  Three fit
// a compute unit, 768 the chip: about two rounds.  Eight 25^3 grids: 88 us, 89 in one
// round (730) and 91 in three (2,250), each with more partials to add.
constexpr int64_t kWgradWgs = 1480;
constexpr int64_t kWgradRanges = 512;   // of a layer, at most

struct WgradPlan {
  WgradJobs jobs;
  int64_t wgs = 0, red = 0, floats = 0;
};

static WgradPlan wgrad_plan(const Net& net, const int* N, int B) {
  WgradPlan P{};
  static const int level[15] = {0, 0, 1, 1, 2, 2, 3, 3, 2, 2, 1, 1, 0, 0, 0};
  int64_t total = 0;
  for (int l = 0; l < 15; ++l) {
    WgradJob& J = P.jobs.j[l];
    J.Ci = net.ci[l];
    J.Co = net.co[l];
    J.N = N[level[l]];
    J.nb = (J.N + 3) / 4;
    J.up = l == 8 || l == 10 || l == 12;
    J.nic = (J.Ci + 15) / 16;
    J.nop = (J.Co + 15) / 16;
    J.nbricks = (int64_t)B * J.nb * J.nb * J.nb;
    J.woff = net.woff[l];
    J.boff = net.boff[l];
    total += J.nbricks * J.nic * J.nop;
  }
  for (int l = 0; l < 15; ++l) {
    WgradJob& J = P.jobs.j[l];
    J.per = std::max((total + kWgradWgs - 1) / kWgradWgs,
                     (J.nbricks + kWgradRanges - 1) / kWgradRanges);
    J.nrange = (int)((J.nbricks + J.per - 1) / J.per);
    const int64_t nout = (int64_t)28 * J.Co * J.Ci;
    J.part = P.floats;
    J.wg0 = (int)P.wgs;
    J.red0 = (int)P.red;
    P.floats += J.nrange * nout;
    P.wgs += (int64_t)J.nrange * J.nic * J.nop;
    P.red += (nout + 31) / 32;
  }
  return P;
}

fc_status NetWs::ensure(const Net& net, int B_, int N0) {
  if (B_ <= capB && N0 == N[0] && buf) return FC_OK;
  release();
  B = B_;
  N[0] = N0;
  for (int l = 1; l < 4; ++l) N[l] = (N[l - 1] + 1) / 2;
  int64_t total = 0;
  for (int l = 0; l < 4; ++l)
    for (int k = 0; k < kSlots; ++k) {
      // every tensor of a level has its width; the pooled input the one above
      const int64_t width = k == kIn && l > 0 ? net.ch[l - 1] : net.ch[l];
      off[l][k] = total;
      if (k == kIn ? l > 0 : l < 3 || k == kA || k == kB || k == kGa || k == kGb)
        total += (int64_t)B * width * vox(l);
    }
  off_y = total;
  total += 2 * (int64_t)B * vox(0);   // output and its gradient
  // a smaller batch may be cut into more ranges of some layers
  wslots = 0;
  for (int b = 1; b <= B; ++b) wslots = std::max(wslots, wgrad_plan(net, N, b).floats);
  hipError_t e = dev_malloc(&buf, total * sizeof(float));
  if (e == hipSuccess) e = dev_malloc(&partial, 1024 * sizeof(double));
  if (e == hipSuccess) e = dev_malloc(&wpart, (size_t)wslots * sizeof(float));
  if (e != hipSuccess) {
    release();
    set_error("network workspace allocation failed");
    return FC_E_NOMEM;
  }
  capB = B_;
  return FC_OK;
}

void NetWs::release() {
  if (buf) (void)hipFree(buf);
  if (partial) (void)hipFree(partial);
  if (wpart) (void)hipFree(wpart);
  buf = nullptr;
  partial = nullptr;
  wpart = nullptr;
  capB = 0;
}

hipError_t net_forward(const Net& net, NetWs& ws, const float* x, float* y, int B, hipStream_t s) {
  const int* N = ws.N;
  hipError_t e;
  const float* in = x;
  for (int l = 0; l < 4; ++l) {
    float *a = ws.t(l, kA), *b = ws.t(l, kB);
    if ((e = launch_conv(conv_args(net, 2 * l, false, in, a, N[l], kConvRelu), B, s)) != hipSuccess)
      return e;
    ConvArgs c = conv_args(net, 2 * l + 1, false, a, b, N[l], l < 3 ? kConvReluPool : kConvRelu);
    if (l < 3) {
      c.y2 = ws.t(l + 1, kIn);
      c.N2 = N[l + 1];
      in = c.y2;
    }
    if ((e = launch_conv(c, B, s)) != hipSuccess) return e;
  }
  const float* h = ws.t(3, kB);
  for (int l = 2; l >= 0; --l) {
    const int la = 8 + 2 * (2 - l), lb = la + 1;
    ConvArgs c = conv_args(net, la, false, h, ws.t(l, kDa), N[l], kConvReluAdd);
    c.up = 1;
    c.e1 = ws.t(l, kB);
    c.y2 = ws.t(l, kM);
    if ((e = launch_conv(c, B, s)) != hipSuccess) return e;
    if ((e = launch_conv(conv_args(net, lb, false, ws.t(l, kM), ws.t(l, kDb), N[l], kConvRelu), B,
                         s)) != hipSuccess)
      return e;
    h = ws.t(l, kDb);
  }
  return launch_conv(conv_args(net, 14, false, h, y, N[0], kConvPlain), B, s);
}

// Backward from gy (B,1,N0^3) into net.g (parameters); x is the input.  The
// gradients of the tensors first, then those of all weights from them.
hipError_t net_backward(Net& net, NetWs& ws, const float* x, float* gy, int B, hipStream_t s) {
  const int* N = ws.N;
  hipError_t e;
  WgradPlan P = wgrad_plan(net, N, B);
  auto weights = [&](int l, const float* xin, const float* g) {
    P.jobs.j[l].x = xin;
    P.jobs.j[l].g = g;
  };
  // data gradient of layer l on grid n
  auto data = [&](int l, const float* g, float* y, int n, int mode, const float* e1,
                  float* y2 = nullptr, const float* e2 = nullptr, int N2 = 0) {
    ConvArgs c = conv_args(net, l, true, g, y, n, mode);
    c.e1 = e1;
    c.e2 = e2;
    c.y2 = y2;
    c.N2 = N2;
    return launch_conv(c, B, s);
  };
  weights(14, ws.t(0, kDb), gy);
  if ((e = data(14, gy, ws.t(0, kGdb), N[0], kConvMask, ws.t(0, kDb))) != hipSuccess) return e;
  for (int l = 0; l < 3; ++l) {
    const int la = 8 + 2 * (2 - l), lb = la + 1;
    const float* below = l < 2 ? ws.t(l + 1, kDb) : ws.t(3, kB);
    float* gbelow = l < 2 ? ws.t(l + 1, kGdb) : ws.t(3, kGb);
    weights(lb, ws.t(l, kM), ws.t(l, kGdb));
    // the gradient flows to the skip (kGm) and, masked, to the decoder (kGda)
    if ((e = data(lb, ws.t(l, kGdb), ws.t(l, kGm), N[l], kConvMaskTwo, ws.t(l, kDa),
                  ws.t(l, kGda))) != hipSuccess)
      return e;
    weights(la, below, ws.t(l, kGda));
    if ((e = data(la, ws.t(l, kGda), nullptr, N[l], kConvSumMask, below, gbelow, nullptr,
                  N[l + 1])) != hipSuccess)
      return e;
  }
  for (int l = 3; l >= 0; --l) {
    weights(2 * l + 1, ws.t(l, kA), ws.t(l, kGb));
    if ((e = data(2 * l + 1, ws.t(l, kGb), ws.t(l, kGa), N[l], kConvMask, ws.t(l, kA))) !=
        hipSuccess)
      return e;
    weights(2 * l, l == 0 ? x : ws.t(l, kIn), ws.t(l, kGa));
    if (l > 0 && (e = data(2 * l, ws.t(l, kGa), ws.t(l - 1, kGb), N[l], kConvExpand,
                           ws.t(l - 1, kB), nullptr, ws.t(l - 1, kGm), N[l - 1])) != hipSuccess)
      return e;
  }
  hipLaunchKernelGGL(k_conv3d_wgrad, dim3((unsigned)P.wgs), dim3(kWgradThreads), 0, s, P.jobs,
                     ws.wpart);
  hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)P.red), dim3(256), 0, s, P.jobs, ws.wpart,
                     net.g);
  return hipGetLastError();
}

hipError_t net_mse(NetWs& ws, const float* target, float* gy, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_mse, dim3(1024), dim3(256), 0, s, ws.y(), target, gy, n, ws.partial);
  return hipGetLastError();
}

hipError_t net_adam(Net& net, float lr, int64_t step, hipStream_t s) {
  const double b1 = 0.9, b2 = 0.999;
  const float c1 = (float)(1.0 - std::pow(b1, (double)step));
  const float c2 = (float)(1.0 - std::pow(b2, (double)step));
  hipLaunchKernelGGL(k_adam, grid1(net.nparam), dim3(256), 0, s, net.p, net.g, net.m, net.v,
                     net.nparam, lr, (float)b1, (float)b2, (float)(1.0 - b1), (float)(1.0 - b2),
                     1e-8f, c1, c2);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return net_sync_bf16(net, s);
}

hipError_t net_sync_bf16(Net& net, hipStream_t s) {
  for (int l = 0; l < 15; ++l) {
    const int ci = net.ci[l], co = net.co[l];
    const ConvK kf = conv_k(ci), kt = conv_k(co);
    hipLaunchKernelGGL(k_pack_conv, grid1((int64_t)co * kf.krow), dim3(256), 0, s,
                       net.p + net.woff[l], co, ci, 0, kf.cc, kf.ksteps, kf.krow,
                       net.wpk + net.wfoff[l]);
    hipLaunchKernelGGL(k_pack_conv, grid1((int64_t)ci * kt.krow), dim3(256), 0, s,
                       net.p + net.woff[l], co, ci, 1, kt.cc, kt.ksteps, kt.krow,
                       net.wpk + net.wtoff[l]);
  }
  return hipGetLastError();
}

}  // namespace fc
