// libnsk: the learned closure's C ABI (include/nsk.h): setting the network
// of a context, the nudging step that produces training pairs, and the
// training kernels (loss and gradient, Adam, target moments).  Device code of
// the network and the features is in closure.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

#include "../../include/nsk.h"
#include "closure.hpp"
#include "dg_kernels.hpp"
#include "host_common.hpp"

namespace nsk {
namespace {

// Network outputs on a list of feature vectors X[n][4] -> Y[n][2] (no output
// scaling).  256 nodes per workgroup.
__global__ void __launch_bounds__(kClosureThreads)
mlp_forward_kernel(const uint16_t* __restrict__ w, const float* __restrict__ X, long long n, float* __restrict__ Y) {
  __shared__ float4 sX[kClosureThreads];
  __shared__ __attribute__((aligned(16))) uint16_t sW[2 * kMlpHid * kWPad];
  __shared__ __attribute__((aligned(16))) float sP[kCSmall];
  mlp_stage_params(w, sW, sP);
  const int t = threadIdx.x;
  const long long s = (long long)blockIdx.x * kClosureThreads + t;
  sX[t] = s < n ? reinterpret_cast<const float4*>(X)[s] : make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();
  float y[2];
  mlp_wave(sX, sW, sP, (t >> 6) << 6, y);
  if (s < n) {
    Y[2 * s] = y[0];
    Y[2 * s + 1] = y[1];
  }
}


// ---- training: loss and gradient --------------------------------------------------
// A workgroup of four waves takes tiles of 128 samples (optionally gathered
// through idx), gridDim.x tiles apart, and writes its sum of the gradient
// (kMlpParams values) and loss to part[blockIdx.x][0 .. kMlpParams].  Backward
// treats the BF16 rounding of the activations as the identity.
//
// A wave carries 32 samples, the columns of its matrix products, through the
// forward and the backward chain in registers: the accumulator layout of one
// layer is the operand layout of the next.  Only the weight gradients, sums
// over samples, go through LDS ([unit][sample]); there wave w forms the 32x32
// block (w / 2, w % 2) of both 64x64 gradients over all 128 samples, so that
// no sum crosses waves.
//
// All four 64x64 products of the backward pass multiply an FP32 value (dz) by
// a BF16 one (a weight or an activation).  dz is split into three BF16 terms of 8
// bits, which hold its 24 exactly; the products are then exact and are added in
// FP32 in the accumulators.  That is three BF16 matrix products of 16 steps where
// the FP32 ones would take eight of 2 (96 cycles against 512).  An infinite dz is
// in every term, so that its products are what they are in FP32.
//
// Sums over samples are FP32 within a tile, 8 matrix steps of 16 samples or 32
// additions, and FP64 beyond it, over the tiles of a workgroup and over the
// workgroups (the kernel with one thread a value added 32 samples in FP32 and the
// rest in FP64).  FP32 over a workgroup's tiles loses what they add to a large sum: with
// 32 tiles, the first with residuals of 1 and the others of 2^-22, 124 2^-24 of the
// result.  The FP64 sums take 12 % where a workgroup walks (372 -> 422 us at 2^20
// samples); up to 256 tiles each workgroup has one (WALK false) and there are none.
//
// Measured at a batch of 32768: 21 us, and 4.5 us for the sum over workgroups
// (76 and 38 us with 1024 workgroups of 32 samples in vector arithmetic, whose
// partial gradients were 36 MB).  Bound by the serial chain of one tile at one
// wave per SIMD; the LDS (157 KB) allows one workgroup per CU.
constexpr int kTrainTile = 32;      // samples that the workspace is sized by
constexpr int kTrainSamples = 128;  // samples of a workgroup's tile, 32 a wave
constexpr int kTrainThreads = 256;
constexpr int kTrainGrid = 256;     // workgroups at most: one per CU
constexpr int kSPad = kTrainSamples + 8;   // BF16 values per unit, rows 16-byte aligned and off the bank period
constexpr int kSPadF = kTrainSamples + 1;  // FP32 values per unit

// 16 bytes of parameters at any address a uint16_t may have
struct __attribute__((packed, aligned(2))) ParamWord16 {
  uint32_t x, y, z, w;
};

// a sample's features and targets (any address a float may have)
struct __attribute__((packed, aligned(4))) Row4 {
  float x, y, z, w;
};
struct __attribute__((packed, aligned(4))) Row2 {
  float x, y;
};

// four consecutive accumulator registers g of block ib hold units
// ib 32 + 8 g + 4 half + (0..3)
__device__ __forceinline__ void acc_bias(f32x16 (&acc)[2], const float* bias, int half) {
#pragma unroll
  for (int ib = 0; ib < 2; ++ib)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 b = *reinterpret_cast<const float4*>(bias + ib * 32 + 8 * g + 4 * half);
      acc[ib][4 * g + 0] = b.x;
      acc[ib][4 * g + 1] = b.y;
      acc[ib][4 * g + 2] = b.z;
      acc[ib][4 * g + 3] = b.w;
    }
}

// acc += W bop, W a 64x64 BF16 matrix in LDS with rows of kWPad
__device__ __forceinline__ void acc_product(f32x16 (&acc)[2], const uint16_t* W, const bf16x4 (&bop)[8], int half,
                                            int col) {
#pragma unroll
  for (int S = 0; S < 4; ++S)
#pragma unroll
    for (int ib = 0; ib < 2; ++ib) {
      const uint16_t* wr = W + (ib * 32 + col) * kWPad + 16 * S + 4 * half;
      const bf16x8 a = bf16_cat8(*reinterpret_cast<const bf16x4*>(wr), *reinterpret_cast<const bf16x4*>(wr + 8));
      acc[ib] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bf16_cat8(bop[2 * S], bop[2 * S + 1]), acc[ib], 0, 0, 0);
    }
}

// bit ib 16 + r: accumulator register r of block ib is positive
__device__ __forceinline__ uint32_t acc_mask(const f32x16 (&acc)[2]) {
  uint32_t m = 0;
#pragma unroll
  for (int ib = 0; ib < 2; ++ib)
#pragma unroll
    for (int r = 0; r < 16; ++r) m |= acc[ib][r] > 0.f ? 1u << (ib * 16 + r) : 0u;
  return m;
}

// The BF16 activations of z as the next operand, and into sH[unit][sample].
__device__ __forceinline__ void put_activation(const f32x16 (&z)[2], bf16x4 (&bop)[8], uint16_t* sH, int half,
                                               int sample) {
#pragma unroll
  for (int ib = 0; ib < 2; ++ib)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const bf16x4 v =
          act_bf16x4(bf16_pack4(z[ib][4 * g], z[ib][4 * g + 1], z[ib][4 * g + 2], z[ib][4 * g + 3]));
      bop[4 * ib + g] = v;
#pragma unroll
      for (int q = 0; q < 4; ++q) sH[(ib * 32 + 8 * g + 4 * half + q) * kSPad + sample] = uint16_t(v[q]);
    }
}

// d *= g'(z) from the bits of m.  True where the wave holds an infinite or NaN
// value: there a product, as infinity times 0 is NaN and has to stay so.
__device__ __forceinline__ bool mask_gradient(f32x16 (&d)[2], uint32_t m) {
  float s = 0.f;
#pragma unroll
  for (int ib = 0; ib < 2; ++ib)
#pragma unroll
    for (int r = 0; r < 16; ++r) s = fmaf(d[ib][r], 0.f, s);
  const bool bad = __any(s != s);
  if (bad) {
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r) d[ib][r] *= float((m >> (ib * 16 + r)) & 1u);
  } else {
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r) d[ib][r] = (m >> (ib * 16 + r)) & 1u ? d[ib][r] : 0.f;
  }
  return bad;
}

// The three BF16 terms of dz, largest first, as operands and into
// sDz[term][unit][sample]: the upper half of its bits, then of what is left.
// INF: values may be infinite; what is left of one is taken to be itself.
template <bool INF>
__device__ __forceinline__ void put_split(const f32x16 (&dz)[2], bf16x4 (&term)[3][8], uint16_t* sDz, int half,
                                          int sample) {
  typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int ib = 0; ib < 2; ++ib)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      float v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = dz[ib][4 * g + q];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const auto up = [&](int q) {
          return __builtin_amdgcn_perm(__float_as_uint(v[q + 1]), __float_as_uint(v[q]), 0x07060302u);
        };
        const bf16x4 b = __builtin_bit_cast(bf16x4, (u32x2_t){up(0), up(2)});
        term[p][4 * ib + g] = b;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          sDz[(p * kMlpHid + ib * 32 + 8 * g + 4 * half + q) * kSPad + sample] = uint16_t(b[q]);
          const float t = __uint_as_float(__float_as_uint(v[q]) & 0xFFFF0000u);
          v[q] = INF && fabsf(t) == INFINITY ? t : v[q] - t;
        }
      }
    }
}

// register k of g
__device__ __forceinline__ float acc_at(const f32x16& g, int k) {
  float v = g[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) v = k == r ? g[r] : v;
  return v;
}

// gw += the 32x32 block (ub, jb) of sum_s dz[u][s] h[j][s] over the tile, and
// with bias gb += sum_s dz[u][s] (in every column), smallest terms first.
__device__ __forceinline__ void weight_gradient(f32x16& gw, f32x16& gb, bool bias, const uint16_t* sDz,
                                                const uint16_t* sH, int ub, int jb, int half, int col) {
  const uint16_t* h = sH + (jb * 32 + col) * kSPad + 8 * half;
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const bf16x8 ones = __builtin_bit_cast(bf16x8, (s16x8){0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80, 0x3F80});
#pragma unroll
  for (int p = 2; p >= 0; --p) {
    const uint16_t* d = sDz + (p * kMlpHid + ub * 32 + col) * kSPad + 8 * half;
#pragma unroll
    for (int t = 0; t < kTrainSamples / 16; ++t) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(d + 16 * t);
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(h + 16 * t);
      gw = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, gw, 0, 0, 0);
      if (bias) gb = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, ones, gb, 0, 0, 0);
    }
  }
}

// WALK: a workgroup may have more than one tile.
template <bool WALK>
__global__ void __launch_bounds__(kTrainThreads, 1)
mlp_train_kernel(const uint16_t* __restrict__ w, const float* __restrict__ X, const float* __restrict__ Yt,
                 const int* __restrict__ idx, long long n, float inv_n, float tscale0, float tscale1,
                 float* __restrict__ part) {
  constexpr int T = kTrainSamples, Hd = kMlpHid;
  __shared__ __attribute__((aligned(16))) uint16_t sW[2 * Hd * kWPad];   // W2, W3
  __shared__ __attribute__((aligned(16))) uint16_t sWT[2 * Hd * kWPad];  // their transposes
  __shared__ __attribute__((aligned(16))) float sP[kCSmall];
  __shared__ __attribute__((aligned(16))) uint16_t sH[2][Hd * kSPad];    // h1, h2
  __shared__ __attribute__((aligned(16))) uint16_t sDz[3 * Hd * kSPad];  // dz3, then dz2
  __shared__ float sF[Hd * kSPadF];                                      // h3, then dz1
  __shared__ float4 sX[T];
  __shared__ float sDy[kMlpOut][T];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, half = lane >> 5, col = lane & 31;
  const int smp = wave * 32 + col;  // the lane's sample of the tile
  {
    // parameters into LDS, every load issued before the first is used (2 us
    // less than one after the other)
    constexpr int CH = Hd / 8, NW = 2 * Hd * CH / kTrainThreads, NS = (kCSmall + kTrainThreads - 1) / kTrainThreads;
    ParamWord16 v[NW];
    uint16_t small[NS];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int k = t + i * kTrainThreads, l = k / (Hd * CH), r = (k / CH) % Hd, cc = k % CH;
      v[i] = *reinterpret_cast<const ParamWord16*>(w + (l ? kOffW3 : kOffW2) + r * Hd + 8 * cc);
    }
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const int k = min(t + i * kTrainThreads, kCSmall - 1);
      small[i] = w[k < kCB2 ? k : (k < kCB3 ? kOffB2 + (k - kCB2) : kOffB3 + (k - kCB3))];
    }
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int k = t + i * kTrainThreads, l = k / (Hd * CH), r = (k / CH) % Hd, cc = k % CH;
      uint2* dst = reinterpret_cast<uint2*>(sW + l * Hd * kWPad + r * kWPad + 8 * cc);
      dst[0] = make_uint2(v[i].x, v[i].y);
      dst[1] = make_uint2(v[i].z, v[i].w);
      const uint32_t q[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
      for (int j = 0; j < 8; ++j)
        sWT[l * Hd * kWPad + (8 * cc + j) * kWPad + r] = uint16_t(q[j / 2] >> (16 * (j % 2)));
    }
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const int k = t + i * kTrainThreads;
      if (k < kCSmall) sP[k] = bf16_to_f32(small[i]);
    }
  }
  const int ub = wave >> 1, jb = wave & 1;
  // sums of a tile, and FP64 ones of the tiles before it; every column of gB2 and
  // gB3 is the same, a lane keeps register col % 16
  f32x16 gW2, gW3, gB2, gB3;
  float gV[8], loss;  // W4 (2), b4, W1 (4), b1
  double aW2[WALK ? 16 : 1], aW3[WALK ? 16 : 1], aB2 = 0.0, aB3 = 0.0, aV[8], aLoss = 0.0;
#pragma unroll
  for (int r = 0; WALK && r < 16; ++r) aW2[r] = aW3[r] = 0.0;
#pragma unroll
  for (int k = 0; k < 8; ++k) aV[k] = 0.0;
  const auto clear = [&]() {
#pragma unroll
    for (int r = 0; r < 16; ++r) gW2[r] = gW3[r] = gB2[r] = gB3[r] = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) gV[k] = 0.f;
    loss = 0.f;
  };
  clear();
  const int vu = t & 63, vq = t >> 6;  // unit and quarter of the samples in the vector sums
  __syncthreads();

  const long long tiles = (n + T - 1) / T;
  for (long long tile = blockIdx.x; tile < (WALK ? tiles : blockIdx.x + 1); tile += gridDim.x) {
    if (WALK && tile != blockIdx.x) {
#pragma unroll
      for (int r = 0; WALK && r < 16; ++r) {
        aW2[r] += double(gW2[r]);
        aW3[r] += double(gW3[r]);
      }
      aB2 += double(acc_at(gB2, col & 15));
      aB3 += double(acc_at(gB3, col & 15));
#pragma unroll
      for (int k = 0; k < 8; ++k) aV[k] += double(gV[k]);
      aLoss += double(loss);
      clear();
    }
    const long long g = tile * T + smp;
    const long long src = g < n ? (idx ? (long long)idx[g] : g) : 0;
    const Row4 x = g < n ? reinterpret_cast<const Row4*>(X)[src] : Row4{0.f, 0.f, 0.f, 0.f};
    const Row2 yt = g < n ? reinterpret_cast<const Row2*>(Yt)[src] : Row2{0.f, 0.f};
    if (half == 0) sX[smp] = make_float4(x.x, x.y, x.z, x.w);
    // forward; layer 1 on the FP32 matrix cores, half-wave h supplying inputs h and 2 + h
    f32x16 acc[2];
    bf16x4 bop[8];
    acc_bias(acc, sP + kCB1, half);
    {
      const float xk0 = half ? x.y : x.x, xk1 = half ? x.w : x.z;
#pragma unroll
      for (int ib = 0; ib < 2; ++ib) {
        const float* w1 = sP + kCW1 + (ib * 32 + col) * kMlpIn + half;
        acc[ib] = __builtin_amdgcn_mfma_f32_32x32x2f32(w1[0], xk0, acc[ib], 0, 0, 0);
        acc[ib] = __builtin_amdgcn_mfma_f32_32x32x2f32(w1[2], xk1, acc[ib], 0, 0, 0);
      }
    }
    const uint32_t m1 = acc_mask(acc);
    put_activation(acc, bop, sH[0], half, smp);
    acc_bias(acc, sP + kCB2, half);
    acc_product(acc, sW, bop, half, col);
    const uint32_t m2 = acc_mask(acc);
    put_activation(acc, bop, sH[1], half, smp);
    acc_bias(acc, sP + kCB3, half);
    acc_product(acc, sW + Hd * kWPad, bop, half, col);
    const uint32_t m3 = acc_mask(acc);
    // output layer, residual and dz3 = (W4^T dy) g'(z3)
    float dy[kMlpOut];
    {
      float y0 = 0.f, y1 = 0.f;
#pragma unroll
      for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int u = ib * 32 + mfma_row(r, half);
          const float h = act_f(acc[ib][r]);
          sF[u * kSPadF + smp] = h;
          y0 += sP[kCW4 + u] * h;
          y1 += sP[kCW4 + Hd + u] * h;
        }
      y0 = sP[kCB4 + 0] + (y0 + __shfl_xor(y0, 32, 64));
      y1 = sP[kCB4 + 1] + (y1 + __shfl_xor(y1, 32, 64));
      const float r0 = g < n ? y0 - tscale0 * yt.x : 0.f, r1 = g < n ? y1 - tscale1 * yt.y : 0.f;
      dy[0] = r0 * inv_n;
      dy[1] = r1 * inv_n;
      if (half == 0) {
        loss += 0.5f * r0 * r0 + 0.5f * r1 * r1;
        sDy[0][smp] = dy[0];
        sDy[1][smp] = dy[1];
      }
    }
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int u = ib * 32 + mfma_row(r, half);
        acc[ib][r] = sP[kCW4 + u] * dy[0] + sP[kCW4 + Hd + u] * dy[1];
      }
    bf16x4 term[3][8];
    if (mask_gradient(acc, m3))
      put_split<true>(acc, term, sDz, half, smp);
    else
      put_split<false>(acc, term, sDz, half, smp);
    // dz2 = (W3^T dz3) g'(z2), smallest terms first
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ib][r] = 0.f;
#pragma unroll
    for (int p = 2; p >= 0; --p) acc_product(acc, sWT + Hd * kWPad, term[p], half, col);
    const bool bad = mask_gradient(acc, m2);
    __syncthreads();
    // layer 3 and output layer gradients
    weight_gradient(gW3, gB3, jb == 0, sDz, sH[1], ub, jb, half, col);
#pragma unroll 8
    for (int i = 0; i < T / 4; ++i) {
      const int s = vq * (T / 4) + i;
      const float h = sF[vu * kSPadF + s], d0 = sDy[0][s], d1 = sDy[1][s];
      gV[0] += d0 * h;
      gV[1] += d1 * h;
      gV[2] += vu == 0 ? d0 : d1;
    }
    __syncthreads();
    if (bad)
      put_split<true>(acc, term, sDz, half, smp);
    else
      put_split<false>(acc, term, sDz, half, smp);
    // dz1 = (W2^T dz2) g'(z1)
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ib][r] = 0.f;
#pragma unroll
    for (int p = 2; p >= 0; --p) acc_product(acc, sWT, term[p], half, col);
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        sF[(ib * 32 + mfma_row(r, half)) * kSPadF + smp] = acc[ib][r] * float((m1 >> (ib * 16 + r)) & 1u);
    __syncthreads();
    // layer 2 and layer 1 gradients
    weight_gradient(gW2, gB2, jb == 0, sDz, sH[0], ub, jb, half, col);
#pragma unroll 8
    for (int i = 0; i < T / 4; ++i) {
      const int s = vq * (T / 4) + i;
      const float d = sF[vu * kSPadF + s];
      const float4 xs = sX[s];
      gV[3] += d * xs.x;
      gV[4] += d * xs.y;
      gV[5] += d * xs.z;
      gV[6] += d * xs.w;
      gV[7] += d;
    }
    __syncthreads();  // the next tile overwrites the buffers
  }

  float gb2 = acc_at(gB2, col & 15), gb3 = acc_at(gB3, col & 15);
  if (WALK) {
#pragma unroll
    for (int r = 0; WALK && r < 16; ++r) {
      gW2[r] = float(aW2[r] + double(gW2[r]));
      gW3[r] = float(aW3[r] + double(gW3[r]));
    }
    gb2 = float(aB2 + double(gb2));
    gb3 = float(aB3 + double(gb3));
#pragma unroll
    for (int k = 0; k < 8; ++k) gV[k] = float(aV[k] + double(gV[k]));
    loss = float(aLoss + double(loss));
  }
  float* out = part + (long long)blockIdx.x * (kMlpParams + 1);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int u = ub * 32 + mfma_row(r, half);
    out[kOffW3 + u * Hd + jb * 32 + col] = gW3[r];
    out[kOffW2 + u * Hd + jb * 32 + col] = gW2[r];
  }
  if (jb == 0 && col < 16) {
    const int u = ub * 32 + mfma_row(col, half);
    out[kOffB3 + u] = gb3;
    out[kOffB2 + u] = gb2;
  }
  // the quarters' vector sums and the waves' losses, added in order
  float* red = sF;  // [quarter][8][unit]
#pragma unroll
  for (int k = 0; k < 8; ++k) red[(vq * 8 + k) * 64 + vu] = gV[k];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) loss += __shfl_xor(loss, off, 64);
  if (lane == 0) sDy[0][wave] = loss;
  __syncthreads();
  if (t < 64) {
    float s[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      s[k] = red[k * 64 + t];
      for (int q = 1; q < 4; ++q) s[k] += red[(q * 8 + k) * 64 + t];
    }
    out[kOffW4 + t] = s[0];
    out[kOffW4 + Hd + t] = s[1];
    if (t < kMlpOut) out[kOffB4 + t] = s[2];
#pragma unroll
    for (int k = 0; k < kMlpIn; ++k) out[kOffW1 + t * kMlpIn + k] = s[3 + k];
    out[kOffB1 + t] = s[7];
    if (t == 0) out[kMlpParams] = (((sDy[0][0] + sDy[0][1]) + sDy[0][2]) + sDy[0][3]) * inv_n;
  }
}

// Sum of the partial gradients (and loss) over the training workgroups, in
// a fixed order. A workgroup owns 64 consecutive parameters (one per lane, so
// each partial row is read 256 bytes at a time); each of its waves sums one
// contiguous range of the partials, eight loads in flight, and the wave sums
// are added in wave order.
constexpr int kRedCols = 64, kRedWaves = 16;
__global__ void __launch_bounds__(kRedCols * kRedWaves)
mlp_reduce_kernel(const float* __restrict__ part, int nparts, float* __restrict__ grad, float* __restrict__ loss) {
  __shared__ double sp[kRedWaves][kRedCols];
  const int lane = (int)threadIdx.x % kRedCols, wv = (int)threadIdx.x / kRedCols;
  const int k = (int)blockIdx.x * kRedCols + lane;
  const int q = (nparts + kRedWaves - 1) / kRedWaves;
  const int p0 = min(nparts, wv * q), p1 = min(nparts, p0 + q);
  double s = 0.0;
  if (k <= kMlpParams) {
#pragma unroll 8
    for (int p = p0; p < p1; ++p) s += part[(long long)p * (kMlpParams + 1) + k];
  }
  sp[wv][lane] = s;
  __syncthreads();
  if (wv != 0 || k > kMlpParams) return;
  double t = 0.0;
  for (int w = 0; w < kRedWaves; ++w) t += sp[w][lane];
  if (k < kMlpParams) grad[k] = float(t);
  else if (loss) *loss = float(t);
}

// Adam (Kingma and Ba) on the FP32 master copy; the BF16 parameters the
// network reads are the master values rounded to nearest even.
__global__ void mlp_adam_kernel(float* __restrict__ master, uint16_t* __restrict__ w, float* __restrict__ m,
                                float* __restrict__ v, const float* __restrict__ g, float lr, float b1, float b2,
                                float eps, float c1, float c2) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= kMlpParams) return;
  const float gk = g[k];
  const float mk = b1 * m[k] + (1.f - b1) * gk;
  const float vk = b2 * v[k] + (1.f - b2) * gk * gk;
  m[k] = mk;
  v[k] = vk;
  const float wk = master[k] - lr * (mk / c1) / (sqrtf(vk / c2) + eps);
  master[k] = wk;
  w[k] = f32_to_bf16(wk);
}

// Column means and standard deviations of Y[n][ncol] (ncol <= 4): partial
// sums per workgroup, then a fixed-order final sum.
constexpr int kMomThreads = 256;
__global__ void __launch_bounds__(kMomThreads)
moments_partial_kernel(const float* __restrict__ Y, long long n, int ncol, double* __restrict__ part) {
  __shared__ double s1[kMomThreads][4], s2[kMomThreads][4];
  const int t = threadIdx.x;
  double a[4] = {0, 0, 0, 0}, b[4] = {0, 0, 0, 0};
  for (long long i = (long long)blockIdx.x * kMomThreads + t; i < n; i += (long long)gridDim.x * kMomThreads)
    for (int cc = 0; cc < ncol; ++cc) {
      const double y = Y[i * ncol + cc];
      a[cc] += y;
      b[cc] += y * y;
    }
  for (int cc = 0; cc < 4; ++cc) { s1[t][cc] = a[cc]; s2[t][cc] = b[cc]; }
  __syncthreads();
  for (int h = kMomThreads / 2; h > 0; h >>= 1) {
    if (t < h)
      for (int cc = 0; cc < 4; ++cc) { s1[t][cc] += s1[t + h][cc]; s2[t][cc] += s2[t + h][cc]; }
    __syncthreads();
  }
  if (t == 0)
    for (int cc = 0; cc < 4; ++cc) {
      part[blockIdx.x * 8 + cc] = s1[0][cc];
      part[blockIdx.x * 8 + 4 + cc] = s2[0][cc];
    }
}

__global__ void moments_final_kernel(const double* __restrict__ part, int nparts, long long n, int ncol,
                                     double* __restrict__ out) {
  const int cc = threadIdx.x;
  if (cc >= ncol) return;
  double a = 0.0, b = 0.0;
  for (int p = 0; p < nparts; ++p) { a += part[p * 8 + cc]; b += part[p * 8 + 4 + cc]; }
  const double mean = a / double(n);
  out[cc] = mean;
  out[ncol + cc] = sqrt(fmax(b / double(n) - mean * mean, 0.0));
}


}  // namespace
}  // namespace nsk

using namespace nsk;

namespace {

constexpr int kMomParts = 1024;

ClosureArgs nudge_args(const nsk_ctx* c, const nsk_closure_norm& q) {
  ClosureArgs a;
  std::memset(&a, 0, sizeof(a));
  for (int i = 0; i < c->np; ++i)
    for (int j = 0; j < c->np; ++j) a.D[i][j] = c->basis.D[i][j];
  a.s0 = q.s0; a.k0 = q.k0; a.s1 = q.s1; a.k1 = q.k1; a.k2 = q.k2; a.k3 = q.k3; a.g0 = q.g0;
  a.out_m = q.out_m; a.out_c = q.out_c;
  return a;
}

bool norm_ok(const nsk_closure_norm* q) {
  const float v[9] = {q->s0, q->k0, q->s1, q->k1, q->k2, q->k3, q->g0, q->out_m, q->out_c};
  for (float x : v)
    if (!std::isfinite(x)) return false;
  return q->g0 > 0.f;
}

template <int DIM, int NP>
int launch_nudge_t(nsk_ctx* c, const ClosureArgs& ca, const double* Ur, double relax, double inv_tau, double cmap,
                   float* X, float* Y) {
  using CS = ClosureShape<DIM, NP>;
  const unsigned blocks = (unsigned)((c->E + CS::EPB - 1) / CS::EPB);
  double* U = c->cur == 0 ? c->U : reinterpret_cast<double*>(c->work + c->off_U2);
  hipLaunchKernelGGL((nudge_kernel<DIM, NP>), dim3(blocks), dim3(kClosureThreads), 0, c->stream, U, Ur, mesh_args(c),
                     ca, relax, inv_tau, cmap, X, Y);
  return hipGetLastError() == hipSuccess ? NSK_OK : NSK_EHIP;
}

template <int DIM>
int launch_nudge_np(nsk_ctx* c, const ClosureArgs& ca, const double* Ur, double relax, double inv_tau, double cmap,
                    float* X, float* Y) {
  switch (c->np) {
    case 2: return launch_nudge_t<DIM, 2>(c, ca, Ur, relax, inv_tau, cmap, X, Y);
    case 3: return launch_nudge_t<DIM, 3>(c, ca, Ur, relax, inv_tau, cmap, X, Y);
    case 4: return launch_nudge_t<DIM, 4>(c, ca, Ur, relax, inv_tau, cmap, X, Y);
    case 5: return launch_nudge_t<DIM, 5>(c, ca, Ur, relax, inv_tau, cmap, X, Y);
    case 6: return launch_nudge_t<DIM, 6>(c, ca, Ur, relax, inv_tau, cmap, X, Y);
    case 7:
      if constexpr (DIM < 3) return launch_nudge_t<DIM, 7>(c, ca, Ur, relax, inv_tau, cmap, X, Y);
      break;
  }
  return NSK_EUNSUPPORTED;
}

// number of parameters whose BF16 exponent is all ones (infinite or NaN),
// as a double in *out; one workgroup
constexpr int kParamCheckThreads = 256;
__global__ void __launch_bounds__(kParamCheckThreads)
param_nonfinite_kernel(const uint16_t* __restrict__ w, int n, double* __restrict__ out) {
  __shared__ int red[kParamCheckThreads / 64];
  int cnt = 0;
  for (int i = threadIdx.x; i < n; i += kParamCheckThreads) cnt += (w[i] & 0x7F80u) == 0x7F80u ? 1 : 0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int k = 0; k < kParamCheckThreads / 64; ++k) t += red[k];
    *out = (double)t;
  }
}

bool same_mesh(const nsk_ctx* a, const nsk_ctx* b) {
  if (a->dim != b->dim || a->N != b->N || a->E != b->E || a->nvar != b->nvar) return false;
  for (int d = 0; d < 3; ++d)
    if (a->nel[d] != b->nel[d] || a->h2[d] != b->h2[d]) return false;
  return true;
}

// D2D copy of one context's state into another's, finished before return
// (the two contexts may be bound to different streams)
int copy_state(nsk_ctx* dst, nsk_ctx* src) {
  if (hipStreamSynchronize(src->stream) != hipSuccess) return NSK_EHIP;
  int rc = nsk_set_state(dst, src->U);
  if (rc) return rc;
  return hipStreamSynchronize(dst->stream) == hipSuccess ? NSK_OK : NSK_EHIP;
}

}  // namespace

extern "C" {

int nsk_closure_run(nsk_ctx* cl, nsk_ctx* ref, double dt, int nsteps, int ratio, int check_every,
                    double energy_tol, nsk_closure_report* report) {
  if (!cl || !ref || cl == ref || !report) return NSK_EINVAL;
  if (cl->par.closure != 1 || !cl->cl_w || ref->par.closure != 0) return NSK_EINVAL;
  if (cl->par.model != 0 || ref->par.model != 0 || !same_mesh(cl, ref)) return NSK_EINVAL;
  if (!(dt > 0.0) || !std::isfinite(dt) || nsteps < 0 || ratio < 1 || check_every < 1) return NSK_EINVAL;
  if (!std::isfinite(energy_tol)) return NSK_EINVAL;
  if (!cl->bound || !ref->bound) return NSK_EUNBOUND;
  std::memset(report, 0, sizeof(*report));
  // the parameters, counted on the device
  double* out = reinterpret_cast<double*>(cl->work + cl->off_out) + kDiagSlots;
  hipLaunchKernelGGL(param_nonfinite_kernel, dim3(1), dim3(kParamCheckThreads), 0, cl->stream, cl->cl_w,
                     kMlpParams, out);
  double bad = 0.0;
  if (hipGetLastError() != hipSuccess ||
      hipMemcpyAsync(&bad, out, sizeof(double), hipMemcpyDeviceToHost, cl->stream) != hipSuccess ||
      hipStreamSynchronize(cl->stream) != hipSuccess)
    return NSK_EHIP;
  nsk_diag d;
  int rc = nsk_diagnostics(cl, &d);
  if (rc) return rc;  // NSK_ENONPHYS: no state to start either run from
  report->e_start = report->e_last = d.e_total;
  rc = copy_state(ref, cl);
  if (rc) return rc;
  long long done = 0;
  int reason = bad > 0.0 ? NSK_CLOSURE_PARAMS : NSK_CLOSURE_KEPT;
  while (reason == NSK_CLOSURE_KEPT && done < nsteps) {
    const int n = (int)std::min<long long>(check_every, nsteps - done);
    rc = nsk_rk_step(cl, dt, n);
    if (rc) return rc;
    rc = nsk_diagnostics(cl, &d);  // waits for cl's stream
    if (rc == NSK_ENONPHYS) {
      reason = NSK_CLOSURE_NONPHYS;
    } else if (rc) {
      return rc;
    } else if (energy_tol >= 0.0 && d.e_total > report->e_start + energy_tol * std::fabs(report->e_start)) {
      reason = NSK_CLOSURE_ENERGY;
    } else {
      done += n;
      report->e_last = d.e_total;
      rc = copy_state(ref, cl);  // the last state that passed
      if (rc) return rc;
    }
  }
  report->closure_steps = done;
  report->reason = reason;
  if (reason == NSK_CLOSURE_KEPT) return NSK_OK;
  // the rest of the time on the large-alpha run, from the last state that passed
  report->fell_back = 1;
  long long left = (nsteps - done) * (long long)ratio;
  report->fallback_steps = left;
  const double dtr = dt / ratio;
  while (left > 0) {
    const int n = (int)std::min<long long>(left, 1 << 30);
    rc = nsk_rk_step(ref, dtr, n);
    if (rc) return rc;
    left -= n;
  }
  rc = nsk_diagnostics(ref, &d);
  if (rc) return rc;
  return copy_state(cl, ref);
}


int nsk_closure_set(nsk_ctx* c, const uint16_t* d_w_bf16, const nsk_closure_norm* norm, int every_stage) {
  if (!c || !d_w_bf16 || !norm || (every_stage != 0 && every_stage != 1)) return NSK_EINVAL;
  if ((reinterpret_cast<uintptr_t>(d_w_bf16) & 15) != 0) return NSK_EINVAL;  // staged 8 values at a time
  if (c->par.closure != 1 || !norm_ok(norm)) return NSK_EINVAL;
  c->cl_every_stage = every_stage;
  const float q[9] = {norm->s0, norm->k0, norm->s1, norm->k1, norm->k2, norm->k3, norm->g0, norm->out_m, norm->out_c};
  std::memcpy(c->cl_norm, q, sizeof(q));
  c->cl_w = d_w_bf16;
  return NSK_OK;
}

int nsk_closure_nudge(nsk_ctx* c, const nsk_closure_norm* norm, const double* d_Uref, double dt, double tau,
                      double cmap, float* d_X, float* d_Y) {
  if (!c || !norm || !d_Uref || !(tau > 0.0) || !(dt >= 0.0) || !std::isfinite(cmap)) return NSK_EINVAL;
  if (!norm_ok(norm)) return NSK_EINVAL;
  if (!c->bound) return NSK_EUNBOUND;
  const ClosureArgs ca = nudge_args(c, *norm);
  switch (c->dim) {
    case 1: return launch_nudge_np<1>(c, ca, d_Uref, dt / tau, 1.0 / tau, cmap, d_X, d_Y);
    case 2: return launch_nudge_np<2>(c, ca, d_Uref, dt / tau, 1.0 / tau, cmap, d_X, d_Y);
    case 3: return launch_nudge_np<3>(c, ca, d_Uref, dt / tau, 1.0 / tau, cmap, d_X, d_Y);
  }
  return NSK_EUNSUPPORTED;
}

int nsk_mlp_forward(const uint16_t* d_w, const float* d_X, long long n, float* d_Y, void* hip_stream) {
  if (!d_w || n < 0 || (n > 0 && (!d_X || !d_Y))) return NSK_EINVAL;
  if (((reinterpret_cast<uintptr_t>(d_X) | reinterpret_cast<uintptr_t>(d_w)) & 15) != 0) return NSK_EINVAL;
  if (n == 0) return NSK_OK;
  const long long blocks = (n + kClosureThreads - 1) / kClosureThreads;
  if (blocks > (1LL << 31) - 1) return NSK_EINVAL;
  hipLaunchKernelGGL(mlp_forward_kernel, dim3((unsigned)blocks), dim3(kClosureThreads), 0,
                     static_cast<hipStream_t>(hip_stream), d_w, d_X, n, d_Y);
  return hipGetLastError() == hipSuccess ? NSK_OK : NSK_EHIP;
}

size_t nsk_mlp_workspace_bytes(long long batch) {
  if (batch < 1) batch = 1;
  const size_t tiles = (size_t)((batch + kTrainTile - 1) / kTrainTile);
  const size_t grad = tiles * (size_t)(kMlpParams + 1) * sizeof(float);
  const size_t mom = (size_t)kMomParts * 8 * sizeof(double);
  return grad > mom ? grad : mom;
}

int nsk_mlp_loss_grad(const uint16_t* d_w, const float* d_X, const float* d_Y, const int* d_idx, long long n,
                      float tscale0, float tscale1, void* d_ws, float* d_grad, float* d_loss, void* hip_stream) {
  if (!d_w || !d_X || !d_Y || !d_ws || !d_grad || n < 1) return NSK_EINVAL;
  if (!std::isfinite(tscale0) || !std::isfinite(tscale1)) return NSK_EINVAL;
  if ((n + kTrainTile - 1) / kTrainTile > (1LL << 30)) return NSK_EINVAL;
  const int grid = (int)std::min<long long>((n + kTrainSamples - 1) / kTrainSamples, kTrainGrid);
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  float* part = static_cast<float*>(d_ws);
  const auto train = n > (long long)kTrainSamples * kTrainGrid ? mlp_train_kernel<true> : mlp_train_kernel<false>;
  hipLaunchKernelGGL(train, dim3((unsigned)grid), dim3(kTrainThreads), 0, s, d_w, d_X, d_Y, d_idx, n,
                     float(1.0 / double(n)), tscale0, tscale1, part);
  hipLaunchKernelGGL(mlp_reduce_kernel, dim3((kMlpParams + 1 + kRedCols - 1) / kRedCols), dim3(kRedCols * kRedWaves), 0,
                     s, part, grid, d_grad, d_loss);
  return hipGetLastError() == hipSuccess ? NSK_OK : NSK_EHIP;
}

int nsk_mlp_adam(float* d_master, uint16_t* d_w, float* d_m, float* d_v, const float* d_grad, int t, double lr,
                 double beta1, double beta2, double eps, void* hip_stream) {
  if (!d_master || !d_w || !d_m || !d_v || !d_grad || t < 1) return NSK_EINVAL;
  if (!(lr > 0.0) || !(beta1 >= 0.0 && beta1 < 1.0) || !(beta2 >= 0.0 && beta2 < 1.0) || !(eps > 0.0))
    return NSK_EINVAL;
  const double c1 = 1.0 - std::pow(beta1, t), c2 = 1.0 - std::pow(beta2, t);
  hipLaunchKernelGGL(mlp_adam_kernel, dim3((kMlpParams + 255) / 256), dim3(256), 0,
                     static_cast<hipStream_t>(hip_stream), d_master, d_w, d_m, d_v, d_grad, float(lr), float(beta1),
                     float(beta2), float(eps), float(c1), float(c2));
  return hipGetLastError() == hipSuccess ? NSK_OK : NSK_EHIP;
}

int nsk_mlp_moments(const float* d_Y, long long n, int ncol, void* d_ws, double* d_out, void* hip_stream) {
  if (!d_Y || n < 1 || ncol < 1 || ncol > 4 || !d_ws || !d_out) return NSK_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  long long blocks = (n + kMomThreads - 1) / kMomThreads;
  if (blocks > kMomParts) blocks = kMomParts;
  double* part = static_cast<double*>(d_ws);
  hipLaunchKernelGGL(moments_partial_kernel, dim3((unsigned)blocks), dim3(kMomThreads), 0, s, d_Y, n, ncol, part);
  hipLaunchKernelGGL(moments_final_kernel, dim3(1), dim3(64), 0, s, part, (int)blocks, n, ncol, d_out);
  return hipGetLastError() == hipSuccess ? NSK_OK : NSK_EHIP;
}

}  // extern "C"
