// Closure network for a coarse periodic 2D field: three periodic 3x3 convolutions
// 1 -> 32 -> 32 -> 1 channels with GELU between them (exact erf form).  Weights and
// activations are stored in bfloat16 and products accumulated in FP32; the 32 -> 32 layer
// runs on MFMA (bf16 x bf16 -> f32 forward; f32 x f32 -> f32 for its input cotangent and
// weight gradient).  The network is not part of the paper's method: its output is added to
// the explicit term F of the coarse problem, and its parameters receive gradients through
// the discrete adjoint like any parameter of F (equ:efficient_gradient).
//
// Layouts: images [B][H][W] (FP64 in and out); activations NHWC [B][H*W][32]; parameters as
// one FP64 vector in the order w1 (32x1x3x3), b1 (32), w2 (32x32x3x3), b2 (32), w3 (1x32x3x3),
// b3 (1), w[o][c][dy+1][dx+1] multiplying the input at (y + dy, x + dx) (periodic).
#include <hip/hip_runtime.h>
#include <math.h>

#include <functional>
#include <vector>

#include "cnn.h"
#include "sps_internal.h"

namespace sps {
namespace {

constexpr int CH = 32;                  // hidden channels
constexpr int NP1 = CH * 9, NP2 = CH * CH * 9, NP3 = CH * 9;
constexpr int OFF_W1 = 0, OFF_B1 = NP1, OFF_W2 = OFF_B1 + CH, OFF_B2 = OFF_W2 + NP2, OFF_W3 = OFF_B2 + CH,
              OFF_B3 = OFF_W3 + NP3, NPARAM = OFF_B3 + 1;
constexpr int NTC = 256;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct CnnDev {
  int B, H, W;
  const float* w1;     // [32][9]   bf16-rounded
  const float* b1;     // [32]
  const __bf16* w2r;   // [9][32 co][32 ci] bf16 (forward MFMA operand)
  const float* w2f;    // [9][32 co][32 ci] the same values in FP32
  const float* b2;     // [32]
  const float* w3;     // [32][9]   bf16-rounded
  const float* b3;     // [1]
  __bf16 *a0, *a1, *a2;   // a0: [B][HW]; a1, a2: [B][HW][32]
  float *dz1, *dz2;       // gelu' of the pre-activations z1, z2 [B][HW][32] (backward passes)
  float *g1, *g2;         // cotangents of z1, z2
};

__device__ __forceinline__ int nb(int p, int t, int H, int W) {
  // pixel index of the neighbour (y + dy, x + dx) of pixel p for tap t = (dy+1)*3 + (dx+1)
  const int y = p / W, x = p - y * W;
  const int dy = t / 3 - 1, dx = t % 3 - 1;
  int yy = y + dy, xx = x + dx;
  yy += (yy < 0) ? H : (yy >= H ? -H : 0);
  xx += (xx < 0) ? W : (xx >= W ? -W : 0);
  return yy * W + xx;
}
__device__ __forceinline__ int nb_t(int p, int t, int H, int W) { return nb(p, 8 - t, H, W); }   // (y - dy, x - dx)

// GELU z Phi(z) and its derivative, with e = erff(z / sqrt 2): the forward kernels of a backward pass, which have e for
// the activation, store the derivative in place of z (evaluated again from z, erff and expf were more than half the
// vector instructions of layer 3's backward), those of a forward pass neither.  At 65536 pixels: layers 1 and 2 8.1 and
// 10.4 us -> 6.9 and 8.2 in a forward pass, 9.2 and 12.5 in a backward pass, whose layer 3 takes 6.0 us, so 8.0, and
// layer 2's input cotangent 17.8, so 20.2.
__device__ __forceinline__ float gelu_e(float z) { return erff(z * 0.70710678118654752f); }
__device__ __forceinline__ float gelu_f(float z, float e) { return 0.5f * z * (1.0f + e); }
__device__ __forceinline__ float gelu_df(float z, float e) {
  return 0.5f * (1.0f + e) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// Block i of n as a block of pixels: the blocks of one XCD (i mod 8) take one contiguous part of them, in every
// kernel the same, so that the rows that neighbouring blocks, the nine taps and the next kernel read again are in
// that XCD's L2 (dealt out one by one, each L2 read every image).  At 65536 pixels: layer 2 11.4 -> 10.4 us, layer 3
// 6.0 -> 5.1, its backward 8.4 -> 8.0, layer 2's input cotangent 24.5 -> 20.3 (with its pre-activations loaded early).
__device__ __forceinline__ int slab(int i, int n) {
  const int xcd = i & 7, q = n >> 3, r = n & 7;
  return xcd * q + min(xcd, r) + (i >> 3);
}

// parameters (FP64) -> stored tables
__global__ void cnn_prepare(const double* th, float* w1, float* b1, __bf16* w2r, float* w2f, float* b2, float* w3,
                            float* b3) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  auto r16 = [](double v) { return (float)(__bf16)(float)v; };
  if (i < NP1) w1[i] = r16(th[OFF_W1 + i]);
  if (i < CH) {
    b1[i] = (float)th[OFF_B1 + i];
    b2[i] = (float)th[OFF_B2 + i];
  }
  if (i < NP2) {   // i = (co * 32 + ci) * 9 + t
    const int t = i % 9, ci = (i / 9) % CH, co = i / (9 * CH);
    const float v = r16(th[OFF_W2 + i]);
    w2r[(t * CH + co) * CH + ci] = (__bf16)v;
    w2f[(t * CH + co) * CH + ci] = v;
  }
  if (i < NP3) w3[i] = r16(th[OFF_W3 + i]);
  if (i == 0) b3[0] = (float)th[OFF_B3];
}

// ---------------------------------------------------------------------------- forward
// layer 1 (1 -> 32) and GELU: four lanes per pixel, eight channels each, so that a wave's 16-byte
// stores fill whole lines (one lane per pixel wrote 64 lines per store instruction).  Bound by the
// 192 bytes a pixel writes in a backward pass, 64 in a forward one: 15.3 -> 9.2 and 6.9 us at 65536 pixels.
constexpr int L1_PIX = NTC / 4;   // pixels per block
template <bool GRAD>
__global__ void __launch_bounds__(NTC) cnn_l1(CnnDev d, const double* x) {
  __shared__ float w[9 * CH];   // [t][c]
  __shared__ float bs[CH];
  for (int e = threadIdx.x; e < NP1; e += NTC) w[(e % 9) * CH + e / 9] = d.w1[e];
  if (threadIdx.x < CH) bs[threadIdx.x] = d.b1[threadIdx.x];
  __syncthreads();
  const int HW = d.H * d.W;
  const int g = slab(blockIdx.x, gridDim.x) * L1_PIX + (threadIdx.x >> 2), c0 = (threadIdx.x & 3) * 8;
  if (g >= d.B * HW) return;
  const int b = g / HW, p = g - b * HW;
  float v[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) v[t] = (float)(__bf16)(float)x[(long long)b * HW + nb(p, t, d.H, d.W)];
  if (c0 == 0) d.a0[g] = (__bf16)v[4];
  float z[8];
  bf16x8 a;
#pragma unroll
  for (int j = 0; j < 8; ++j) z[j] = bs[c0 + j];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int j = 0; j < 8; ++j) z[j] = fmaf(w[t * CH + c0 + j], v[t], z[j]);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float e = gelu_e(z[j]);
    a[j] = (__bf16)gelu_f(z[j], e);
    if (GRAD) z[j] = gelu_df(z[j], e);
  }
  if (GRAD) {
    float4* zo = reinterpret_cast<float4*>(d.dz1 + (long long)g * CH + c0);
    zo[0] = make_float4(z[0], z[1], z[2], z[3]);
    zo[1] = make_float4(z[4], z[5], z[6], z[7]);
  }
  *reinterpret_cast<bf16x8*>(d.a1 + (long long)g * CH + c0) = a;
}

// layer 2 (32 -> 32) and GELU on MFMA: each wave computes 32 pixels (a row segment) x 32
// output channels; K = 9 taps x 32 input channels in 18 steps of 16.  LDS: w2r.
template <bool GRAD>
__global__ void __launch_bounds__(NTC) cnn_l2(CnnDev d) {
  __shared__ __bf16 w[9 * CH * CH];
  for (int e = threadIdx.x; e < 9 * CH * CH / 8; e += NTC)
    reinterpret_cast<bf16x8*>(w)[e] = reinterpret_cast<const bf16x8*>(d.w2r)[e];
  __syncthreads();
  const int HW = d.H * d.W, lane = threadIdx.x & 63;
  const int tile = slab(blockIdx.x, gridDim.x) * (NTC / 64) + (threadIdx.x >> 6);   // 32-pixel tiles
  const int tiles_per_img = HW / 32;
  if (tile >= d.B * tiles_per_img) return;
  const int b = tile / tiles_per_img, p0 = (tile - b * tiles_per_img) * 32;
  const int row = lane & 31, half = lane >> 5;
  const int p = p0 + row;
  const __bf16* A = d.a1 + (long long)b * HW * CH;
  f32x16 acc = {};
#pragma unroll
  for (int s = 0; s < 18; ++s) {
    const int t = s >> 1, ci0 = (s & 1) * 16 + half * 8;
    const bf16x8 av = *reinterpret_cast<const bf16x8*>(A + (long long)nb(p, t, d.H, d.W) * CH + ci0);
    const bf16x8 bv = *reinterpret_cast<const bf16x8*>(w + (t * CH + row) * CH + ci0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc, 0, 0, 0);
  }
  // acc[r]: pixel p0 + 8 (r / 4) + 4 half + r % 4, channel `row`
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int pi = p0 + 8 * (r >> 2) + 4 * half + (r & 3);
    const float z = acc[r] + d.b2[row];
    const long long o = ((long long)b * HW + pi) * CH + row;
    const float e = gelu_e(z);
    d.a2[o] = (__bf16)gelu_f(z, e);
    if (GRAD) d.dz2[o] = gelu_df(z, e);
  }
}

// layer 3 (32 -> 1): one thread per pixel; y (FP64) = scale * output (+= when accumulate)
__global__ void __launch_bounds__(NTC) cnn_l3(CnnDev d, double* y, double scale, int accumulate) {
  const int HW = d.H * d.W;
  const int g = slab(blockIdx.x, gridDim.x) * NTC + threadIdx.x;
  if (g >= d.B * HW) return;
  const int b = g / HW, p = g - b * HW;
  float s = d.b3[0];
  for (int t = 0; t < 9; ++t) {
    const bf16x8* a8 = reinterpret_cast<const bf16x8*>(d.a2 + ((long long)b * HW + nb(p, t, d.H, d.W)) * CH);
#pragma unroll
    for (int c8 = 0; c8 < CH / 8; ++c8) {
      const bf16x8 a = a8[c8];
#pragma unroll
      for (int j = 0; j < 8; ++j) s = fmaf(d.w3[(c8 * 8 + j) * 9 + t], (float)a[j], s);
    }
  }
  const double v = scale * (double)s;
  y[g] = accumulate ? y[g] + v : v;
}

// ---------------------------------------------------------------------------- backward
// layer 3: g2 = (w3 conv^T ybar) * gelu'(z2); eight lanes per pixel, four channels each, so that
// the 16-byte loads and stores of a wave are contiguous.  Bound by the 256 bytes a pixel moves:
// 12.4 -> 6.0 us at 65536 pixels.
constexpr int L3B_PIX = NTC / 8;   // pixels per block
__global__ void __launch_bounds__(NTC) cnn_l3_back(CnnDev d, const double* yb) {
  __shared__ float w[9 * CH];   // [t][c]
  for (int e = threadIdx.x; e < NP3; e += NTC) w[(e % 9) * CH + e / 9] = d.w3[e];
  __syncthreads();
  const int HW = d.H * d.W;
  const int g = slab(blockIdx.x, gridDim.x) * L3B_PIX + (threadIdx.x >> 3), c0 = (threadIdx.x & 7) * 4;
  if (g >= d.B * HW) return;
  const int b = g / HW, p = g - b * HW;
  const float4 z = *reinterpret_cast<const float4*>(d.dz2 + (long long)g * CH + c0);
  float ys[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) ys[t] = (float)yb[(long long)b * HW + nb_t(p, t, d.H, d.W)];
  const float zz[4] = {z.x, z.y, z.z, z.w};
  float r[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < 9; ++t) s = fmaf(w[t * CH + c0 + j], ys[t], s);
    r[j] = s * zz[j];
  }
  *reinterpret_cast<float4*>(d.g2 + (long long)g * CH + c0) = make_float4(r[0], r[1], r[2], r[3]);
}

// layer 2 input cotangent on MFMA f32: g1[p][ci] = gelu'(z1) sum_{t, co} w2[co][ci][t] g2[p - d_t][co];
// each wave 32 pixels x 32 input channels, K = 9 x 32 in 144 steps of 2.
__global__ void __launch_bounds__(NTC) cnn_l2_back_input(CnnDev d) {
  __shared__ float w[9 * CH * CH];
  for (int e = threadIdx.x; e < 9 * CH * CH / 4; e += NTC)
    reinterpret_cast<float4*>(w)[e] = reinterpret_cast<const float4*>(d.w2f)[e];
  __syncthreads();
  const int HW = d.H * d.W, lane = threadIdx.x & 63;
  const int tile = slab(blockIdx.x, gridDim.x) * (NTC / 64) + (threadIdx.x >> 6);
  const int tiles_per_img = HW / 32;
  if (tile >= d.B * tiles_per_img) return;
  const int b = tile / tiles_per_img, p0 = (tile - b * tiles_per_img) * 32;
  const int row = lane & 31, half = lane >> 5;
  const float* G = d.g2 + (long long)b * HW * CH;
  f32x16 acc = {};
  // 16-byte loads: lane (pixel row, half) holds channels 8j + 4 half .. 8j + 4 half + 3, and
  // each of the four MFMAs pairs channel 8j + m (half 0) with 8j + 4 + m (half 1); a tap's loads are
  // issued before the MFMAs of the tap before it (31 -> 25 us at 65536 pixels)
  float4 nq[CH / 8];
  auto load = [&](int t) {
    const float4* Gt = reinterpret_cast<const float4*>(G + (long long)nb_t(p0 + row, t, d.H, d.W) * CH);
#pragma unroll
    for (int j = 0; j < CH / 8; ++j) nq[j] = Gt[2 * j + half];
  };
  load(0);
  float z[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = d.dz1[((long long)b * HW + p0 + 8 * (r >> 2) + 4 * half + (r & 3)) * CH + row];
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    float4 cq[CH / 8];
#pragma unroll
    for (int j = 0; j < CH / 8; ++j) cq[j] = nq[j];
    if (t < 8) load(t + 1);
#pragma unroll
    for (int j = 0; j < CH / 8; ++j) {
      const float4 q = cq[j];
      const float qa[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int co = 8 * j + 4 * half + m;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qa[m], w[(t * CH + co) * CH + row], acc, 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int pi = p0 + 8 * (r >> 2) + 4 * half + (r & 3);
    const long long o = ((long long)b * HW + pi) * CH + row;
    d.g1[o] = acc[r] * z[r];
  }
}

// layer 2 weight gradient on MFMA f32: dw2[co][ci][t] = sum_q g2[q][co] a1[q + d_t][ci].  One
// block per (tap, chunk of W2_CHUNK pixels), its four waves on a quarter of the chunk each,
// summed in a fixed order; the chunk's partial is written to (add == 0) or added to the FP64
// accumulator acc2[chunk][t][co][ci] (each slot has one owner: deterministic).
constexpr int W2_CHUNK = 512;
__device__ __forceinline__ void l2_back_weight(const CnnDev& d, int t, int chunk, double* acc2, int add,
                                               float (&red)[3][16][64]) {
  const int HW = d.H * d.W, lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q0 = chunk * W2_CHUNK + wv * (W2_CHUNK / 4);
  const int total = d.B * HW;
  const int row = lane & 31, half = lane >> 5;
  f32x16 acc = {};
  const int dy = t / 3 - 1, dx = t % 3 - 1;
  // acc[r]: co = 8 (r / 4) + 4 half + r % 4, ci = row
  double* o = acc2 + ((long long)chunk * 9 + t) * CH * CH + 4 * half * CH + row;
  double old[16];
  if (wv == 0 && add) {
#pragma unroll
    for (int r = 0; r < 16; ++r) old[r] = o[(8 * (r >> 2) + (r & 3)) * CH];
  }
  // a segment of 32 pixels lies within one image row (W is a multiple of 32), so its loads need no division or
  // branch, are all issued before its MFMAs and, but for the first and the last pixel,
  // which may be on the row's other end, have constant offsets (with an address a load, and the accumulator read at
  // the end, 27.5 us by itself at 65536 pixels, so 20.2; the MFMAs alone take 7.7)
  for (int s0 = 0; s0 < W2_CHUNK / 4; s0 += 32) {
    const int qs = q0 + s0;
    if (qs >= total) break;   // the total is a multiple of 32
    const int b = qs / HW, ps = qs - b * HW, y = ps / d.W, x0 = ps - y * d.W;
    const int yy = (y + dy < 0) ? d.H - 1 : (y + dy >= d.H ? 0 : y + dy);
    const float* gp = d.g2 + (long long)qs * CH + half * CH + row;
    const __bf16* ap = d.a1 + ((long long)b * HW + (long long)yy * d.W + x0 + dx) * CH + half * CH + row;
    const __bf16* a_first = (x0 + dx + half < 0) ? ap + d.W * CH : ap;
    const __bf16* a_last = ((x0 + 30 + dx + half >= d.W) ? ap - d.W * CH : ap) + 30 * CH;
    float av[16];
    __bf16 bv[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      av[k] = gp[2 * k * CH];
      bv[k] = *(k == 0 ? a_first : k == 15 ? a_last : ap + 2 * k * CH);
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[k], (float)bv[k], acc, 0, 0, 0);
  }
  if (wv > 0) {
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wv - 1][r][lane] = acc[r];
  }
  __syncthreads();
  if (wv != 0) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const double v = (double)(((acc[r] + red[0][r][lane]) + red[1][r][lane]) + red[2][r][lane]);
    o[(8 * (r >> 2) + (r & 3)) * CH] = add ? old[r] + v : v;
  }
}

// layer 1 input cotangent, one thread per pixel: xb = xscale sum_{t, c} w1[c][t] g1[p - d_t][c]
__device__ __forceinline__ void l1_back_input(const CnnDev& d, int block, double* xb, double xscale, int accumulate) {
  const int HW = d.H * d.W;
  const int g = block * NTC + threadIdx.x;
  if (g >= d.B * HW) return;
  const int b = g / HW, p = g - b * HW;
  float s = 0.f;
  for (int t = 0; t < 9; ++t) {
    const float4* G = reinterpret_cast<const float4*>(d.g1 + ((long long)b * HW + nb_t(p, t, d.H, d.W)) * CH);
#pragma unroll
    for (int c4 = 0; c4 < CH / 4; ++c4) {
      const float4 q = G[c4];
      s = fmaf(d.w1[(4 * c4 + 0) * 9 + t], q.x, s);
      s = fmaf(d.w1[(4 * c4 + 1) * 9 + t], q.y, s);
      s = fmaf(d.w1[(4 * c4 + 2) * 9 + t], q.z, s);
      s = fmaf(d.w1[(4 * c4 + 3) * 9 + t], q.w, s);
    }
  }
  const double v = xscale * (double)s;
  xb[g] = accumulate ? xb[g] + v : v;
}

// the small parameter gradients (dw1, db1, dw3, db3, db2) of one chunk of SW_CHUNK pixels, one wave: a lane per pair of
// channels and row of three taps, which share the loads of a0 and a2 as a window along the image row (a thread per
// tap read every vector nine times over, at 16 bytes a lane and pixel the L1's limit), the last 16 lanes for
// the bias of layer 2.  Sums are over the pixels in order; written to (add == 0) or added to the FP64
// accumulator acc1[chunk][SMALL] (one owner per slot).  SMALL layout: dw1 [c][t], db1 [c],
// dw3 [c][t], db3, db2 [c].
constexpr int SMALL = NP1 + CH + NP3 + 1 + CH;
constexpr int SW_CHUNK = 64;
constexpr int SW_LOADS = 8;       // pixels whose loads are issued at once
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void small_weight(const CnnDev& d, int chunk, const double* yb, double* acc1, int add) {
  const int HW = d.H * d.W, total = d.B * HW, lane = threadIdx.x & 63;
  const int c2 = lane & 15, part = lane >> 4, dy = (part == 3) ? 0 : part - 1;
  const int q0 = chunk * SW_CHUNK;
  double* o = acc1 + (long long)chunk * SMALL;
  double* o1 = o + 2 * c2 * 9 + 3 * part;
  double* o3 = o1 + NP1 + CH;
  double* ob = o + 2 * c2 + (part == 3 ? NP1 + CH + NP3 + 1 : NP1);
  double* oy = o + NP1 + CH + NP3;
  const bool taps = part < 3, bias = part == 0 || part == 3;
  double old1[2][3], old3[2][3], oldb[2], oldy = 0.0;
  if (add) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (taps) {
          old1[j][k] = o1[9 * j + k];
          old3[j][k] = o3[9 * j + k];
        }
      if (bias) oldb[j] = ob[j];
    }
    if (lane == 0) oldy = *oy;
  }
  float s1[2][3] = {}, s3[2][3] = {}, sb[2] = {}, sy = 0.f;
  // segments of 32 pixels lie within one image row (W is a multiple of 32): constant offsets but for the first and the
  // last pixel of the window, as in l2_back_weight
  for (int qs = q0; qs < q0 + SW_CHUNK && qs < total; qs += 32) {
    const int b = qs / HW, ps = qs - b * HW, y = ps / d.W, x0 = ps - y * d.W;
    const int yy = (y + dy < 0) ? d.H - 1 : (y + dy >= d.H ? 0 : y + dy);
    const long long n0 = (long long)b * HW + (long long)yy * d.W + x0 - 1;   // the window's first pixel
    const long long nf = n0 + (x0 == 0 ? d.W : 0), nl = n0 + 33 - (x0 + 32 >= d.W ? d.W : 0);
    const float* gp = (part == 3 ? d.g2 : d.g1) + (long long)qs * CH + 2 * c2;
    const __bf16* a2p = d.a2 + 2 * c2;
#pragma unroll
    for (int i0 = 0; i0 < 32; i0 += SW_LOADS) {
      float2 g[SW_LOADS];
      bf16x2 a2[SW_LOADS + 2];
      __bf16 a0[SW_LOADS + 2];
      double yv[SW_LOADS];
#pragma unroll
      for (int i = 0; i < SW_LOADS + 2; ++i) {
        const int e = i0 + i;
        a2[i] = *reinterpret_cast<const bf16x2*>(e == 0 ? a2p + nf * CH : e == 33 ? a2p + nl * CH : a2p + n0 * CH + e * CH);
        a0[i] = *(e == 0 ? d.a0 + nf : e == 33 ? d.a0 + nl : d.a0 + n0 + e);
      }
#pragma unroll
      for (int i = 0; i < SW_LOADS; ++i) {
        g[i] = *reinterpret_cast<const float2*>(gp + (i0 + i) * CH);
        yv[i] = yb[qs + i0 + i];
      }
#pragma unroll
      for (int i = 0; i < SW_LOADS; ++i) {
        const float yf = (float)yv[i];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const float a0v = (float)a0[i + k];
          s1[0][k] = fmaf(g[i].x, a0v, s1[0][k]);
          s1[1][k] = fmaf(g[i].y, a0v, s1[1][k]);
          s3[0][k] = fmaf(yf, (float)a2[i + k][0], s3[0][k]);
          s3[1][k] = fmaf(yf, (float)a2[i + k][1], s3[1][k]);
        }
        sb[0] += g[i].x;
        sb[1] += g[i].y;
        sy += yf;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (taps) {
        o1[9 * j + k] = add ? old1[j][k] + (double)s1[j][k] : (double)s1[j][k];
        o3[9 * j + k] = add ? old3[j][k] + (double)s3[j][k] : (double)s3[j][k];
      }
    if (bias) ob[j] = add ? oldb[j] + (double)sb[j] : (double)sb[j];
  }
  if (lane == 0) *oy = add ? oldy + (double)sy : (double)sy;
}

// Everything that follows g1 and g2, in one launch: the weight gradients of layer 2 (matrix instructions, nw blocks), the
// small gradients (chains of loads, four chunks a block) and the input cotangent of layer 1, none of which depends on
// another or fills the chip's units by itself: 28.1 + 26.0 + 10.1 us at 65536 pixels as three launches, now 34.5 (20.2,
// 10.3 and 9.7 by themselves).  At most 128 registers, so four blocks share a CU (178 and two blocks: 40.2 us).  The parts start at multiples of eight blocks, for slab().
__host__ __device__ constexpr int up8(int n) { return (n + 7) & ~7; }
__global__ void __launch_bounds__(NTC, 4) cnn_back_tail(CnnDev d, const double* yb, double* acc1, int n1, double* acc2, int n2,
                                                     int add, double* xb, double xscale, int accumulate) {
  __shared__ float red[3][16][64];
  const int nw = 9 * n2, ns = (n1 + 3) / 4;
  int i = blockIdx.x;
  if (i < up8(nw)) {
    if (i >= nw) return;
    i = slab(i, nw);
    l2_back_weight(d, i % 9, i / 9, acc2, add, red);
    return;
  }
  i -= up8(nw);
  if (i < up8(ns)) {
    if (i >= ns) return;
    const int chunk = 4 * slab(i, ns) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (chunk < n1) small_weight(d, chunk, yb, acc1, add);
    return;
  }
  i -= up8(ns);
  l1_back_input(d, slab(i, gridDim.x - up8(nw) - up8(ns)), xb, xscale, accumulate);
}

// Sums the FP64 partials over chunks in a fixed order and adds them to the parameter gradient.  A
// block takes 32 neighbouring slots (one line each of a chunk's row), its 32 groups of lanes every
// 32nd chunk, then the groups are added in order.  Bound by reading the partials once; one thread
// per parameter walking all chunks was a serial chain of up to 1024 strided loads (16 images of
// 64 x 64: 481 -> 7 us).
constexpr int RED_OUT = 32, RED_GRP = 32;
constexpr int RED_B1 = (SMALL + RED_OUT - 1) / RED_OUT;   // blocks of the small gradients
constexpr int RED_B2 = NP2 / RED_OUT;                      // blocks of the layer-2 weights
__global__ void __launch_bounds__(RED_OUT * RED_GRP) cnn_reduce(const double* acc1, int n1, const double* acc2, int n2,
                                                                double* th_bar) {
  __shared__ double red[RED_GRP][RED_OUT];
  const int j = threadIdx.x % RED_OUT, grp = threadIdx.x / RED_OUT;
  const bool small = blockIdx.x < RED_B1;
  const int slot = (small ? blockIdx.x : blockIdx.x - RED_B1) * RED_OUT + j;
  const int n = small ? n1 : n2, ld = small ? SMALL : NP2;
  const bool act = slot < ld;
  const double* p = (small ? acc1 : acc2) + (act ? slot : 0);
  double s = 0.0;
#pragma unroll 4
  for (int k = grp; k < n; k += RED_GRP) s += p[(long long)k * ld];
  red[grp][j] = s;
  __syncthreads();
  if (grp != 0 || !act) return;
  s = red[0][j];
  for (int q = 1; q < RED_GRP; ++q) s += red[q][j];
  int out;
  if (small) {   // dw1, db1, dw3, db3, db2
    out = slot < NP1 + CH ? OFF_W1 + slot
                          : (slot < NP1 + CH + NP3 + 1 ? OFF_W3 + slot - (NP1 + CH) : OFF_B2 + slot - (NP1 + CH + NP3 + 1));
  } else {       // [t][co][ci] -> (co * 32 + ci) * 9 + t
    const int t = slot / (CH * CH), cc = slot - t * CH * CH;
    out = OFF_W2 + cc * 9 + t;
  }
  th_bar[out] += s;
}

__global__ void cnn_zero(double* p, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

}  // namespace

// ---------------------------------------------------------------------------- host
struct Cnn::Impl {
  int B, H, W;
  hipStream_t s;
  DevArena arena;
  CnnDev d{};
  float *w1, *b1, *w2f, *b2, *w3, *b3;
  double *acc1, *acc2;
  __bf16* w2r;
  int n1, n2;   // chunks of the small and the layer-2 weight gradients
};

Cnn::Cnn(int batch, int H, int W, hipStream_t s) : p_(new Impl) {
  SPS_REQUIRE(batch >= 1 && H >= 3 && W >= 32 && W % 32 == 0, "closure images need W a multiple of 32");
  Impl& m = *p_;
  m.B = batch;
  m.H = H;
  m.W = W;
  m.s = s;
  const long long HW = (long long)H * W, n = batch * HW;
  m.w1 = m.arena.alloc<float>(NP1);
  m.b1 = m.arena.alloc<float>(CH);
  m.w2r = m.arena.alloc<__bf16>(NP2);
  m.w2f = m.arena.alloc<float>(NP2);
  m.b2 = m.arena.alloc<float>(CH);
  m.w3 = m.arena.alloc<float>(NP3);
  m.b3 = m.arena.alloc<float>(1);
  m.n1 = (int)((n + SW_CHUNK - 1) / SW_CHUNK);
  m.n2 = (int)((n + W2_CHUNK - 1) / W2_CHUNK);
  m.acc1 = m.arena.alloc<double>((size_t)m.n1 * SMALL);
  m.acc2 = m.arena.alloc<double>((size_t)m.n2 * 9 * CH * CH);
  CnnDev& d = m.d;
  d.B = batch;
  d.H = H;
  d.W = W;
  d.w1 = m.w1;
  d.b1 = m.b1;
  d.w2r = m.w2r;
  d.w2f = m.w2f;
  d.b2 = m.b2;
  d.w3 = m.w3;
  d.b3 = m.b3;
  d.a0 = m.arena.alloc<__bf16>(n);
  d.a1 = m.arena.alloc<__bf16>(n * CH);
  d.a2 = m.arena.alloc<__bf16>(n * CH);
  d.dz1 = m.arena.alloc<float>(n * CH);
  d.dz2 = m.arena.alloc<float>(n * CH);
  d.g1 = m.arena.alloc<float>(n * CH);
  d.g2 = m.arena.alloc<float>(n * CH);
}
Cnn::~Cnn() = default;

int Cnn::nparam() { return NPARAM; }

void Cnn::set_params(const double* theta_dev) {
  Impl& m = *p_;
  hipLaunchKernelGGL(cnn_prepare, dim3((NP2 + 255) / 256), dim3(256), 0, m.s, theta_dev, m.w1, m.b1, m.w2r, m.w2f,
                     m.b2, m.w3, m.b3);
  SPS_CHECK_LAUNCH();
}

void Cnn::forward(const double* x, double* y, double scale, bool accumulate) {
  Impl& m = *p_;
  const long long n = (long long)m.B * m.H * m.W;
  const int g1 = (int)((n + NTC - 1) / NTC), g2 = (int)((n / 32 + 3) / 4);
  hipLaunchKernelGGL(cnn_l1<false>, dim3((unsigned)((n + L1_PIX - 1) / L1_PIX)), dim3(NTC), 0, m.s, m.d, x);
  SPS_CHECK_LAUNCH();
  hipLaunchKernelGGL(cnn_l2<false>, dim3(g2), dim3(NTC), 0, m.s, m.d);
  SPS_CHECK_LAUNCH();
  hipLaunchKernelGGL(cnn_l3, dim3(g1), dim3(NTC), 0, m.s, m.d, y, scale, (int)accumulate);
  SPS_CHECK_LAUNCH();
}

void Cnn::backward(const double* x, const double* yb, double* xb, double xscale, bool accumulate, bool params, bool add) {
  Impl& m = *p_;
  const long long n = (long long)m.B * m.H * m.W;
  const int g1 = (int)((n + NTC - 1) / NTC), g2 = (int)((n / 32 + 3) / 4);
  // the forward activations of this input (recomputed: the adjoint sweep revisits states)
  hipLaunchKernelGGL(cnn_l1<true>, dim3((unsigned)((n + L1_PIX - 1) / L1_PIX)), dim3(NTC), 0, m.s, m.d, x);
  SPS_CHECK_LAUNCH();
  hipLaunchKernelGGL(cnn_l2<true>, dim3(g2), dim3(NTC), 0, m.s, m.d);
  SPS_CHECK_LAUNCH();
  hipLaunchKernelGGL(cnn_l3_back, dim3((unsigned)((n + L3B_PIX - 1) / L3B_PIX)), dim3(NTC), 0, m.s, m.d, yb);
  SPS_CHECK_LAUNCH();
  hipLaunchKernelGGL(cnn_l2_back_input, dim3(g2), dim3(NTC), 0, m.s, m.d);
  SPS_CHECK_LAUNCH();
  const auto tail = [&](int n1, int n2, int blocks) {
    hipLaunchKernelGGL(cnn_back_tail, dim3(up8(9 * n2) + up8((n1 + 3) / 4) + blocks), dim3(NTC), 0, m.s, m.d, yb, m.acc1, n1,
                       m.acc2, n2, (int)add, xb, xscale, (int)accumulate);
    SPS_CHECK_LAUNCH();
  };
  // a caller may have xb on yb, which the small gradients read
  const bool apart = std::less<const double*>()(xb, yb + n) && std::less<const double*>()(yb, xb + n);
  if (params && apart) tail(m.n1, m.n2, 0);
  tail(params && !apart ? m.n1 : 0, params && !apart ? m.n2 : 0, g1);
}

void Cnn::vjp(const double* x, const double* yb, double* xb, double xscale, bool accumulate, double* th_bar) {
  backward(x, yb, xb, xscale, accumulate, th_bar != nullptr, false);
  if (th_bar) grad_flush(th_bar);
}

void Cnn::vjp_accumulate(const double* x, const double* yb, double* xb, double xscale, bool accumulate) {
  backward(x, yb, xb, xscale, accumulate, true, true);
}

void Cnn::grad_reset() {
  Impl& m = *p_;
  const long long n1 = (long long)m.n1 * SMALL, n2 = (long long)m.n2 * 9 * CH * CH;
  hipLaunchKernelGGL(cnn_zero, dim3((unsigned)((n1 + 255) / 256)), dim3(256), 0, m.s, m.acc1, n1);
  SPS_CHECK_LAUNCH();
  hipLaunchKernelGGL(cnn_zero, dim3((unsigned)((n2 + 255) / 256)), dim3(256), 0, m.s, m.acc2, n2);
  SPS_CHECK_LAUNCH();
}

void Cnn::grad_flush(double* th_bar) {
  Impl& m = *p_;
  hipLaunchKernelGGL(cnn_reduce, dim3(RED_B1 + RED_B2), dim3(RED_OUT * RED_GRP), 0, m.s, m.acc1, m.n1, m.acc2, m.n2, th_bar);
  SPS_CHECK_LAUNCH();
}

}  // namespace sps
