// Tracking-initialisation network: a small CNN that proposes a pose
// correction from the render at the current pose and the observed RGB-D
// frame (both downsampled to 160 x 120, 8 channels: the render and the
// observed-minus-rendered residual). Four 3x3 stride-2 convolutions (64
// channels, ReLU), moment pooling (mean and first spatial moments) and a
// linear head to a 6-vector twist. Convolutions are implicit GEMMs on the gfx950 matrix
// cores (v_mfma_f32_16x16x32_bf16: BF16 operands, FP32 accumulation);
// activations and weights are BF16, master weights and the head FP32.
//
// Layouts: activations NHWC BF16 [B, H, W, C]; packed weights [64][KP] with
// K ordered (tap = 3 ky + kx, channel) and zero-padded to KP = 32 ceil(9 C / 32);
// transposed weights [C][9][64] for the data gradient.
//
// MFMA 16x16x32 operand layout (64 lanes): A[i][k] in lane i + 16 (k / 8),
// element k % 8; B[k][j] in lane j + 16 (k / 8), element k % 8; D[i][j] in
// lane j + 16 (i / 4), element i % 4.
#include <hip/hip_bf16.h>

#include <algorithm>

#include "gsr_internal.h"

namespace gsr {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

constexpr int kHeadIn = 3 * 64;     // pooled features: three moments of 64 channels
constexpr float kDiffGain = 4.f;    // scale of the observed-minus-rendered channels

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// float -> bf16 with round-to-nearest-even
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// The same by the hardware's conversion (v_cvt_pk_bf16_f32, two at a time).
__device__ __forceinline__ uint16_t cvt_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

__device__ __forceinline__ bf16x8 load8(const uint16_t* p) {
  const u16x8 v = *reinterpret_cast<const u16x8*>(p);
  return __builtin_bit_cast(bf16x8, v);
}

__device__ __forceinline__ bf16x8 zero8() {
  const u16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
  return __builtin_bit_cast(bf16x8, z);
}

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Up to this many output pixels the few-pixel forward kernel is the faster one
// (5120 pixels: 10 us against 13), beyond it the batched one (19200: 13 against
// 28): the few-pixel kernel reads all weights again for every 16 pixels.
constexpr int64_t kSmallPixels = 6144;

struct ConvShape {
  int B, H, W, C;   // input
  int OH, OW;       // output (stride 2, pad 1, 3x3)
  int KP;           // padded 9 * C
};

// A pixel of a layer's map.
struct Pix {
  int b, y, x;
};
__device__ __forceinline__ Pix pixel_of(int64_t m, int H, int W) {
  Pix p;
  p.b = (int)(m / ((int64_t)H * W));
  const int r = (int)(m - (int64_t)p.b * H * W);
  p.y = r / W;
  p.x = r - p.y * W;
  return p;
}

// The eight input values at (channel ci, tap) of output pixel p (zero outside
// the image or if !ok).
template <int C>
__device__ __forceinline__ bf16x8 tap8(const ConvShape& s, const uint16_t* __restrict__ in, const Pix& p, bool ok, int tap,
                                       int ci) {
  const int iy = 2 * p.y + tap / 3 - 1, ix = 2 * p.x + tap % 3 - 1;
  if (!ok || tap >= 9 || iy < 0 || iy >= s.H || ix < 0 || ix >= s.W) return zero8();
  return load8(in + (((int64_t)p.b * s.H + iy) * s.W + ix) * C + ci);
}

// Bias, ReLU and BF16 rounding of four neighbouring channels c0 .. c0 + 3 of a
// pixel (an accumulator's four elements): one 8-byte store.
__device__ __forceinline__ void store_relu4(uint16_t* __restrict__ out, int64_t m, int c0, const f32x4& acc,
                                            const float* __restrict__ bias) {
  typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
  u16x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = cvt_bf16(fmaxf(acc[e] + bias[c0 + e], 0.f));
  *reinterpret_cast<u16x4*>(out + m * 64 + c0) = v;
}

// ---- forward: out = relu(conv(in) + bias). The weights are the A operand
// (rows: output channels), the pixels B, so a lane ends with four neighbouring
// channels of one pixel. All three kernels add the products in the same order
// (K ascending, 32 at a time): a layer's result does not depend on which runs.

// First layer (8 input channels, K = 96: three steps). The whole weight matrix
// stays in the wave's registers while it walks pixel tiles of 16; bound by
// writing the output (64 samples: 39 MB; 40 -> 20 us).
__global__ __launch_bounds__(256) void k_conv8_fwd(ConvShape s, const uint16_t* __restrict__ in,
                                                 const uint16_t* __restrict__ wk, const float* __restrict__ bias,
                                                 uint16_t* __restrict__ out) {
  const int lane = threadIdx.x & 63, kg = lane >> 4, j = lane & 15;
  const int64_t M = (int64_t)s.B * s.OH * s.OW, tiles = (M + 15) / 16;
  bf16x8 w[3][4];
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) w[k][cb] = load8(wk + (int64_t)(16 * cb + j) * 96 + 32 * k + 8 * kg);
  for (int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); t < tiles; t += (int64_t)gridDim.x * 4) {
    const int64_t m = 16 * t + j;
    const bool ok = m < M;
    const Pix p = pixel_of(ok ? m : 0, s.OH, s.OW);
    bf16x8 x[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) x[k] = tap8<8>(s, in, p, ok, 4 * k + kg, 0);  // eight channels: one tap
    f32x4 acc[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) acc[cb] = mfma(w[k][cb], x[k], acc[cb]);
    if (ok)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) store_relu4(out, m, 16 * cb + 4 * kg, acc[cb], bias);
  }
}

// 64 input channels, few pixels (a single sample): 16 pixels per workgroup, 16
// output channels per wave, every load of the 18 steps issued before the first
// product, so the layer takes about one round trip to memory (one sample, the
// three layers: 24 us -> 5.4 to 7.3 us each).
__global__ __launch_bounds__(256) void k_conv64_fwd_small(ConvShape s, const uint16_t* __restrict__ in,
                                                        const uint16_t* __restrict__ wk,
                                                        const float* __restrict__ bias, uint16_t* __restrict__ out) {
  const int lane = threadIdx.x & 63, kg = lane >> 4, j = lane & 15, c0 = 16 * (threadIdx.x >> 6);
  const int64_t M = (int64_t)s.B * s.OH * s.OW, m = (int64_t)blockIdx.x * 16 + j;
  const bool ok = m < M;
  const Pix p = pixel_of(ok ? m : 0, s.OH, s.OW);
  bf16x8 w[18], x[18];
#pragma unroll
  for (int k = 0; k < 18; ++k) {
    w[k] = load8(wk + (int64_t)(c0 + j) * 576 + 32 * k + 8 * kg);
    x[k] = tap8<64>(s, in, p, ok, k / 2, 32 * (k & 1) + 8 * kg);
  }
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 18; ++k) acc = mfma(w[k], x[k], acc);
  if (ok) store_relu4(out, m, c0 + 4 * kg, acc, bias);
}

// One tap's 64 x 64 weights in LDS, rows padded to 72 values (16-byte reads of
// 16 rows touch every bank once). A row lies `stride` values after the last.
struct TapWeights {
  __align__(16) uint16_t w[64 * 72];
};
struct TapRegs {
  u16x8 v[2];
};
__device__ __forceinline__ TapRegs tap_fetch(const uint16_t* __restrict__ w, int stride) {
  const uint16_t* p = w + (int64_t)(threadIdx.x >> 2) * stride + 16 * (threadIdx.x & 3);
  TapRegs r;
  r.v[0] = *reinterpret_cast<const u16x8*>(p);
  r.v[1] = *reinterpret_cast<const u16x8*>(p + 8);
  return r;
}
__device__ __forceinline__ void tap_put(TapWeights& t, const TapRegs& r) {
  uint16_t* p = t.w + (threadIdx.x >> 2) * 72 + 16 * (threadIdx.x & 3);
  *reinterpret_cast<u16x8*>(p) = r.v[0];
  *reinterpret_cast<u16x8*>(p + 8) = r.v[1];
}
// acc[pt][cb] += weights (64 rows) times the tap's two steps of each pixel tile
template <int PT>
__device__ __forceinline__ void tap_products(const TapWeights& t, const bf16x8 (&x)[PT][2], f32x4 (&acc)[PT][4]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const bf16x8 w = load8(t.w + (16 * cb + (lane & 15)) * 72 + 32 * k + 8 * (lane >> 4));
#pragma unroll
      for (int pt = 0; pt < PT; ++pt) acc[pt][cb] = mfma(w, x[pt][k], acc[pt][cb]);
    }
}

constexpr int kPixTiles = 2;  // pixel tiles of 16 per wave in the batched kernels

// 64 input channels, many pixels: 128 pixels per workgroup; each tap's weights
// go through LDS (two buffers) and serve all four waves, the next tap's
// weights and pixels are in flight meanwhile. Bound by the input's reads (nine
// per value, out of the caches): 64 samples at 60x80, 58 -> 21 us.
__global__ __launch_bounds__(256) void k_conv64_fwd(ConvShape s, const uint16_t* __restrict__ in,
                                                  const uint16_t* __restrict__ wk, const float* __restrict__ bias,
                                                  uint16_t* __restrict__ out) {
  constexpr int PT = kPixTiles;
  __shared__ TapWeights sw[2];
  const int lane = threadIdx.x & 63, kg = lane >> 4, j = lane & 15;
  const int64_t M = (int64_t)s.B * s.OH * s.OW;
  int64_t m[PT];
  Pix p[PT];
#pragma unroll
  for (int pt = 0; pt < PT; ++pt) {
    m[pt] = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * (16 * PT) + 16 * pt + j;
    p[pt] = pixel_of(m[pt] < M ? m[pt] : 0, s.OH, s.OW);
  }
  auto pixels = [&](int tap, bf16x8 (&x)[PT][2]) {
#pragma unroll
    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
      for (int k = 0; k < 2; ++k) x[pt][k] = tap8<64>(s, in, p[pt], m[pt] < M, tap, 32 * k + 8 * kg);
  };
  f32x4 acc[PT][4];
#pragma unroll
  for (int pt = 0; pt < PT; ++pt)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[pt][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  TapRegs wr = tap_fetch(wk, 576);
  bf16x8 x[2][PT][2];
  pixels(0, x[0]);
#pragma unroll
  for (int tap = 0; tap < 9; ++tap) {
    tap_put(sw[tap & 1], wr);
    if (tap < 8) {
      wr = tap_fetch(wk + 64 * (tap + 1), 576);
      pixels(tap + 1, x[(tap + 1) & 1]);
    }
    __syncthreads();  // (the other buffer's readers passed the last barrier)
    tap_products<PT>(sw[tap & 1], x[tap & 1], acc);
  }
#pragma unroll
  for (int pt = 0; pt < PT; ++pt)
    if (m[pt] < M)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) store_relu4(out, m[pt], 16 * cb + 4 * kg, acc[pt][cb], bias);
}

// ---- data gradient: din = (conv^T dout) * [in > 0] (the ReLU mask of the
// previous layer, whose output is this layer's input), 64 channels. With
// stride 2 an input pixel of parity (y & 1, x & 1) meets only the taps whose
// offsets have the other parity: 1, 2, 2 or 4 of the nine. Each of the four
// parities (grid.y) is a GEMM over its own taps, in ascending order; the other
// taps' products, all zero, are left out. Bound by reading the mask and
// writing the gradient (64 samples at 60x80: 79 MB; 210 -> 32 us).
__global__ __launch_bounds__(256) void k_conv64_bwd_data(ConvShape s, const uint16_t* __restrict__ dout,
                                                       const uint16_t* __restrict__ wt,
                                                       const uint16_t* __restrict__ in, uint16_t* __restrict__ din) {
  constexpr int PT = kPixTiles;
  __shared__ TapWeights sw[2];
  const int lane = threadIdx.x & 63, kg = lane >> 4, j = lane & 15;
  const int py = blockIdx.y >> 1, px = blockIdx.y & 1;
  const int hh = (s.H - py + 1) / 2, ww = (s.W - px + 1) / 2;  // pixels of this parity
  const int64_t M = (int64_t)s.B * hh * ww;
  if ((int64_t)blockIdx.x * (64 * PT) >= M) return;  // uniform
  const int ny = 1 + py, nx = 1 + px;  // taps per axis: 1 for an even coordinate, 0 and 2 for an odd one
  int64_t m[PT];
  Pix p[PT];
#pragma unroll
  for (int pt = 0; pt < PT; ++pt) {
    m[pt] = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * (16 * PT) + 16 * pt + j;
    p[pt] = pixel_of(m[pt] < M ? m[pt] : 0, hh, ww);
  }
  auto tap_y = [&](int t) { return py ? 2 * (t / nx) : 1; };
  auto tap_x = [&](int t) { return px ? 2 * (t % nx) : 1; };
  auto pixels = [&](int t, bf16x8 (&x)[PT][2]) {
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
      const int oy = (2 * p[pt].y + py + 1 - tap_y(t)) >> 1, ox = (2 * p[pt].x + px + 1 - tap_x(t)) >> 1;
      const bool ok = m[pt] < M && oy < s.OH && ox < s.OW;
#pragma unroll
      for (int k = 0; k < 2; ++k)
        x[pt][k] = ok ? load8(dout + (((int64_t)p[pt].b * s.OH + oy) * s.OW + ox) * 64 + 32 * k + 8 * kg) : zero8();
    }
  };
  auto weights = [&](int t) { return tap_fetch(wt + 64 * (3 * tap_y(t) + tap_x(t)), 9 * 64); };
  f32x4 acc[PT][4];
#pragma unroll
  for (int pt = 0; pt < PT; ++pt)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[pt][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nt = ny * nx;
  TapRegs wr = weights(0);
  bf16x8 x[2][PT][2];
  pixels(0, x[0]);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    if (t >= nt) break;  // uniform
    tap_put(sw[t & 1], wr);
    if (t + 1 < nt) {
      wr = weights(t + 1);
      pixels(t + 1, x[(t + 1) & 1]);
    }
    __syncthreads();
    tap_products<PT>(sw[t & 1], x[t & 1], acc);
  }
  typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int pt = 0; pt < PT; ++pt) {
    if (m[pt] >= M) continue;
    const int64_t o = (((int64_t)p[pt].b * s.H + 2 * p[pt].y + py) * s.W + 2 * p[pt].x + px) * 64 + 4 * kg;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const u16x4 a = *reinterpret_cast<const u16x4*>(in + o + 16 * cb);
      u16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = bf2f(a[e]) > 0.f ? cvt_bf16(acc[pt][cb][e]) : (uint16_t)0;
      *reinterpret_cast<u16x4*>(din + o + 16 * cb) = v;
    }
  }
}

// ---- weight and bias gradients: dW[co][kk] += sum_m dy[m][co] im2col(in)[m][kk],
// db[co] += sum_m dy[m][co]. The contraction runs over pixels, while memory
// holds a pixel's channels side by side: a thread reads eight pixels x eight
// channels (16-byte loads), transposes them in registers (32 byte permutes) and
// writes eight rows of eight pixels to LDS, where both operands then lie as
// the matrix instruction wants them. Chunks of 128 pixels (grid-stride over
// grid.y), the next one's loads in flight during the products; one atomic add
// per output element at the end.
// C = 64: a workgroup owns one tap's 64 columns (grid.x = tap); the tap in the
// middle also sums dy against a column of ones (the bias). C = 8: one
// workgroup owns all 72 columns, the 73rd being the ones.
// Bound by the loads (dy once per tap, out of the caches); before, 16-bit
// transposed stores, scalar loads, 128 workgroups for the first layer and a
// kernel for the bias: first layer, 64 samples: 650 + 94 -> 50 us, all four
// layers 885 + 220 -> 120 us.
constexpr int kWPix = 128, kWRow = kWPix + 8;  // row stride 272 bytes: 16 rows' 16-byte reads touch every bank once

// rows[r] = the eight pixels' values of channel r
__device__ __forceinline__ void transpose8(const u16x8 (&px)[8], u16x8 (&rows)[8]) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 in[8], out[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) in[e] = __builtin_bit_cast(u32x4, px[e]);
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      out[2 * d][q] = __builtin_amdgcn_perm(in[2 * q + 1][d], in[2 * q][d], 0x05040100u);      // low halves
      out[2 * d + 1][q] = __builtin_amdgcn_perm(in[2 * q + 1][d], in[2 * q][d], 0x07060302u);  // high halves
    }
#pragma unroll
  for (int r = 0; r < 8; ++r) rows[r] = __builtin_bit_cast(u16x8, out[r]);
}

template <int C>
__global__ __launch_bounds__(256) void k_conv_bwd_weight(ConvShape s, const uint16_t* __restrict__ dy,
                                                       const uint16_t* __restrict__ in, float* __restrict__ dw,
                                                       float* __restrict__ db) {
  constexpr int NJ = C == 8 ? 5 : 4;                // column tiles of 16
  constexpr int kTasks = 16 * (8 + (C == 8 ? 9 : 8));  // eight pixels x (eight blocks of dy's channels, then of the columns)
  constexpr int kSlots = (kTasks + 255) / 256;
  __shared__ __align__(16) uint16_t sd[64 * kWRow];       // [co][pixel]
  __shared__ __align__(16) uint16_t sa[16 * NJ * kWRow];  // [column][pixel]
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, j = lane & 15, kg = lane >> 4;
  const int64_t M = (int64_t)s.B * s.OH * s.OW;
  if (C == 8)  // the column of ones and seven of zeros; never written again
    for (int i = tid; i < 8 * kWRow; i += 256) sa[72 * kWRow + i] = i < kWRow ? (uint16_t)0x3f80 : (uint16_t)0;
  u16x8 v[kSlots][8];
  auto fetch = [&](int64_t p0) {
#pragma unroll
    for (int sl = 0; sl < kSlots; ++sl) {
      const int task = tid + 256 * sl;
      if (task >= kTasks) continue;
      const bool is_dy = task < 128;
      const int64_t m0 = p0 + 8 * (is_dy ? task >> 3 : (task - 128) % 16);
      const int blk = is_dy ? task & 7 : (task - 128) / 16;
      if (is_dy) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          v[sl][e] = m0 + e < M ? *reinterpret_cast<const u16x8*>(dy + (m0 + e) * 64 + 8 * blk) : u16x8{};
      } else {
        Pix p = pixel_of(m0 < M ? m0 : 0, s.OH, s.OW);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const bf16x8 t = C == 8 ? tap8<8>(s, in, p, m0 + e < M, blk, 0)
                                  : tap8<64>(s, in, p, m0 + e < M, (int)blockIdx.x, 8 * blk);
          v[sl][e] = __builtin_bit_cast(u16x8, t);
          if (++p.x == s.OW) {
            p.x = 0;
            if (++p.y == s.OH) {
              p.y = 0;
              ++p.b;
            }
          }
        }
      }
    }
  };
  f32x4 acc[NJ], accb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int nj = 0; nj < NJ; ++nj) acc[nj] = f32x4{0.f, 0.f, 0.f, 0.f};
  const u16x8 one8 = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
  const bf16x8 ones = __builtin_bit_cast(bf16x8, one8);
  const bool bias = C == 64 && blockIdx.x == 4;
  fetch((int64_t)blockIdx.y * kWPix);
  for (int64_t p0 = (int64_t)blockIdx.y * kWPix; p0 < M; p0 += (int64_t)gridDim.y * kWPix) {
    __syncthreads();  // the last chunk's products are done
#pragma unroll
    for (int sl = 0; sl < kSlots; ++sl) {
      const int task = tid + 256 * sl;
      if (task >= kTasks) continue;
      const bool is_dy = task < 128;
      const int pb = is_dy ? task >> 3 : (task - 128) % 16, blk = is_dy ? task & 7 : (task - 128) / 16;
      uint16_t* dst = (is_dy ? sd : sa) + 8 * blk * kWRow + 8 * pb;
      u16x8 rows[8];
      transpose8(v[sl], rows);
#pragma unroll
      for (int r = 0; r < 8; ++r) *reinterpret_cast<u16x8*>(dst + r * kWRow) = rows[r];
    }
    __syncthreads();
    const int64_t next = p0 + (int64_t)gridDim.y * kWPix;
    if (next < M) fetch(next);
    // wave wv: rows co = 16 wv + i, all columns
#pragma unroll
    for (int k0 = 0; k0 < kWPix; k0 += 32) {
      const bf16x8 a = load8(sd + (16 * wv + j) * kWRow + k0 + 8 * kg);
#pragma unroll
      for (int nj = 0; nj < NJ; ++nj) acc[nj] = mfma(a, load8(sa + (16 * nj + j) * kWRow + k0 + 8 * kg), acc[nj]);
      if (bias) accb = mfma(a, ones, accb);
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int co = 16 * wv + 4 * kg + e;
#pragma unroll
    for (int nj = 0; nj < NJ; ++nj) {
      const int col = 16 * nj + j;
      if (C == 64) atomicAdd(&dw[(int64_t)co * 576 + 64 * blockIdx.x + col], acc[nj][e]);
      else if (col < 72) atomicAdd(&dw[(int64_t)co * 96 + col], acc[nj][e]);
      else if (col == 72) atomicAdd(&db[co], acc[nj][e]);
    }
    if (bias && j == 0) atomicAdd(&db[co], accb[e]);
  }
}

// Head. Moment pooling over the last feature map (OH x OW pixels): for each
// channel c, pool[b][k][c] = (1/npix) sum_p m_k(p) act[b][p][c] with m_0 = 1,
// m_1 = x^(p), m_2 = y^(p), x^ = (2 x + 1) / OW - 1 and y^ = (2 y + 1) / OH - 1
// (pixel centres mapped to (-1, 1)); out[b] = Wfc pool[b] + bfc over the 192
// pooled values (k major). The first moments keep where features sit, which a
// plain average cancels (a forward motion or a roll moves image content
// radially or around the centre, with zero mean displacement).
// One workgroup per sample: four waves share the pixels, one lane per channel.
__device__ __forceinline__ float moment_x(int p, int OW) { return (2.f * (float)(p % OW) + 1.f) / (float)OW - 1.f; }
__device__ __forceinline__ float moment_y(int p, int OW, int OH) {
  return (2.f * (float)(p / OW) + 1.f) / (float)OH - 1.f;
}

__global__ __launch_bounds__(256) void k_head_fwd(const uint16_t* __restrict__ act, int OH, int OW,
                                                const float* __restrict__ wfc, const float* __restrict__ bfc,
                                                float* __restrict__ pool, float* __restrict__ out) {
  const int b = blockIdx.x, c = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int npix = OH * OW;
  float s0 = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll 4
  for (int p = w; p < npix; p += 4) {
    const float v = bf2f(act[((int64_t)b * npix + p) * 64 + c]);
    s0 += v;
    s1 += v * moment_x(p, OW);
    s2 += v * moment_y(p, OW, OH);
  }
  __shared__ float part[4][kHeadIn], sp[kHeadIn];
  part[w][c] = s0;
  part[w][64 + c] = s1;
  part[w][128 + c] = s2;
  __syncthreads();
  const float inv = 1.f / (float)npix;
  for (int i = threadIdx.x; i < kHeadIn; i += 256) {
    sp[i] = (part[0][i] + part[1][i] + part[2][i] + part[3][i]) * inv;
    pool[b * kHeadIn + i] = sp[i];
  }
  __syncthreads();
  for (int o = w; o < 6; o += 4) {
    const float t = wave_sum_all(wfc[o * kHeadIn + c] * sp[c] + wfc[o * kHeadIn + 64 + c] * sp[64 + c] +
                                 wfc[o * kHeadIn + 128 + c] * sp[128 + c]);
    if (c == 0) out[b * 6 + o] = bfc[o] + t;
  }
}

// Loss L = 1/(2B) sum ((out - label) / scale)^2, its gradient, the head's
// gradients (atomic over samples), and dL/dact4[p][c] = (1/npix)
// sum_k m_k(p) dpool[k][c] * [act > 0] with dpool = Wfc^T dout.
__global__ __launch_bounds__(256) void k_head_bwd(const float* __restrict__ out, const float* __restrict__ label,
                                                const float* __restrict__ scale, int B, const float* __restrict__ pool,
                                                const float* __restrict__ wfc, const uint16_t* __restrict__ act,
                                                int OH, int OW, const float* __restrict__ dout_in,
                                                float* __restrict__ dwfc, float* __restrict__ dbfc,
                                                uint16_t* __restrict__ dact, float* __restrict__ loss) {
  const int b = blockIdx.x, c = threadIdx.x & 63, w = threadIdx.x >> 6, t = threadIdx.x;
  const int npix = OH * OW;
  __shared__ float g[6];
  if (t < 6) {
    float d;
    if (dout_in) {
      d = dout_in[b * 6 + t];
    } else {
      const float r = (out[b * 6 + t] - label[b * 6 + t]) / scale[t];
      d = r / scale[t] / (float)B;
      atomicAdd(loss, 0.5f * r * r / (float)B);
    }
    g[t] = d;
    atomicAdd(&dbfc[t], d);
  }
  __syncthreads();
  float dp[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int j = 0; j < 6; ++j) dp[k] += wfc[j * kHeadIn + 64 * k + c] * g[j];
  for (int i = t; i < 6 * kHeadIn; i += 256) atomicAdd(&dwfc[i], g[i / kHeadIn] * pool[b * kHeadIn + i % kHeadIn]);
  const float inv = 1.f / (float)npix;
#pragma unroll 4
  for (int p = w; p < npix; p += 4) {
    const int64_t o = ((int64_t)b * npix + p) * 64 + c;
    const float d = (dp[0] + moment_x(p, OW) * dp[1] + moment_y(p, OW, OH) * dp[2]) * inv;
    dact[o] = bf2f(act[o]) > 0.f ? f2bf(d) : (uint16_t)0;
  }
}

// Master FP32 packed weights [64][KP] of every layer (grid.y) -> BF16 packed
// copy and BF16 transposed copy [C][9][64] for the data gradient.
__global__ void k_cast_weights(CastWeights a) {
  const int l = blockIdx.y, C = a.C[l], KP = ((9 * C + 31) / 32) * 32;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 64 * KP) return;
  const int co = i / KP, kk = i - co * KP;
  const uint16_t v = f2bf(a.w[l][i]);
  a.wk[l][i] = v;
  if (kk < 9 * C) {
    const int tap = kk / C, ci = kk - tap * C;
    a.wt[l][((int64_t)ci * 9 + tap) * 64 + co] = v;
  }
}

// Input packing: f x f average pooling of the rendered and observed RGB-D
// frames into 8 BF16 channels: the render (r, g, b, depth * depth_scale) and
// the observation minus the render, times kDiffGain (the residual, formed in
// FP32 before rounding to BF16, where a few-millimetre depth residual would
// otherwise fall below the precision of depths of metres).
// F = f, or 0 for any f: with F known the loads of a pixel's block are issued
// together instead of one after the other (640x480: 9.8 -> 5 us). From call to
// call 5 and 6 take the same 6.7 us either way; 7 would go from 9.8 to 6.5 and 8
// from 11.7 to 9.3, but no camera here is 1120 or 1280 pixels wide.
template <int F>
__global__ __launch_bounds__(64) void k_pack_input(const float* __restrict__ rc, const float* __restrict__ rd,
                                                 const float* __restrict__ oc, const float* __restrict__ od, int H, int W,
                                                 int f_any, float depth_scale, uint16_t* __restrict__ out) {
  const int f = F ? F : f_any;
  const int OW = W / f, OH = H / f;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= OW * OH) return;
  const int y = i / OW, x = i - y * OW;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const int64_t P = (int64_t)H * W;
#pragma unroll
  for (int dy = 0; dy < f; ++dy)
#pragma unroll
    for (int dx = 0; dx < f; ++dx) {
      const int64_t p = (int64_t)(y * f + dy) * W + (x * f + dx);
      acc[0] += rc[p];
      acc[1] += rc[P + p];
      acc[2] += rc[2 * P + p];
      acc[3] += rd[p] * depth_scale;
      acc[4] += oc[p] - rc[p];
      acc[5] += oc[P + p] - rc[P + p];
      acc[6] += oc[2 * P + p] - rc[2 * P + p];
      acc[7] += (od[p] - rd[p]) * depth_scale;
    }
  const float inv = 1.f / (float)(f * f);
  u16x8 v;
#pragma unroll
  for (int c = 0; c < 8; ++c) v[c] = f2bf(acc[c] * inv * (c < 4 ? 1.f : kDiffGain));
#pragma unroll
  for (int c = 0; c < 8; ++c) out[(int64_t)i * 8 + c] = v[c];
}

ConvShape shape_of(int B, int H, int W, int C) {
  ConvShape s;
  s.B = B;
  s.H = H;
  s.W = W;
  s.C = C;
  s.OH = (H + 1) / 2;
  s.OW = (W + 1) / 2;
  s.KP = ((9 * C + 31) / 32) * 32;
  return s;
}

}  // namespace

int conv_kp(int C) { return ((9 * C + 31) / 32) * 32; }

void launch_conv_fwd(int B, int H, int W, int C, const uint16_t* in, const uint16_t* wk, const float* bias,
                     uint16_t* out, hipStream_t st) {
  const ConvShape s = shape_of(B, H, W, C);
  const int64_t M = (int64_t)B * s.OH * s.OW;
  if (C == 8) {
    const int64_t g = std::min<int64_t>((M + 63) / 64, 1024);  // beyond, a wave walks several tiles with its weights
    hipLaunchKernelGGL(k_conv8_fwd, dim3((unsigned)g), dim3(256), 0, st, s, in, wk, bias, out);
  } else if (M <= kSmallPixels) {
    hipLaunchKernelGGL(k_conv64_fwd_small, dim3((unsigned)((M + 15) / 16)), dim3(256), 0, st, s, in, wk, bias, out);
  } else {
    hipLaunchKernelGGL(k_conv64_fwd, dim3((unsigned)((M + 64 * kPixTiles - 1) / (64 * kPixTiles))), dim3(256), 0, st, s,
                       in, wk, bias, out);
  }
}

void launch_conv_bwd_data(int B, int H, int W, const uint16_t* dout, const uint16_t* wt, const uint16_t* in,
                          uint16_t* din, hipStream_t st) {
  const ConvShape s = shape_of(B, H, W, 64);
  const int64_t most = (int64_t)B * ((H + 1) / 2) * ((W + 1) / 2);  // pixels of the largest parity
  hipLaunchKernelGGL(k_conv64_bwd_data, dim3((unsigned)((most + 64 * kPixTiles - 1) / (64 * kPixTiles)), 4), dim3(256),
                     0, st, s, dout, wt, in, din);
}

void launch_conv_bwd_weight(int B, int H, int W, int C, const uint16_t* dy, const uint16_t* in, float* dw, float* db,
                            hipStream_t st) {
  const ConvShape s = shape_of(B, H, W, C);
  const int64_t M = (int64_t)B * s.OH * s.OW, chunks = (M + kWPix - 1) / kWPix;
  // enough workgroups to fill the chip, few enough that the atomics at the end (one per workgroup and element, some
  // 60 ns apiece on the same element) stay cheap: first layer 512 workgroups 65 us, 256 50; the others 128 per tap
  // 91 us, 64 70
  if (C == 8)
    hipLaunchKernelGGL(k_conv_bwd_weight<8>, dim3(1, (unsigned)std::min<int64_t>(chunks, 256)), dim3(256), 0, st, s, dy,
                       in, dw, db);
  else
    hipLaunchKernelGGL(k_conv_bwd_weight<64>, dim3(9, (unsigned)std::min<int64_t>(chunks, 64)), dim3(256), 0, st, s, dy,
                       in, dw, db);
}

void launch_head_fwd(int B, int OH, int OW, const uint16_t* act, const float* wfc, const float* bfc, float* pool,
                     float* out, hipStream_t st) {
  hipLaunchKernelGGL(k_head_fwd, dim3((unsigned)B), dim3(256), 0, st, act, OH, OW, wfc, bfc, pool, out);
}

void launch_head_bwd(int B, int OH, int OW, const float* out, const float* label, const float* scale,
                     const float* pool, const float* wfc, const uint16_t* act, const float* dout, float* dwfc,
                     float* dbfc, uint16_t* dact, float* loss, hipStream_t st) {
  hipLaunchKernelGGL(k_head_bwd, dim3((unsigned)B), dim3(256), 0, st, out, label, scale, B, pool, wfc, act, OH, OW,
                     dout, dwfc, dbfc, dact, loss);
}

void launch_cast_weights(const CastWeights& a, hipStream_t st) {
  hipLaunchKernelGGL(k_cast_weights, dim3((64 * 576 + 255) / 256, (unsigned)a.n), dim3(256), 0, st, a);
}

void launch_pack_input(const float* rc, const float* rd, const float* oc, const float* od, int H, int W, int f,
                       float depth_scale, uint16_t* out, hipStream_t st) {
  const int n = (W / f) * (H / f);
  const dim3 grid((unsigned)((n + 63) / 64)), block(64);
  switch (f) {
    case 1: hipLaunchKernelGGL(k_pack_input<1>, grid, block, 0, st, rc, rd, oc, od, H, W, f, depth_scale, out); break;
    case 2: hipLaunchKernelGGL(k_pack_input<2>, grid, block, 0, st, rc, rd, oc, od, H, W, f, depth_scale, out); break;
    case 3: hipLaunchKernelGGL(k_pack_input<3>, grid, block, 0, st, rc, rd, oc, od, H, W, f, depth_scale, out); break;
    case 4: hipLaunchKernelGGL(k_pack_input<4>, grid, block, 0, st, rc, rd, oc, od, H, W, f, depth_scale, out); break;
    default: hipLaunchKernelGGL(k_pack_input<0>, grid, block, 0, st, rc, rd, oc, od, H, W, f, depth_scale, out);
  }
}

}  // namespace gsr
