// Swap-proposal CNN: forward, backward and Adam, hand-written for gfx950 MFMA.
//
// The network ranks pixel interchanges for the annealer (the paper leaves the modification
// operator open, Sec. 4); the exact lineal-path change still judges every move.
//   X0 = (pixel, interface flag)   -> conv3x3 16 -> relu -> conv3x3 16 -> relu -> conv3x3 16
//   -> relu -> 1x1 head = per-pixel score S.   Periodic 'same' padding on the cell.
// Activations and weights are bfloat16, accumulation fp32.  Tensors are channels-last:
// X0 [B][H][W][4] (2 used), A_l [B][H][W][16]; forward weights Wf[tap][co][ci], backward-data
// weights Wt[tap][ci][co] (tap = 3 dy + dx, input offset (dy-1, dx-1)).
//
// A convolution is an implicit GEMM: a wave computes 16 pixels x 16 output channels with one
// v_mfma_f32_16x16x16_bf16 per tap (K = 16 input channels).  MFMA 16x16x16 operand layout on a
// 64-lane wave: lane l holds A[l%16][4(l/16)+j], B[4(l/16)+j][l%16] and D[4(l/16)+j][l%16],
// j = 0..3.  Pixel rows of A come from the (periodically) shifted neighbours, so the 8-byte
// operand of a lane is 4 consecutive channels of one pixel.
#include <math.h>

#include <algorithm>

#include "lpf_internal.h"

namespace lpf {

typedef short s4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x7fffffu)) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// ------------------------------------------------------------------------------- features
__global__ void k_cnn_features(const uint64_t *__restrict__ bits, int W, int H, int64_t npix,
                               uint16_t *__restrict__ X0) {
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;  // at most 2^28 pixels in a batch
  if (p >= (uint32_t)npix) return;
  const uint32_t row = p / (uint32_t)W, b = row / (uint32_t)H;  // image b starts at row b H
  const int x = (int)(p - row * (uint32_t)W), y = (int)(row - b * (uint32_t)H);
  const int wpr = (W + 63) >> 6;
  const uint64_t *img = bits + (size_t)b * H * wpr;
  auto at = [&](int yy, int xx) -> int {
    return (int)((img[(size_t)yy * wpr + (xx >> 6)] >> (xx & 63)) & 1ull);
  };
  const int v = at(y, x);
  const int xl = x ? x - 1 : W - 1, xr = x + 1 == W ? 0 : x + 1;
  const int yu = y ? y - 1 : H - 1, yd = y + 1 == H ? 0 : y + 1;
  const int itf = at(y, xl) != v || at(y, xr) != v || at(yu, x) != v || at(yd, x) != v;
  uint2 o;
  o.x = (uint32_t)(v ? 0x3f80u : 0u) | ((uint32_t)(itf ? 0x3f80u : 0u) << 16);
  o.y = 0;
  *reinterpret_cast<uint2 *>(X0 + (size_t)4 * p) = o;
}

// ---------------------------------------------------------------------------------- strips
// The layered kernels give a wave a strip: 16 pixels of kStrip image rows (one row of an MFMA tile
// per image row).  A row's three shifted operands (x - 1, x, x + 1) serve the three output rows
// that read them, so a tile of nine taps loads three operands instead of nine, and a strip's
// indices are computed once (a tile of 16 consecutive pixels took two 64-bit divisions).
constexpr int kStrip = 8;

struct Strip {
  int64_t img;  // first pixel of the image
  int y0, x;    // first row; the lane's column, clamped into the row
  int xs[3];    // columns x - 1, x, x + 1, periodic
  bool in;      // the lane's column lies in the row
};
__host__ __device__ inline int64_t strip_count(int W, int H, int batch, int rows) {
  return (int64_t)batch * ((H + rows - 1) / rows) * ((W + 15) / 16);
}
__device__ __forceinline__ Strip strip_of(int64_t i, int W, int H, int rows, int m) {
  const uint32_t segs = (uint32_t)(W + 15) / 16, bands = (uint32_t)(H + rows - 1) / rows;
  const uint32_t u = (uint32_t)i;  // at most 2^28 pixels in a batch
  const uint32_t r = u / segs, b = r / bands;
  Strip s;
  s.img = (int64_t)b * W * H;
  s.y0 = (int)(r - b * bands) * rows;
  const int x = (int)(u - r * segs) * 16 + m;
  s.in = x < W;
  s.x = min(x, W - 1);
  s.xs[0] = s.x ? s.x - 1 : W - 1;
  s.xs[1] = s.x;
  s.xs[2] = s.x + 1 == W ? 0 : s.x + 1;
  return s;
}
// Channels 4 g .. 4 g + 3 of the strip's pixels in row y (periodic, -1 <= y <= H), shifted by -1,
// 0, 1; of C channels per pixel (channels past C are zero).
template <int C>
__device__ __forceinline__ void strip_row(const uint16_t *__restrict__ X, const Strip &s, int y,
                                          int W, int H, int g, s4v (&a)[3]) {
  y += y < 0 ? H : 0;
  y -= y >= H ? H : 0;
  const uint16_t *row = X + (s.img + (int64_t)y * W) * C;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    a[d] = s4v{0, 0, 0, 0};
    if (C == 16 || g == 0) a[d] = *reinterpret_cast<const s4v *>(row + s.xs[d] * C + (C == 16 ? 4 * g : 0));
  }
}
__device__ __forceinline__ uint2 pack4(const uint16_t (&v)[4]) {
  return make_uint2((uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16));
}

// -------------------------------------------------------------------------------- forward
// A_out = bf16(relu(conv3x3(X) + bias)); X has C (4 or 16) channels, of which 16 (or 4) enter the
// 16-wide K of the MFMA.  The weights are the MFMA's A operand and the pixels its B operand, so
// that a lane holds four consecutive channels of one pixel and stores them together (with the
// pixels as A, four 2-byte stores of four pixels).  HEAD: also the scores S, summed over the
// channels in their order as head_score does, and a zeroed score gradient dS (when given).
// 8 images of 256 x 256: 24 -> 10 us for a 16-channel layer (13 with the scores).
template <int C, bool HEAD>
__global__ void __launch_bounds__(256)
k_cnn_conv_fwd(const uint16_t *__restrict__ X, const uint16_t *__restrict__ Wf,
               const float *__restrict__ bias, uint16_t *__restrict__ A_out, int W, int H,
               int64_t nstrips, const float *__restrict__ W4bf, const float *__restrict__ b4,
               float *__restrict__ S, int64_t *__restrict__ dS) {
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, m = lane & 15;
  const int64_t i = (int64_t)blockIdx.x * (blockDim.x >> 6) +
                    __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (i >= nstrips) return;
  s4v Bw[9];
#pragma unroll
  for (int t = 0; t < 9; ++t)
    Bw[t] = *reinterpret_cast<const s4v *>(Wf + (t * 16 + m) * 16 + 4 * g);
  float bco[4], w4[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    bco[j] = bias[4 * g + j];
    w4[j] = HEAD ? W4bf[4 * g + j] : 0.f;
  }
  const Strip q = strip_of(i, W, H, kStrip, m);
  s4v a[kStrip + 2][3];
  strip_row<C>(X, q, q.y0 - 1, W, H, g, a[0]);
  strip_row<C>(X, q, q.y0, W, H, g, a[1]);
#pragma unroll
  for (int r = 0; r < kStrip; ++r) {
    const int y = q.y0 + r;
    if (y >= H) return;
    strip_row<C>(X, q, y + 1, W, H, g, a[r + 2]);
    f4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t)
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(Bw[t], a[r + t / 3][t % 3], acc, 0, 0, 0);
    uint16_t v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = f2bf(fmaxf(acc[j] + bco[j], 0.f));
    const int64_t p = q.img + (int64_t)y * W + q.x;
    if (q.in) *reinterpret_cast<uint2 *>(A_out + p * 16 + 4 * g) = pack4(v);
    if constexpr (HEAD) {
      float sum = 0.f;  // channels 0..3 in lanes g = 0, then 4..7 in g = 1, ...
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float t = sum;
#pragma unroll
        for (int j = 0; j < 4; ++j) t += bf2f(v[j]) * w4[j];
        sum = __shfl(t, 16 * k + m, 64);
      }
      if (g == 0 && q.in) {
        S[p] = sum + b4[0];
        if (dS) dS[p] = 0;
      }
    }
  }
}

// Score of one pixel from its 16 layer-3 activations: sum_c A3[c] W4[c] + b4 (W4 rounded to
// bf16), summed in channel order.
__device__ __forceinline__ float head_score(const uint16_t *a3, const float *__restrict__ W4bf,
                                            const float *__restrict__ b4) {
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < 16; ++c) s += bf2f(a3[c]) * W4bf[c];
  return s + b4[0];
}

// ---------------------------------------------------------------- single-image scores, fused
// The annealer's re-scoring of its cell in one launch.  A workgroup computes a 16 x 16 tile of
// scores: the features of the tile and a 3-pixel periodic halo (22 x 22), then each layer's
// activations on a halo one pixel narrower (20 x 20, 18 x 18, 16 x 16), all in LDS.  Halo pixels
// are real pixels of the periodic cell, so their activations are the ones the layered kernels
// compute; each output uses the same MFMA taps in the same order, the same bias, ReLU and bf16
// rounding and the same head, so the scores equal cnn_forward's bit for bit.
constexpr int kScoreTile = 16;

// One 3x3 layer on LDS regions: `in` is a (wout + 2)^2 region with cin (4 or 16) channels per
// pixel, `out` the wout^2 region inside it with 16; the workgroup's waves take 16-pixel tiles in
// turn.
__device__ __forceinline__ void conv_region(const uint16_t *in, int cin, uint16_t *out, int wout,
                                            const uint16_t *__restrict__ Wf,
                                            const float *__restrict__ bias) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, m = lane & 15;
  const int win = wout + 2, nout = wout * wout;
  s4v Bw[9];
#pragma unroll
  for (int t = 0; t < 9; ++t)
    Bw[t] = *reinterpret_cast<const s4v *>(Wf + (t * 16 + m) * 16 + 4 * g);
  const float bco = bias[m];
  const int nwaves = (int)(blockDim.x >> 6);
  for (int tile = wave; tile * 16 < nout; tile += nwaves) {
    const int i = tile * 16 + m;
    const bool pin = i < nout;
    const int ry = pin ? i / wout : 0, rx = pin ? i - ry * wout : 0;
    f4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int src = (ry + t / 3) * win + rx + t % 3;  // input offset (t / 3 - 1, t % 3 - 1)
      s4v a = {0, 0, 0, 0};
      if (pin && 4 * g < cin) a = *reinterpret_cast<const s4v *>(in + src * cin + 4 * g);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, Bw[t], acc, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int po = tile * 16 + 4 * g + j;
      if (po < nout) out[po * 16 + m] = f2bf(fmaxf(acc[j] + bco, 0.f));
    }
  }
}

// 1024 threads: each layer's tiles spread over 16 waves (four per SIMD), so that the chains of
// MFMA and LDS latency of one wave overlap those of the others.
__global__ void __launch_bounds__(1024)
k_cnn_score(const uint64_t *__restrict__ bits, int W, int H, const uint16_t *__restrict__ Wf,
            const float *__restrict__ prm, const float *__restrict__ W4bf,
            float *__restrict__ S) {
  constexpr int T = kScoreTile;
  __shared__ __attribute__((aligned(16))) uint16_t X0[(T + 6) * (T + 6) * 4];
  __shared__ __attribute__((aligned(16))) uint16_t A1[(T + 4) * (T + 4) * 16];
  __shared__ __attribute__((aligned(16))) uint16_t A2[(T + 2) * (T + 2) * 16];
  __shared__ __attribute__((aligned(16))) uint16_t A3[T * T * 16];
  const int tx0 = blockIdx.x * T, ty0 = blockIdx.y * T;
  const int wpr = (W + 63) >> 6;
  auto at = [&](int y, int x) -> int {
    return (int)((bits[(size_t)y * wpr + (x >> 6)] >> (x & 63)) & 1ull);
  };
  for (int i = threadIdx.x; i < (T + 6) * (T + 6); i += blockDim.x) {
    const int ry = i / (T + 6), rx = i - ry * (T + 6);
    const int y = (((ty0 - 3 + ry) % H) + H) % H, x = (((tx0 - 3 + rx) % W) + W) % W;
    const int v = at(y, x);
    const int xl = x ? x - 1 : W - 1, xr = x + 1 == W ? 0 : x + 1;
    const int yu = y ? y - 1 : H - 1, yd = y + 1 == H ? 0 : y + 1;
    const int itf = at(y, xl) != v || at(y, xr) != v || at(yu, x) != v || at(yd, x) != v;
    uint2 o;
    o.x = (uint32_t)(v ? 0x3f80u : 0u) | ((uint32_t)(itf ? 0x3f80u : 0u) << 16);
    o.y = 0;
    *reinterpret_cast<uint2 *>(X0 + 4 * i) = o;
  }
  __syncthreads();
  conv_region(X0, 4, A1, T + 4, Wf, prm + 288);
  __syncthreads();
  conv_region(A1, 16, A2, T + 2, Wf + 2304, prm + 2608);
  __syncthreads();
  conv_region(A2, 16, A3, T, Wf + 4608, prm + 4928);
  __syncthreads();
  const int ry = threadIdx.x / T, rx = threadIdx.x - ry * T;
  const int y = ty0 + ry, x = tx0 + rx;
  if (threadIdx.x < T * T && y < H && x < W)
    S[(size_t)y * W + x] = head_score(A3 + threadIdx.x * 16, W4bf, prm + 4960);
}

// ------------------------------------------------------------------------------ loss / head
constexpr double kFx = 1099511627776.0;  // 2^40: fixed-point scale of the score gradient

// r_i = S[img][a] + S[img][b] - y; dS[img][a], dS[img][b] += 2 r_i / n in 2^-40 fixed point
// (integer atomics: the sum does not depend on their order).  lpart: sum r^2 of each workgroup's
// 256 samples, in a fixed order.
__global__ void __launch_bounds__(256)
k_cnn_loss(const float *__restrict__ S, const CnnSample *__restrict__ smp, int n, int64_t hw,
           int batch, long long *__restrict__ dS_fx, double *__restrict__ lpart) {
  __shared__ double part[256];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  float r = 0.f;
  if (i < n) {
    const CnnSample s = smp[i];
    const bool ok = s.img >= 0 && s.img < batch && s.a >= 0 && s.a < hw && s.b >= 0 && s.b < hw;
    if (ok) {
      const int64_t o = (int64_t)s.img * hw;
      r = S[o + s.a] + S[o + s.b] - s.y;
      const long long g = llrint((2.0 * (double)r / (double)n) * kFx);
      atomicAdd((unsigned long long *)&dS_fx[o + s.a], (unsigned long long)g);
      atomicAdd((unsigned long long *)&dS_fx[o + s.b], (unsigned long long)g);
    }
  }
  part[threadIdx.x] = (double)r * (double)r;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) part[threadIdx.x] += part[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) lpart[blockIdx.x] = part[0];
}

// dZ3 = bf16(dS * W4 * [A3 > 0]); per-block partials of dW4 (16) and db4 (1), fixed order: a thread
// adds over its pixels, then the lanes of a wave, then the waves.
constexpr int kHeadBlocks = 1024;
__global__ void __launch_bounds__(256)
k_cnn_head_bwd(const long long *__restrict__ dS_fx, const uint16_t *__restrict__ A3,
               const float *__restrict__ W4bf, int64_t npix, uint16_t *__restrict__ dZ3,
               float *__restrict__ part /* [blocks][17] */) {
  __shared__ float red[4][17];
  float loc[17], w4[16];
#pragma unroll
  for (int c = 0; c < 17; ++c) loc[c] = 0.f;
#pragma unroll
  for (int c = 0; c < 16; ++c) w4[c] = W4bf[c];
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < npix;
       p += (int64_t)gridDim.x * blockDim.x) {
    const float d = (float)((double)dS_fx[p] / kFx);
    const uint4 *src = reinterpret_cast<const uint4 *>(A3 + p * 16);
    uint4 in[2] = {src[0], src[1]}, out[2];
    const uint32_t *iw = reinterpret_cast<const uint32_t *>(in);
    uint32_t *ow = reinterpret_cast<uint32_t *>(out);
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      const float a0 = __uint_as_float(iw[h] << 16), a1 = __uint_as_float(iw[h] & 0xffff0000u);
      ow[h] = (uint32_t)f2bf(a0 > 0.f ? d * w4[2 * h] : 0.f) |
              ((uint32_t)f2bf(a1 > 0.f ? d * w4[2 * h + 1] : 0.f) << 16);
      loc[2 * h] += d * a0;
      loc[2 * h + 1] += d * a1;
    }
    loc[16] += d;
    uint4 *dst = reinterpret_cast<uint4 *>(dZ3 + p * 16);
    dst[0] = out[0];
    dst[1] = out[1];
  }
#pragma unroll
  for (int c = 0; c < 17; ++c) {
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) loc[c] += __shfl_xor(loc[c], k, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][c] = loc[c];
  }
  __syncthreads();
  if (threadIdx.x < 17)
    part[(size_t)blockIdx.x * 17 + threadIdx.x] =
        ((red[0][threadIdx.x] + red[1][threadIdx.x]) + red[2][threadIdx.x]) + red[3][threadIdx.x];
}

// ------------------------------------------------------------------------- backward (data)
// dZ_prev = bf16(conv3x3^T(dZ; W) * [A_prev > 0]) with dX[p] = sum_t W[t]^T dZ[p - off(t)]; strips
// and operands as in the forward pass.  Workgroup `block` takes four strips.
__device__ __forceinline__ void conv_bwd_data(int64_t block, const uint16_t *__restrict__ dZ,
                                              const uint16_t *__restrict__ Wt,
                                              const uint16_t *__restrict__ A_prev,
                                              uint16_t *__restrict__ dZ_prev, int W, int H,
                                              int64_t nstrips) {
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, m = lane & 15;
  const int64_t i = block * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (i >= nstrips) return;
  s4v Bw[9];
#pragma unroll
  for (int t = 0; t < 9; ++t)
    Bw[t] = *reinterpret_cast<const s4v *>(Wt + (t * 16 + m) * 16 + 4 * g);
  const Strip q = strip_of(i, W, H, kStrip, m);
  s4v a[kStrip + 2][3];
  strip_row<16>(dZ, q, q.y0 - 1, W, H, g, a[0]);
  strip_row<16>(dZ, q, q.y0, W, H, g, a[1]);
#pragma unroll
  for (int r = 0; r < kStrip; ++r) {
    const int y = q.y0 + r;
    if (y >= H) return;
    strip_row<16>(dZ, q, y + 1, W, H, g, a[r + 2]);
    const int64_t p = q.img + (int64_t)y * W + q.x;
    const uint2 ap = *reinterpret_cast<const uint2 *>(A_prev + p * 16 + 4 * g);
    f4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t)  // tap t reads dZ at (1 - t / 3, 1 - t % 3)
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(Bw[t], a[r + 2 - t / 3][2 - t % 3], acc, 0, 0, 0);
    const float av[4] = {__uint_as_float(ap.x << 16), __uint_as_float(ap.x & 0xffff0000u),
                         __uint_as_float(ap.y << 16), __uint_as_float(ap.y & 0xffff0000u)};
    uint16_t v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = f2bf(av[j] > 0.f ? acc[j] : 0.f);
    if (q.in) *reinterpret_cast<uint2 *>(dZ_prev + p * 16 + 4 * g) = pack4(v);
  }
}

// ----------------------------------------------------------------------- backward (weights)
// Per-block partials of dW[t][co][ci] = sum_p dZ[p][co] X[p + off(t)][ci] and db[co] = sum_p
// dZ[p][co]; MFMA with M = co, N = ci, K = 16 pixels.
//
// Its operands hold four pixels of one channel per lane where memory holds four channels of one
// pixel.  Lane 16 g + 4 a + b loads channels 4 a .. 4 a + 3 of pixel 4 g + b (8 bytes), so that the
// four lanes of a quad hold a 4 x 4 block, which they transpose among themselves: eight vector
// operations, whatever values the channels hold.  (A product with the identity is one MFMA and two
// operations, and as fast, but makes NaN of every channel of a pixel with a value that is not
// finite.)  A row's three transposed fragments serve three output rows.  (The gather of single
// 2-byte values that this replaces took 121 us a layer for 8 images of 256 x 256, this 14.)
constexpr int kWeightStrip = 16;
constexpr int kWeightBlocks = 512;

// Channel c of pixel b in lane b, c = 0 .. 3, becomes channel b of pixel c.
__device__ __forceinline__ s4v transpose4(s4v a) {
  union {
    s4v v;
    uint32_t u[2];
  } o;
  o.v = a;
  const bool odd = threadIdx.x & 1, upper = threadIdx.x & 2;
  const uint32_t sel = odd ? 0x03020706u : 0x05040100u;
#pragma unroll
  for (int h = 0; h < 2; ++h) {  // lanes 0 and 1, 2 and 3 exchange halves
    const uint32_t x = (uint32_t)__builtin_amdgcn_mov_dpp((int)o.u[h], 0xb1, 0xf, 0xf, true);
    o.u[h] = __builtin_amdgcn_perm(x, o.u[h], sel);
  }
  // lanes 0 and 2, 1 and 3 exchange words
  const uint32_t t0 = (uint32_t)__builtin_amdgcn_mov_dpp((int)o.u[0], 0x4e, 0xf, 0xf, true);
  const uint32_t t1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)o.u[1], 0x4e, 0xf, 0xf, true);
  const uint32_t w0 = upper ? t1 : o.u[0], w1 = upper ? o.u[1] : t0;
  o.u[0] = w0;
  o.u[1] = w1;
  return o.v;
}

// A layer's backward pass: workgroups 0 .. wb - 1 the weights, the others (dZ_prev given) the data,
// in one launch, since both wait on memory more than they compute (13 + 14 us apart).
template <int C>
__global__ void __launch_bounds__(256)
k_cnn_conv_bwd(const uint16_t *__restrict__ dZ, const uint16_t *__restrict__ X, int W, int H, int wb,
               int64_t nstrips, float *__restrict__ part /* [wb][9*256+16] */,
               const uint16_t *__restrict__ Wt, uint16_t *__restrict__ dZ_prev, int64_t ndata) {
  if constexpr (C == 16) {
    if ((int)blockIdx.x >= wb) {
      conv_bwd_data((int64_t)blockIdx.x - wb, dZ, Wt, X, dZ_prev, W, H, ndata);
      return;
    }
  }
  __shared__ float red[4][9 * 256 + 16];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, m = lane & 15;
  const int chunk = m >> 2, pixel = 4 * g + (m & 3);  // what the lane loads
  f4v acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) acc[t] = f4v{0.f, 0.f, 0.f, 0.f};
  float dbl = 0.f;
  const s4v zero = {0, 0, 0, 0};
  for (int64_t i = (int64_t)blockIdx.x * 4 + wave; i < nstrips; i += (int64_t)wb * 4) {
    const Strip q = strip_of(i, W, H, kWeightStrip, pixel);
    s4v xt[3][3];  // transposed rows y - 1, y, y + 1 (slot: row mod 3)
    auto row = [&](int y, s4v(&t)[3]) {
      s4v a[3];
      strip_row<C>(X, q, y, W, H, chunk, a);
#pragma unroll
      for (int d = 0; d < 3; ++d) t[d] = transpose4(q.in ? a[d] : zero);
    };
    row(q.y0 - 1, xt[0]);
    row(q.y0, xt[1]);
    const int rows = min(kWeightStrip, H - q.y0);
    for (int r0 = 0; r0 < rows; r0 += 3) {
#pragma unroll
      for (int u = 0; u < 3; ++u) {  // row r0 + u: its rows' slots are u, u + 1, u + 2 mod 3
        if (r0 + u >= rows) break;
        const int y = q.y0 + r0 + u;
        const s4v z =
            *reinterpret_cast<const s4v *>(dZ + (q.img + (int64_t)y * W + q.x) * 16 + 4 * chunk);
        row(y + 1, xt[(u + 2) % 3]);
        const s4v a = transpose4(q.in ? z : zero);
#pragma unroll
        for (int j = 0; j < 4; ++j) dbl += bf2f((uint16_t)a[j]);
#pragma unroll
        for (int t = 0; t < 9; ++t)
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, xt[(u + t / 3) % 3][t % 3], acc[t],
                                                            0, 0, 0);
      }
    }
  }
  // lane holds D[co = 4g + j][ci = m] for each tap, and a partial db for co = m
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) red[wave][t * 256 + (4 * g + j) * 16 + m] = acc[t][j];
  // db[co]: lanes m, m+16, m+32, m+48 hold partials of channel m
  dbl += __shfl_xor(dbl, 16, 64);
  dbl += __shfl_xor(dbl, 32, 64);
  if (g == 0) red[wave][9 * 256 + m] = dbl;
  __syncthreads();
  for (int i = threadIdx.x; i < 9 * 256 + 16; i += blockDim.x)
    part[(size_t)blockIdx.x * (9 * 256 + 16) + i] =
        ((red[0][i] + red[1][i]) + red[2][i]) + red[3][i];
}

// --------------------------------------------------------------------- gradient assembly
// The packed gradient (W1 [9][16][2], b1, W2 [9][16][16], b2, W3 [9][16][16], b3, W4 [16], b4)
// from the per-block partials, in a fixed order: slice s of kGradSlices sums its contiguous range
// of blocks in block order (k_cnn_grad_part), then the slices are added in slice order
// (k_cnn_grad_sum).
constexpr int kGradSlices = 64;

__device__ __forceinline__ float grad_partial(const float *__restrict__ p1,
                                              const float *__restrict__ p2,
                                              const float *__restrict__ p3,
                                              const float *__restrict__ ph, int i, int b) {
  const int stride = 9 * 256 + 16;
  if (i < 288) {  // W1[t][co][ci<2]
    const int t = i / 32, co = (i / 2) % 16, ci = i % 2;
    return p1[(size_t)b * stride + t * 256 + co * 16 + ci];
  }
  if (i < 304) return p1[(size_t)b * stride + 9 * 256 + (i - 288)];
  if (i < 2608) return p2[(size_t)b * stride + (i - 304)];
  if (i < 2624) return p2[(size_t)b * stride + 9 * 256 + (i - 2608)];
  if (i < 4928) return p3[(size_t)b * stride + (i - 2624)];
  if (i < 4944) return p3[(size_t)b * stride + 9 * 256 + (i - 4928)];
  return ph[(size_t)b * 17 + (i - 4944)];  // 0..15: W4, 16: b4
}

__global__ void k_cnn_grad_part(const float *__restrict__ p1, const float *__restrict__ p2,
                                const float *__restrict__ p3, int nb_conv,
                                const float *__restrict__ ph, int nb_head,
                                float *__restrict__ slices) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kCnnParams) return;
  const int sl = blockIdx.y;
  const int nb = i < 4944 ? nb_conv : nb_head;
  const int per = (nb + kGradSlices - 1) / kGradSlices;
  const int b0 = min(nb, sl * per), b1 = min(nb, b0 + per);
  float s = 0.f;
  for (int b = b0; b < b1; ++b) s += grad_partial(p1, p2, p3, ph, i, b);
  slices[(size_t)sl * kCnnParams + i] = s;
}

// The last workgroup adds the loss's partials: loss = sum r^2 / n.
__global__ void __launch_bounds__(256)
k_cnn_grad_sum(const float *__restrict__ slices, float *__restrict__ grad,
               const double *__restrict__ lpart, int n, float *__restrict__ loss) {
  if (blockIdx.x + 1 == gridDim.x) {
    __shared__ double part[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < (n + 255) / 256; i += 256) s += lpart[i];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
      if ((int)threadIdx.x < k) part[threadIdx.x] += part[threadIdx.x + k];
      __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = (float)(part[0] / (double)n);
    return;
  }
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kCnnParams) return;
  float s = 0.f;
  for (int sl = 0; sl < kGradSlices; ++sl) s += slices[(size_t)sl * kCnnParams + i];
  grad[i] = s;
}

// ------------------------------------------------------------------------------ parameters
// bf16 weight layouts from the fp32 parameters.
__global__ void k_cnn_pack_weights(const float *__restrict__ prm, uint16_t *__restrict__ Wf,
                                   uint16_t *__restrict__ Wt, float *__restrict__ W4bf) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;  // over 3 layers x 9 taps x 256
  if (i < 3 * 2304) {
    const int l = i / 2304, r = i % 2304, t = r / 256, co = (r / 16) % 16, ci = r % 16;
    float w;
    if (l == 0) w = ci < 2 ? prm[t * 32 + co * 2 + ci] : 0.f;
    else w = prm[(l == 1 ? 304 : 2624) + r];
    const uint16_t h = f2bf(w);
    Wf[l * 2304 + r] = h;                          // [t][co][ci]
    Wt[l * 2304 + t * 256 + ci * 16 + co] = h;     // [t][ci][co]
  }
  if (i < 16) W4bf[i] = bf2f(f2bf(prm[4944 + i]));
}

// One Adam step on the fp32 parameters (Kingma & Ba, 2015); c1 = 1 - beta1^t, c2 = 1 - beta2^t; the
// bf16 weights follow in the same launch (the zeros of layer 1's unused channels stay as
// k_cnn_pack_weights left them).
__global__ void k_cnn_adam(float *__restrict__ prm, const float *__restrict__ grad,
                           float *__restrict__ mom, float *__restrict__ vel, float lr, float b1,
                           float b2, float eps, float c1, float c2, uint16_t *__restrict__ Wf,
                           uint16_t *__restrict__ Wt, float *__restrict__ W4bf) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kCnnParams) return;
  const float g = grad[i];
  const float m = b1 * mom[i] + (1.f - b1) * g;
  const float v = b2 * vel[i] + (1.f - b2) * g * g;
  mom[i] = m;
  vel[i] = v;
  const float mh = m / c1, vh = v / c2;
  const float w = prm[i] - lr * mh / (sqrtf(vh) + eps);
  prm[i] = w;
  // where the parameter stands in the bf16 layouts
  int l = -1, r = 0;
  if (i < 288) {  // W1 [t][co][ci < 2]
    l = 0;
    r = (i / 32) * 256 + (i / 2 % 16) * 16 + i % 2;
  } else if (i >= 304 && i < 2608) {
    l = 1;
    r = i - 304;
  } else if (i >= 2624 && i < 4928) {
    l = 2;
    r = i - 2624;
  } else if (i >= 4944 && i < 4960) {
    W4bf[i - 4944] = bf2f(f2bf(w));
  }
  if (l >= 0) {
    const uint16_t h = f2bf(w);
    Wf[l * 2304 + r] = h;                                                        // [t][co][ci]
    Wt[l * 2304 + (r & ~255) + (r & 15) * 16 + (r >> 4 & 15)] = h;               // [t][ci][co]
  }
}

// ---------------------------------------------------------------------------------- launchers
static int weight_blocks(int W, int H, int batch) {
  return (int)std::min<int64_t>(kWeightBlocks, (strip_count(W, H, batch, kWeightStrip) + 3) / 4);
}

// The layers of a batch; dS: also cleared, when given.
static hipError_t forward(const CnnBufs &B, const uint64_t *bits, int W, int H, int batch, float *S,
                          int64_t *dS, hipStream_t s) {
  const int64_t np = (int64_t)W * H * batch;
  const int nb = (int)((np + 255) / 256);
  const int64_t ns = strip_count(W, H, batch, kStrip);
  const dim3 g((unsigned)((ns + 3) / 4)), b(256);
  hipLaunchKernelGGL(k_cnn_features, dim3(nb), b, 0, s, bits, W, H, np, B.X0);
  hipLaunchKernelGGL((k_cnn_conv_fwd<4, false>), g, b, 0, s, B.X0, B.Wf, B.prm + 288, B.A1, W, H,
                     ns, nullptr, nullptr, nullptr, nullptr);
  hipLaunchKernelGGL((k_cnn_conv_fwd<16, false>), g, b, 0, s, B.A1, B.Wf + 2304, B.prm + 2608, B.A2,
                     W, H, ns, nullptr, nullptr, nullptr, nullptr);
  hipLaunchKernelGGL((k_cnn_conv_fwd<16, true>), g, b, 0, s, B.A2, B.Wf + 4608, B.prm + 4928, B.A3,
                     W, H, ns, B.W4bf, B.prm + 4960, S, dS);
  return hipGetLastError();
}

hipError_t cnn_forward(const CnnBufs &B, const uint64_t *bits, int W, int H, int batch,
                       float *S, hipStream_t s) {
  return forward(B, bits, W, H, batch, S, nullptr, s);
}

hipError_t cnn_score(const CnnBufs &B, const uint64_t *bits, int W, int H, float *S,
                     hipStream_t s) {
  const dim3 grid((unsigned)((W + kScoreTile - 1) / kScoreTile),
                  (unsigned)((H + kScoreTile - 1) / kScoreTile));
  hipLaunchKernelGGL(k_cnn_score, grid, dim3(1024), 0, s, bits, W, H, B.Wf, B.prm, B.W4bf, S);
  return hipGetLastError();
}

hipError_t cnn_grad(const CnnBufs &B, const uint64_t *bits, int W, int H, int batch,
                    const CnnSample *smp, int n, float *grad, float *loss, hipStream_t s) {
  const int64_t np = (int64_t)W * H * batch;
  const int64_t ns = strip_count(W, H, batch, kStrip), nw = strip_count(W, H, batch, kWeightStrip);
  const int wb = weight_blocks(W, H, batch);
  const int hb = (int)std::min<int64_t>(kHeadBlocks, (np + 255) / 256);
  const dim3 g((unsigned)((ns + 3) / 4)), b(256);
  hipError_t e = forward(B, bits, W, H, batch, B.S, B.dS, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_cnn_loss, dim3((n + 255) / 256), b, 0, s, B.S, smp, n, (int64_t)W * H, batch,
                     (long long *)B.dS, B.lpart);
  hipLaunchKernelGGL(k_cnn_head_bwd, dim3(hb), b, 0, s, (const long long *)B.dS, B.A3, B.W4bf, np,
                     B.dZ3, B.part_h);
  const dim3 gb((unsigned)(wb + (ns + 3) / 4));
  hipLaunchKernelGGL(k_cnn_conv_bwd<16>, gb, b, 0, s, B.dZ3, B.A2, W, H, wb, nw, B.part3,
                     B.Wt + 4608, B.dZ2, ns);
  hipLaunchKernelGGL(k_cnn_conv_bwd<16>, gb, b, 0, s, B.dZ2, B.A1, W, H, wb, nw, B.part2,
                     B.Wt + 2304, B.dZ1, ns);
  hipLaunchKernelGGL(k_cnn_conv_bwd<4>, dim3(wb), b, 0, s, B.dZ1, B.X0, W, H, wb, nw, B.part1,
                     nullptr, nullptr, (int64_t)0);
  hipLaunchKernelGGL(k_cnn_grad_part, dim3((kCnnParams + 255) / 256, kGradSlices), b, 0, s, B.part1,
                     B.part2, B.part3, wb, B.part_h, hb, B.slices);
  hipLaunchKernelGGL(k_cnn_grad_sum, dim3((kCnnParams + 255) / 256 + 1), b, 0, s, B.slices, grad,
                     B.lpart, n, loss);
  return hipGetLastError();
}

hipError_t cnn_pack(const CnnBufs &B, hipStream_t s) {
  hipLaunchKernelGGL(k_cnn_pack_weights, dim3((3 * 2304 + 255) / 256), dim3(256), 0, s, B.prm,
                     B.Wf, B.Wt, B.W4bf);
  return hipGetLastError();
}

hipError_t cnn_adam(const CnnBufs &B, const float *grad, float lr, float b1, float b2, float eps,
                    float c1, float c2, hipStream_t s) {
  hipLaunchKernelGGL(k_cnn_adam, dim3((kCnnParams + 255) / 256), dim3(256), 0, s, B.prm, grad,
                     B.mom, B.vel, lr, b1, b2, eps, c1, c2, B.Wf, B.Wt, B.W4bf);
  return hipGetLastError();
}

int cnn_weight_blocks() { return kWeightBlocks; }
int cnn_head_blocks() { return kHeadBlocks; }

}  // namespace lpf
