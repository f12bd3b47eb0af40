// Rows of packed images as the full evaluations stage them.  The arithmetic is compiled for the
// host too: the planners' host runs (run_cover and its like) take their words from here.
#pragma once

#include <stdint.h>

#include <vector>

#include <hip/hip_runtime.h>

namespace lpf {

namespace {

// hi:lo shifted right by s (0..31), the low word.
__host__ __device__ __forceinline__ uint32_t funnel(uint32_t hi, uint32_t lo, int s) {
#if __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_alignbit(hi, lo, s);
#else
  return (uint32_t)((((uint64_t)hi << 32) | lo) >> s);
#endif
}
__host__ __device__ __forceinline__ uint32_t bit_reverse(uint32_t v) {
  return __builtin_bitreverse32(v);
}

// The 32 pixels from pixel s on of a packed row, periodic (0 <= s < W).  Bits past W in the row's
// last word are never used.  Without branches for rows of at least a word.
__host__ __device__ __forceinline__ uint32_t periodic32(const uint32_t *__restrict__ row, int W, int s) {
  if (W >= 32) {
    const int q = s >> 5, n = W - s;  // n: pixels left in the row
    // (the dword after the row's last pixel: any value, and never read past the packed row)
    const uint32_t lo = row[q], hi = row[q + 1 < (W - 1) >> 5 ? q + 1 : (W - 1) >> 5];
    const uint32_t v = funnel(hi, lo, s & 31);
    return n < 32 ? (v & ((1u << n) - 1u)) | (row[0] << n) : v;
  }
  uint32_t v = 0;
  for (int b = 0, x = s; b < 32; ++b) {
    v |= ((row[0] >> x) & 1u) << b;
    x = x + 1 == W ? 0 : x + 1;
  }
  return v;
}

// First pixel of word e of a row extended periodically (bit j of the word is pixel (32 e + j) mod
// W), or, mirrored, of the 32 pixels that the word holds in reverse (bit j is pixel W - 1 - (32 e
// + j) mod W).
__host__ __device__ __forceinline__ int word_start(int W, int e, bool mirror) {
  int s = 32 * e;
  if (s >= W) s -= W;
  if (s >= W) s %= W;  // windows of more than twice the row only
  if (mirror) {
    s = W - 32 - s;
    if (s < 0) s += W;
    if (s < 0) s = (s % W + W) % W;
  }
  return s;
}

// 32 pixels of a row of nd dwords (even) from column x on, periodic.  One 8-byte load, and one more
// for the lanes whose pixels go on at the row's start: with 64 candidates per wave every load is
// 64 cache lines.
struct __attribute__((packed, aligned(4))) Dwords2 {
  uint64_t v;
};
__host__ __device__ __forceinline__ uint32_t row_word(const uint32_t *__restrict__ row, int nd, int W, int x) {
  const int e = x >> 5 < nd - 2 ? x >> 5 : nd - 2;
  const uint64_t w = ((const Dwords2 *)(row + e))->v;
  uint32_t v = (uint32_t)(w >> (x - 32 * e));
  const int n = W - x;
  if (n >= 32) return v;
  if (W >= 32) return (v & ((1u << n) - 1u)) | (row[0] << n);
  v &= (1u << n) - 1u;
  const uint32_t all = row[0] & ((1u << W) - 1u);
  for (int t = n; t < 32; t += W) v |= all << t;
  return v;
}
// Bits t, t + W, ... of a word.
__host__ __device__ __forceinline__ uint32_t every(int t, int W) {
  if (W >= 32) return t < 32 ? 1u << t : 0u;
  uint32_t v = 0;
  for (; t < 32; t += W) v |= 1u << t;
  return v;
}
// A byte image as packed rows of wpr dwords, the bits past W of each row set: they are not part of the
// image, and the host runs have to get by without them as the kernels do.
inline std::vector<uint32_t> packed_rows(const uint8_t *img, int W, int H, int wpr) {
  std::vector<uint32_t> rows((size_t)H * wpr, 0);
  for (int y = 0; y < H; ++y)
    for (int x = 0; x < 32 * wpr; ++x)
      if (x >= W || img[(size_t)y * W + x])
        rows[(size_t)y * wpr + (x >> 5)] |= 1u << (x & 31);
  return rows;
}

// Byte address of a word of the workgroup's LDS.
__device__ __forceinline__ uint32_t lds_address(const uint32_t *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint32_t *)p;
}

}  // namespace

}  // namespace lpf
