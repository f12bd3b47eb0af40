// Rows of packed images as the full evaluations stage them.  The arithmetic is compiled for the
// host too: the planners' host runs (run_cover and its like) take their words from here.
#pragma once

#include <stdint.h>

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

// Byte address of a word of the workgroup's LDS.
__device__ __forceinline__ uint32_t lds_address(const uint32_t *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint32_t *)p;
}

}  // namespace

}  // namespace lpf
