// Interchange deltas by shared segments: shared by the planner (plan_swap.hip), the kernels
// (k_swap.hip) and the C ABI.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

#include <hip/hip_runtime.h>

namespace lpf {

constexpr int kSwapMaxCut = 126;      // at most 127 placements: a change is a signed byte
constexpr int kSwapLevels = 4;        // pixels and segments of 2, 4 and 8 pixels
constexpr int kSwapLen = 1 << (kSwapLevels - 1);
constexpr int kSwapSlots = 8191;      // LDS slots of a sector: byte offsets in 16 bits
constexpr int kSwapTiles = 4;         // tiles of a sector, up to 64 vectors each
constexpr int kSwapWaves = 2 * kSwapTiles;  // of a workgroup: two share a tile's placements
constexpr int kSwapReads = 16;        // segments that a placement is read from, at most

// A sector: vectors of neighbouring directions, evaluated by one workgroup.  Slot 0 is zero (no
// placement), then its pixels, then the segments of each level.
struct SwapSector {
  int32_t npix, pix0;           // pixels: pix[pix0 ..], offsets in the window around the pixel
  int32_t off[kSwapLevels];     // first segment of a level: segs[off[l]]
  int32_t cnt[kSwapLevels];     // segments of a level
  int32_t tile0, ntiles;
  int32_t idx0, nvec;           // canonical indices, in canonical order
};
// 64 vectors (lanes; past the last one the placements are slot 0): placement k of a lane is the
// AND of 2 r2 slots, ents[off + (k r2 + j) 64 + lane], two byte offsets each.
struct SwapTile {
  int32_t nk;  // placements of the longest vector, rounded up to a multiple of 4
  int32_t r2;
  int32_t off;
  int32_t nvec;
};

struct SwapHost {
  int cx = 0, cy = 0, slots = 0;  // slots: of the largest sector
  std::vector<SwapSector> sectors;
  std::vector<SwapTile> tiles;
  std::vector<int32_t> idx;
  std::vector<int32_t> rank;   // of a tile's lane among its sector's vectors; 64 per tile
  std::vector<uint32_t> pix;   // (dy + cy) (2 cx + 1) + dx + cx
  std::vector<uint32_t> segs;  // byte offsets of the two halves, lower 16 bits the first
  std::vector<uint32_t> ents;
};

// False when the cutoffs are above kSwapMaxCut or the tables would exceed max_bytes.
bool plan_swap(int cx, int cy, size_t max_bytes, SwapHost &p);

struct SwapLaunch {
  const uint64_t *bits;
  int W, H, cx, cy;
  const int2 *cand;
  int K;
  const SwapSector *sectors;
  const SwapTile *tiles;
  const int32_t *idx, *rank;
  const uint32_t *pix, *segs, *ents;
  int nsectors, slots;
  uint2 *near;  // scratch: swap_near_bytes(cx, cy, phases) for each 32 candidates
  unsigned phase_mask;
  int nv;
  int32_t *delta_out;
};
constexpr size_t kSwapNearMax = (size_t)64 << 20;  // scratch of a context
inline size_t swap_near_bytes(int cx, int cy, unsigned phase_mask) {
  return (size_t)(phase_mask == 3 ? 2 : 1) * (2 * cx + 1) * (2 * cy + 1) * sizeof(uint2);
}
// Groups of 32 candidates per launch.
inline int swap_batch(int cx, int cy, unsigned phase_mask, int K) {
  const int fit = (int)(kSwapNearMax / swap_near_bytes(cx, cy, phase_mask));
  return std::min({(K + 31) / 32, fit, 32768});  // a grid's y extent
}
hipError_t launch_swap(const SwapLaunch &L, hipStream_t stream);

}  // namespace lpf
