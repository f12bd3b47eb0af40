// Cover plans of the full evaluation: shared by the planner (plan_cover.hip), the kernel
// (k_cover.hip) and the C ABI.
#pragma once

#include <stdint.h>

#include <vector>

#include <hip/hip_runtime.h>

#include "lpf_internal.h"

namespace lpf {

// Masks of a group held in LDS beside its image rows, and members (count slots) of a group.
constexpr int kCoverWords = 4;
constexpr int kCoverSlots = 1024;
// Dwords behind a group's arrays that a walk or a build may read without using (the second dword
// of a funnel shift and the words of lanes past the row).
constexpr int kCoverPad = 32;

// Record of a walk (int4, read on the scalar unit):
//   x: step 0 = offset in dwords (bits 0..15) | bit shift << 16 (5 bits), and the flags below
//   y: step 1, the same (when kRecTwo)
//   z: count slot (when kRecCount)
//   w: next record when the wave's count is zero (nothing that extends this path can count)
constexpr uint32_t kRecTwo = 1u << 21;
constexpr int kRecRestore = 22;  // 2 bits: 0 none, 1 the start pixels, 2 and 3 saved products 1, 2
constexpr int kRecSave = 24;     // 2 bits: 0 none, 1 and 2 saved products
constexpr uint32_t kRecCount = 1u << 26;

// One group: neighbouring slopes of one octant, walked by one workgroup.
struct CoverGroup {
  int32_t piece0;        // its pieces' records: piece_off[piece0 + p] .. piece_off[piece0 + p + 1]
  int32_t mem0, nmem;    // its members (count slot = member - mem0)
  int32_t tile, ntiles;  // start rows per tile (whole bands), tiles
  int32_t nwb;           // waves that share a piece, each over every nwb-th band of a tile
  int32_t rows;          // rows staged: tile + the largest row offset of a path
  int32_t rst, wid;      // dwords between rows, dwords staged per row
  int32_t asz;           // dwords of one array (array 0 the image, 1.. the word masks)
  int32_t sh_a, sh_b;    // first dword staged of row y: max(0, ((y - tile + 1) sh_a - sh_b) >> 16)
  uint32_t wid_magic, rows_magic;  // ceil(2^32 / wid), ceil(2^32 / rows); wid and rows are >= 2
  int32_t nw;            // word masks
  int32_t bop[kCoverWords + 1];  // build steps of mask a: bops[bop[a - 1]] .. bops[bop[a]]
  int32_t mirror;        // x reversed (vectors with dx < 0)
};

// Index arithmetic of a group's LDS rows, for the kernel and for the planner's host run of it (G: a
// CoverGroup in whatever address space).
//
// i / n, magic = ceil(2^32 / n), n >= 2: exact for i (n magic - 2^32) < 2^32, and so for the at most
// 2^16 cells of a group.
__host__ __device__ __forceinline__ int cover_div(int i, uint32_t magic) {
  return (int)(((uint64_t)(uint32_t)i * magic) >> 32);
}
// First dword staged of row y.
template <class G>
__host__ __device__ __forceinline__ int cover_first(const G &g, int y) {
  const int d = y - g.tile + 1 > 0 ? y - g.tile + 1 : 0;
  const int e = (d * g.sh_a - g.sh_b) >> 16;
  return e > 0 ? e : 0;
}
// Staged cell i of rows * wid: row y, dword e of the row.
template <class G>
__host__ __device__ __forceinline__ void cover_cell(const G &g, int i, int &y, int &e) {
  y = cover_div(i, g.wid_magic);
  e = cover_first(g, y) + i - y * g.wid;
}
// Item i of a mask's build, C dwords each: chunk i / rows of row i mod rows; the last chunk of a row
// is moved back to end with the row.  Returns the first dword's place in its array.
template <int C>
__host__ __device__ __forceinline__ int cover_mask_items(int wid, int rows) {
  return (wid + C - 1) / C * rows;
}
template <int C, class G>
__host__ __device__ __forceinline__ int cover_mask_item(const G &g, int i) {
  const int ch = cover_div(i, g.rows_magic);
  const int y = i - ch * g.rows;
  const int e = ch * C < g.wid - C ? ch * C : g.wid - C;
  return y * g.rst + cover_first(g, y) + e;
}
// Dwords per item for R words per lane.
constexpr int cover_mask_words(int R) { return R >= 7 ? 8 : R + 1; }

// One image's plan as the kernel reads it.
struct CoverImg {
  const CoverGroup *groups;
  const int32_t *piece_off;
  const int4 *recs;
  const uint32_t *bops;  // offset in dwords | bit shift << 16
  const MemDesc *mems;
  // nsplit workgroups share a group and phase, each over every nsplit-th tile
  int W, H, cx, cy, R, S, nct, nsplit, nv, layout;
};

// Shape of a plan: R words per lane, S lanes per row, wpg waves per workgroup, of which up to nwb
// share a piece (wpg / nwb pieces per group), LDS bytes per workgroup.
struct CoverShape {
  int R = 0, S = 0, wpg = 0, nwb = 0, lds = 0;
};

struct CoverHost {
  CoverShape sh;
  int nct = 1;     // tiles across a row
  int nsplit = 1;  // workgroups per group and phase
  size_t lds_bytes = 0;  // of the launch (the largest group)
  std::vector<CoverGroup> groups;
  std::vector<int32_t> piece_off;
  std::vector<int4> recs;
  std::vector<uint32_t> bops;
  std::vector<MemDesc> mems;
  // work items {group, split} of one phase in launch order: most work first (cost), neighbours
  // in another order than the groups'
  std::vector<int2> items;
  std::vector<int64_t> cost;
  int64_t steps = 0, counts = 0, bsteps = 0;
};

// Lane layout for an image: R in 1..16 and S a power of two.
void cover_lanes(int W, int H, int *R, int *S);
// The plan for an image size and cutoff on a device of `cus` compute units; fR, fS, fW, fL fix the
// shape's R, S, waves and LDS bytes (0: chosen here).  False when the rows do not fit in LDS.  May
// throw std::bad_alloc.
bool plan_cover(int W, int H, int cx, int cy, int fR, int fS, int fW, int fL, int cus,
                CoverHost &out);
// Counts of a byte image by running the plan on the host, word for word as the kernel does;
// false when an access leaves its array.  counts: [|D_c|], of phase `phase`.
bool run_cover(const CoverHost &p, const uint8_t *img, int W, int H, int phase, int64_t *counts);

// Start pixels of a Monte-Carlo position set (packed like the image) as the kernel reads them:
// out[2][H][ceil(W / 32)], plain and mirrored.
hipError_t launch_start_sets(const uint64_t *sample, int W, int H, uint32_t *out,
                             hipStream_t stream);
// One workgroup per item and phase of phase_mask.  sample: the start pixels of
// launch_start_sets, or null (every pixel).
hipError_t launch_cover(const CoverImg &I, const CoverShape &sh, const int2 *items, int n_items,
                        size_t lds_bytes, unsigned phase_mask, const uint64_t *bits,
                        const uint32_t *sample, uint32_t *out, hipStream_t stream);
// Many images: items {image, group, phase, split}, one workgroup each; image i's packed rows at
// pool + bits_off[i], its counts at counts + counts_off[i] (zeroed by launch_cover_zero where an
// image's groups are split).
hipError_t launch_cover_zero(const CoverImg *imgs, const int64_t *counts_off, int n_images,
                             unsigned phase_mask, uint32_t *counts, hipStream_t stream);
hipError_t launch_cover_batch(const CoverImg *imgs, const int64_t *bits_off,
                              const int64_t *counts_off, const int4 *items, int n_items, int wpg,
                              size_t lds_bytes, unsigned phase_mask, const uint64_t *pool,
                              uint32_t *counts, hipStream_t stream);
hipError_t prepare_cover_kernels(int max_lds_bytes);

}  // namespace lpf
