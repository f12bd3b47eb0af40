// Prefix-tree plans of the volume evaluation: shared by the planner (plan_cover3.hip), the kernel
// (k_cover3.hip) and the C ABI.
#pragma once

#include <stdint.h>

#include <vector>

#include <hip/hip_runtime.h>

#include "cover.h"

namespace lpf {

// Longest segment (its steps are two bits each of a 64-bit word: at most 32).  Longer ones share
// less: both phases, this against every voxel walked: 100^3, cutoff 16 553 against 888 us, cutoff
// 24 2.52 against 5.28 ms; 64^3, cutoff 32 4.10 against 3.97 ms.
constexpr int kCover3Cut = 24;
constexpr int kCover3Waves = 16;   // of a workgroup
constexpr int kCover3Slots = 1024;

// A group: vectors of one sign of dx and dy, walked by one workgroup over the start rows of a
// slab.  Its pieces (one per wave, or per two, four, .. waves that take turns over the bands):
// records piece_off[piece0 + p] .. piece_off[piece0 + p + 1].
struct Cover3Group {
  int32_t piece0, mem0, nmem;
  int32_t mirror;  // x reversed (dx < 0)
  int32_t down;    // y offsets run from cy down (dy < 0): halo rows above the start rows
};

// A slab in LDS: zb + cz planes (mod D) of H + cy rows (mod H) of rst dwords, planes ps dwords
// apart.  P words of cover3_rows rows per lane, S lanes per row.
struct Cover3Shape {
  int W, H, D, cx, cy, cz;
  int P, S;
  int rst, ps, wid;  // wid: dwords staged per row
  int zb, nslab;
  int npieces;       // per group
};

// The staged cells that one thread of a workgroup writes: dword e of row pr, which is row yh of plane
// pl; carried forward, not divided out.  For the kernel and for the planner's host run.
struct Cover3Cell {
  int e, pr, pl, yh;
  int dq, dr;
  __host__ __device__ __forceinline__ Cover3Cell(int thread, int wid, int hh) {
    constexpr int step = 64 * kCover3Waves;
    dq = step / wid;
    dr = step - dq * wid;
    pr = thread / wid;
    e = thread - pr * wid;
    pl = pr / hh;
    yh = pr - pl * hh;
  }
  __host__ __device__ __forceinline__ void next(int wid, int hh) {
    e += dr;
    int adv = dq;
    if (e >= wid) {
      e -= wid;
      ++adv;
    }
    pr += adv;
    yh += adv;
    while (yh >= hh) {
      yh -= hh;
      ++pl;
    }
  }
  // The volume's row that is staged there, of a slab from plane Z0 on.
  __host__ __device__ __forceinline__ size_t row(const Cover3Shape &g, bool down, int Z0) const {
    int z = Z0 + pl, y = yh - (down ? g.cy : 0);
    z -= z >= g.D ? g.D : 0;  // cz <= D - 1, cy <= H - 1
    y += y < 0 ? g.H : 0;
    y -= y >= g.H ? g.H : 0;
    return (size_t)z * g.H + y;
  }
};

struct Cover3Host {
  Cover3Shape sh{};
  std::vector<Cover3Group> groups;
  std::vector<int32_t> piece_off, mems;  // mems: canonical indices by count slot
  std::vector<int4> recs;
  size_t lds_bytes = 0;
};

// Rows of a lane: as many as the registers of a walk hold (K words of the running product and of
// the start, of two saved products, and the dwords of two steps: 64 to 121).
constexpr int cover3_rows(int P, bool both) {
  return both ? (P == 1 ? 4 : P == 2 ? 3 : 2) : (P == 4 ? 3 : 4);
}

// False when a cutoff is above kCover3Cut, rows are longer than 16 words or a slab does not fit.
// vec: canonical 3-D vectors (x, y, z), nv of them; cus: compute units.
bool plan_cover3(int W, int H, int D, int cx, int cy, int cz, const int16_t *vec, int64_t nv,
                 int lds, int cus, Cover3Host &p);

struct Cover3Launch {
  Cover3Shape sh;
  const Cover3Group *groups;
  const int32_t *piece_off, *mems;
  const int4 *recs;
  int ngroups;
  size_t lds_bytes;
  int nv;
  const uint64_t *bits;
  unsigned phase_mask;
  uint32_t *counts;
};
hipError_t launch_cover3(const Cover3Launch &L, hipStream_t stream);
hipError_t prepare_cover3_kernels(int max_lds_bytes);

}  // namespace lpf
