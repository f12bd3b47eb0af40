// Exact change of the lineal path function under a pixel interchange (Sec. 4 modification
// operator), for many candidate interchanges at once: placements from shared segments.
//
// Only translations whose segment covers a swapped pixel can change.  With a the phase-1 pixel and
// b the phase-0 pixel of an interchange, P_p the translations whose segment covers p, lambda_i the
// indicator "segment entirely in phase i", J1 = I with b set to 1 and J0 = I with a set to 0:
//     dL_1 = sum_{s in P_b} lambda_1(s; J1) - sum_{s in P_a} lambda_1(s; J1)
//     dL_0 = sum_{s in P_a} lambda_0(s; J0) - sum_{s in P_b} lambda_0(s; J0)
// (a translation covering both pixels appears in both sums with the same value and cancels; one
// covering only a or only b sees exactly the old or the new image).
//
// Words hold 32 candidates, a bit each: k_swap_near writes, for every pixel of the window around
// a (side 0) and around b (side 1), the word of "this pixel is in the phase".  An AND of two words
// then advances 32 candidates at once, and the plan (plan_swap.hip) shares the ANDs of all
// placements of a sector's vectors.  In k_swap a lane is a vector; it reads each of its placements
// as the AND of a few segments and counts them per candidate in bit planes (carry-save adders: 3
// operations per placement and side for 32 candidates).
#include <algorithm>

#include "delta_dev.h"
#include "row_dev.h"
#include "swap.h"

namespace lpf {

namespace {

// Lane i's bit j to lane j's bit i, for the 32 lanes of each half of the wave.
__device__ __forceinline__ uint32_t transpose32(uint32_t v, int lane) {
#pragma unroll
  for (int h = 4; h >= 0; --h) {
    const int s = 1 << h;
    const uint32_t m = s == 16 ? 0x0000ffffu : s == 8 ? 0x00ff00ffu : s == 4 ? 0x0f0f0f0fu
                       : s == 2 ? 0x33333333u : 0x55555555u;
    const uint32_t y = (uint32_t)__shfl_xor((int)v, s, 64);
    v = (lane & s) ? (v & ~m) | ((y >> s) & m) : (v & m) | ((y & m) << s);
  }
  return v;
}

// Window rows of a wave: 512 candidates at cutoff 48 take 27, 29 and 35 us with 1, 2 and 4.
constexpr int kNearRows = 1;
constexpr int kNearWords = 4;  // words of a row in flight

}  // namespace

// near[((g nph + p) npos + pos)]: the words of candidates 32 (g0 + g) .. + 31 for the pixel at
// offset pos of the window around a (x) and around b (y): phase 0, the pixel is 0 or a; phase 1,
// it is 1 or b (the changed pixels never end a segment).  A candidate that is no interchange
// (equal phases, a pixel outside the cell) has zero words and so no change.
//
// A lane loads 32 pixels of one candidate's window row; a 32 x 32 transpose makes them the words
// of 32 positions.  4096 candidates at cutoff 48: 19 MB written in 18 us (three 8-byte loads per
// word of every lane's row: 21 us; a transpose per phase: 1 us more).
__global__ void __launch_bounds__(256)
k_swap_near(const uint64_t *__restrict__ bits, int W, int H, int cx, int cy,
            const int2 *__restrict__ cand, int K, int g0, unsigned phase_mask,
            uint32_t *__restrict__ near) {
  const int lane = threadIdx.x & 63, side = lane >> 5;
  const int k = (g0 + (int)blockIdx.y) * 32 + (lane & 31);
  int a = 0, b = 0;
  bool ok = k < K;
  if (ok) {
    const int2 ab = cand[k];
    a = ab.x;
    b = ab.y;
    const int64_t NN = (int64_t)W * H;
    ok = a >= 0 && b >= 0 && a < NN && b < NN && a != b;
  }
  if (!ok) a = b = 0;
  const int va = pixel_value(bits, W, a), vb = pixel_value(bits, W, b);
  ok = ok && va != vb;
  if (!va) {
    const int t = a;
    a = b;
    b = t;
  }
  const int ay = a / W, ax = a - ay * W, by = b / W, bx = b - by * W;
  const int sx = side ? bx : ax, sy = side ? by : ay;
  const int wid = 2 * cx + 1, rows = 2 * cy + 1, nw = (wid + 31) >> 5;
  const int nph = phase_mask == 3 ? 2 : 1;
  const uint64_t oks = __builtin_amdgcn_ballot_w64(ok);
  const uint32_t live = side ? (uint32_t)(oks >> 32) : (uint32_t)oks;
  const int step = 32 % W, nd = 2 * ((W + 63) >> 6);
  // the wave's rows of the window, each in words of 32 columns
  const int wave = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r1 = min(rows, (wave + 1) * kNearRows);
  for (int r = wave * kNearRows; r < r1; ++r) {
    int y = sy + r - cy, x = sx - cx;  // |offsets| < the cell's sides
    y += y < 0 ? H : 0;
    y -= y >= H ? H : 0;
    x += x < 0 ? W : 0;
    const uint32_t *row = (const uint32_t *)bits + (size_t)y * nd;
    uint32_t *out = near + ((size_t)blockIdx.y * nph * rows + r) * (size_t)wid * 2 + side;
    for (int w0 = 0; w0 < nw; w0 += kNearWords) {
      uint32_t v[kNearWords];
      int xs[kNearWords];
#pragma unroll
      for (int j = 0; j < kNearWords; ++j) {
        xs[j] = x;
        v[j] = row_word(row, nd, W, x);
        x += step;
        x -= x >= W ? W : 0;
      }
      // the transpose of ~v is ~ that of v, and few rows hold a changed pixel
#pragma unroll
      for (int j = 0; j < kNearWords; ++j) v[j] = transpose32(v[j], lane);
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        if (!((phase_mask >> p) & 1u)) continue;
        const bool on_row = y == (p ? by : ay);
        uint32_t *o = out + (p && nph == 2 ? (size_t)rows * wid * 2 : 0);
        const bool any = __builtin_amdgcn_ballot_w64(on_row) != 0;
#pragma unroll
        for (int j = 0; j < kNearWords; ++j) {
          uint32_t word = p ? v[j] : ~v[j];
          if (any) {
            int t = (p ? bx : ax) - xs[j];
            t += t < 0 ? W : 0;
            word |= transpose32(on_row ? every(t, W) : 0u, lane);
          }
          const int pos = 32 * (w0 + j) + (lane & 31);
          if (pos < wid) o[(size_t)pos * 2] = word & live;
        }
      }
    }
  }
}

namespace {

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}
// Counts of 32 candidates: plane p holds bit p of each.
struct Planes {
  uint32_t p[8];  // (7 in use: at most 127 placements)
  // adds x[0 .. 3] into planes 0 and 1 and returns the carry into plane 2
  __device__ __forceinline__ uint32_t four(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3) {
    const uint32_t c0 = maj3(p[0], x0, x1);
    p[0] = xor3(p[0], x0, x1);
    const uint32_t c1 = maj3(p[0], x2, x3);
    p[0] = xor3(p[0], x2, x3);
    const uint32_t c = maj3(p[1], c0, c1);
    p[1] = xor3(p[1], c0, c1);
    return c;
  }
  __device__ __forceinline__ void eight(uint32_t f0, uint32_t f1) {
    uint32_t c = maj3(p[2], f0, f1);
    p[2] = xor3(p[2], f0, f1);
#pragma unroll
    for (int i = 3; i < 7; ++i) {
      const uint32_t t = p[i] & c;
      p[i] ^= c;
      c = t;
    }
  }
  // planes to counts: byte b of p[i] becomes the count of candidate 8 b + i (8 x 8 transposes)
  __device__ __forceinline__ void bytes() {
#pragma unroll
    for (int h = 2; h >= 0; --h) {
      const int s = 1 << h;
      const uint32_t m = s == 4 ? 0x0f0f0f0fu : s == 2 ? 0x33333333u : 0x55555555u;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (i & s) continue;
        const uint32_t a = p[i], b = p[i + s];
        p[i] = __builtin_amdgcn_bitop3_b32(m, a, b << s, 0xCA);
        p[i + s] = __builtin_amdgcn_bitop3_b32(m, a >> s, b, 0xCA);
      }
    }
  }
};

// Placements k0 .. k1 - 1 (multiples of 4) of a tile, R2 pairs of slots each.  The entries of four
// placements are loaded one step ahead (up to 3 pairs: registers).
template <int R2>
__device__ __forceinline__ void count_tile(const uint32_t *__restrict__ e, int k0, int k1,
                                           const char *lds, Planes &A, Planes &B) {
  constexpr bool kAhead = R2 <= 3;
  uint32_t cur[4 * R2], nxt[4 * R2];
  auto load = [&](int k, uint32_t (&d)[4 * R2]) {
#pragma unroll
    for (int i = 0; i < 4 * R2; ++i) d[i] = e[(k * R2 + i) * 64];
  };
  auto four = [&](const uint32_t (&d)[4 * R2], uint32_t &fa, uint32_t &fb) {
    uint32_t xa[4], xb[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      xa[j] = xb[j] = 0xffffffffu;
#pragma unroll
      for (int i = 0; i < R2; ++i) {
        const uint32_t s = d[j * R2 + i];
        const uint2 u = *(const uint2 *)(lds + (s & 0xffffu)), v = *(const uint2 *)(lds + (s >> 16));
        xa[j] = __builtin_amdgcn_bitop3_b32(xa[j], u.x, v.x, 0x80);
        xb[j] = __builtin_amdgcn_bitop3_b32(xb[j], u.y, v.y, 0x80);
      }
    }
    fa = A.four(xa[0], xa[1], xa[2], xa[3]);
    fb = B.four(xb[0], xb[1], xb[2], xb[3]);
  };
  if (k0 >= k1) return;
  load(k0, cur);
  for (int k = k0; k < k1; k += 8) {
    uint32_t a0, b0, a1 = 0, b1 = 0;
    if constexpr (kAhead) load(min(k + 4, k1 - 4), nxt);  // past the end: the last step's again
    four(cur, a0, b0);
    if (k + 4 < k1) {
      if constexpr (kAhead) {
        load(min(k + 8, k1 - 4), cur);
        four(nxt, a1, b1);
      } else {
        load(k + 4, cur);
        four(cur, a1, b1);
      }
    }
    if constexpr (!kAhead) load(min(k + 8, k1 - 4), cur);
    A.eight(a0, a1);
    B.eight(b0, b1);
  }
}

// Sums of signed bytes.
__device__ __forceinline__ uint32_t add_bytes(uint32_t a, uint32_t b) {
  return ((a & 0x7f7f7f7fu) + (b & 0x7f7f7f7fu)) ^ ((a ^ b) & 0x80808080u);
}

}  // namespace

// One sector and phase for 32 candidates.  The pixels' words come from near (coalesced in runs of
// window rows), each level of segments is formed in LDS, then each wave takes a tile.
//
// The workgroups of one group of candidates follow each other on one XCD: the changes of a
// candidate are written in runs of a few vectors, which that XCD's L2 puts together (each XCD
// takes a contiguous range of the work).
//
// 4096 candidates of a 256 x 256 cell at cutoff 48, both phases: 113 us, where the walk of every
// placement (k_delta_diag) took 870.  The changes alone are 154 MB (31 us); vector work is 53 us,
// LDS 41 us, the rest is latency: a workgroup goes through five barriers.  Hence the loads in
// batches ahead of their barriers (151 -> 125 us) and two waves per tile (-> 113 us).
__global__ void __launch_bounds__(64 * kSwapWaves) __attribute__((amdgpu_waves_per_eu(6)))
k_swap(const uint2 *__restrict__ near, int npos, const SwapSector *__restrict__ sectors,
       int nsectors, const SwapTile *__restrict__ tiles, const int32_t *__restrict__ idx,
       const int32_t *__restrict__ rank, const uint32_t *__restrict__ pix, const uint32_t *__restrict__ segs,
       const uint32_t *__restrict__ ents, int K, int g0, int nph, unsigned phase_mask, int nv,
       int32_t *__restrict__ delta_out) {
  extern __shared__ uint2 slot[];
  const uint32_t total = gridDim.x, xcd = blockIdx.x & 7u, j = blockIdx.x >> 3;
  const uint32_t q = total >> 3, rem = total & 7u;
  const uint32_t u = xcd * q + min(xcd, rem) + j;
  const uint32_t per = (uint32_t)(nsectors * nph);
  const int g = (int)(u / per), si = (int)(u - g * per) / nph, p = (int)(u - g * per) % nph;
  const SwapSector &s = sectors[si];
  const uint2 *in = near + ((size_t)g * nph + p) * npos;
  const int npix = s.npix;
  if (threadIdx.x == 0) slot[0] = make_uint2(0, 0);
  // kBatch loads in flight, twice as many of segments (past the end: the last entry again; with
  // twice as many of both 2048 candidates at cutoff 32 take 34.5 us against 33.3)
  constexpr int kBatch = 2, kThreads = 64 * kSwapWaves;
  for (int i0 = threadIdx.x; i0 < npix; i0 += kThreads * kBatch) {
    uint32_t at[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) at[k] = pix[s.pix0 + min(i0 + k * kThreads, npix - 1)];
    uint2 v[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) v[k] = in[at[k]];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) slot[1 + min(i0 + k * kThreads, npix - 1)] = v[k];
  }
  int base = 1 + npix;
  const char *lds = (const char *)slot;
  for (int l = 1; l < kSwapLevels; ++l) {
    const int n = s.cnt[l];
    const uint32_t *e = segs + s.off[l];
    uint32_t d[2 * kBatch];  // the first entries are loaded before the level below is complete
    auto load = [&](int i0) {
#pragma unroll
      for (int k = 0; k < 2 * kBatch; ++k) d[k] = e[min(i0 + k * kThreads, n - 1)];
    };
    if (n) load(threadIdx.x);
    __syncthreads();
    for (int i0 = threadIdx.x; i0 < n; i0 += 2 * kThreads * kBatch) {
      if (i0 != (int)threadIdx.x) load(i0);
#pragma unroll
      for (int k = 0; k < 2 * kBatch; ++k) {
        const int i = i0 + k * kThreads;
        if (k && i >= n) break;
        const uint2 a = *(const uint2 *)(lds + (d[k] & 0xffffu)), b = *(const uint2 *)(lds + (d[k] >> 16));
        slot[base + i] = make_uint2(a.x & b.x, a.y & b.y);
      }
    }
    base += n;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  // longer tiles on other waves from sector to sector
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ti = (wave + si) & (kSwapTiles - 1), part = wave / kSwapTiles;
  Planes A{}, B{};
  const bool mine = ti < s.ntiles;
  const SwapTile &t = tiles[s.tile0 + (mine ? ti : 0)];
  if (mine) {
    const uint32_t *e = ents + t.off + lane;
    const int half = (t.nk + 4) / 8 * 4, ka = part ? half : 0, kb = part ? t.nk : half;
    switch (t.r2) {
      case 1: count_tile<1>(e, ka, kb, lds, A, B); break;
      case 2: count_tile<2>(e, ka, kb, lds, A, B); break;
      case 3: count_tile<3>(e, ka, kb, lds, A, B); break;
      case 4: count_tile<4>(e, ka, kb, lds, A, B); break;
      case 5: count_tile<5>(e, ka, kb, lds, A, B); break;
      case 6: count_tile<6>(e, ka, kb, lds, A, B); break;
      case 7: count_tile<7>(e, ka, kb, lds, A, B); break;
      default: count_tile<8>(e, ka, kb, lds, A, B); break;
    }
    A.bytes();
    B.bytes();
  }
  __syncthreads();  // the slots are free
  // changes as signed bytes, ch[i][rank]: candidates i, 8 + i, 16 + i, 24 + i; the two halves of
  // a tile's placements one after the other
  uint32_t *ch = (uint32_t *)slot;
  constexpr int kRanks = 64 * kSwapTiles;
  const bool phase1 = phase_mask != 1u && p == nph - 1;
  const int r = mine && lane < t.nvec ? rank[(s.tile0 + ti) * 64 + lane] : -1;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t u = phase1 ? B.p[i] : A.p[i], v = phase1 ? A.p[i] : B.p[i];
    A.p[i] = ((u | 0x80808080u) - v) ^ 0x80808080u;
    if (!part && r >= 0) ch[i * kRanks + r] = A.p[i];
  }
  __syncthreads();
  if (part && r >= 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) ch[i * kRanks + r] = add_bytes(ch[i * kRanks + r], A.p[i]);
  }
  __syncthreads();
  // a wave stores four of the eight words of 64 vectors
  const int v = (int)threadIdx.x & (kRanks - 1), i0 = wave / kSwapTiles * 4;
  if (v >= s.nvec) return;
  const int k0 = (g0 + g) * 32;
  int32_t *o = delta_out + ((size_t)k0 * nph + p) * nv;
  const int at = idx[s.idx0 + v];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t d = ch[(i0 + i) * kRanks + v];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int c = 8 * b + i0 + i;
      if (k0 + c < K) o[(size_t)c * nph * nv + at] = __builtin_amdgcn_sbfe((int)d, 8 * b, 8);
    }
  }
}

hipError_t launch_swap(const SwapLaunch &L, hipStream_t stream) {
  const int nph = L.phase_mask == 3 ? 2 : 1, npos = (2 * L.cx + 1) * (2 * L.cy + 1);
  const int groups = (L.K + 31) / 32, batch = swap_batch(L.cx, L.cy, L.phase_mask, L.K);
  const int waves = (2 * L.cy + kNearRows) / kNearRows;
  for (int g0 = 0; g0 < groups; g0 += batch) {
    const int n = std::min(batch, groups - g0);
    hipLaunchKernelGGL(k_swap_near, dim3((unsigned)(waves + 3) / 4, (unsigned)n), dim3(256), 0,
                       stream, L.bits, L.W, L.H, L.cx, L.cy, L.cand, L.K, g0, L.phase_mask,
                       (uint32_t *)L.near);
    hipLaunchKernelGGL(k_swap, dim3((unsigned)(n * L.nsectors * nph)), dim3(64 * kSwapWaves),
                       std::max((size_t)L.slots * sizeof(uint2), (size_t)32 * 64 * kSwapTiles), stream,
                       L.near, npos, L.sectors, L.nsectors,
                       L.tiles, L.idx, L.rank, L.pix, L.segs, L.ents, L.K, g0, nph, L.phase_mask, L.nv,
                       L.delta_out);
  }
  return hipGetLastError();
}

}  // namespace lpf
