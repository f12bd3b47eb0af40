// Full evaluation of the lineal path function on gfx950: paths covered by words.
//
// The paper's Alg. "L2_eval" tests, for every segment and every translation, the segment's
// pixels one by one.  Here 32 translations (start pixels) share one 32-bit word, a lane owns R
// consecutive words of one row, and for a path with pixel offsets p_k the lane forms
//     A = AND_k (image shifted by p_k)    -> bit b set <=> every pixel of the segment is in phase
// and popcounts A.  One phase is counted per workgroup (the staged image is complemented for
// phase 0), so every product is an AND.
//
// Which pixels are taken together is the plan's work (plan_cover.hip): a workgroup owns a group
// of neighbouring slopes and, for each row tile, stages the rows in LDS with their periodic halo,
// builds up to kCoverWords masks beside them (mask bit = the AND over a pixel pattern that the
// group's paths repeat, from that pixel on), and its waves walk the group's prefix trees.  A
// record is one or two steps (a funnel shift per word and step, one 3-input AND per word for two
// steps), after which a count may be taken and the product be saved; a later record can go on
// from a saved product.  Records are wave-uniform and read on the scalar unit.
//
// A count of zero over the wave's rows ends everything that extends that path there (the paper's
// enhanced evaluation, Sec. 3.2): the walk goes on at the record's jump target.
#include "cover.h"
#include "row_dev.h"
#include "walk_dev.h"

namespace lpf {

namespace {

// A plan's tables other than the records are read through the constant address space: their
// wave-uniform reads become scalar loads (plain loads went through the vector memory path).
#define LPF_CONST __attribute__((address_space(4)))
template <class T>
__device__ __forceinline__ const LPF_CONST T *constant(const T *p) {
  return (const LPF_CONST T *)p;
}

// The start pixels of a lane's words: full words below the row's last one, which keeps the bits
// below W mod 32; none for rows past the image; with a position set its members (srow: the row's
// mask words, k_start_sets).
template <int R, bool SAMPLE>
__device__ __forceinline__ void start_pixels(uint32_t (&A)[R], int w0, int W, bool row_ok,
                                             const uint32_t *__restrict__ srow) {
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int left = W - 32 * (w0 + i);  // pixels of the row from this word on
    const bool some = row_ok && left > 0;
    if constexpr (SAMPLE) {
      A[i] = some ? srow[w0 + i] : 0u;
    } else {
      A[i] = some ? (left >= 32 ? 0xffffffffu : (1u << left) - 1u) : 0u;
    }
  }
}

// The records [r0, r1) for the lane's R words of one row (walk_dev.h): the walk of one piece over
// one band.
typedef uint32_t Words2 __attribute__((ext_vector_type(2)));
typedef uint32_t Words4 __attribute__((ext_vector_type(4)));
typedef uint32_t Words8 __attribute__((ext_vector_type(8)));
typedef uint32_t Words16 __attribute__((ext_vector_type(16)));

template <int R>
__device__ __forceinline__ void walk(const int4 *recs, int r0, int r1, uint32_t base,
                                     const uint32_t (&st)[R], uint32_t slots) {
#if __HIP_DEVICE_COMPILE__
#define LPF_WALK(n, WordsK, m, a, s1, s2, d0, x0, d1, x1)                                         \
  {                                                                                               \
    WordsK M = 0u, A, S1, S2, D0, D1;                                                             \
    Words2 X0, X1;                                                                                \
    for (int i = 0; i < R; ++i) M[i] = st[i];                                                     \
    asm volatile(LPF_WALK_ASM                                                                     \
                 : "=&{" a "}"(A), "=&{" s1 "}"(S1), "=&{" s2 "}"(S2), "=&{" d0 "}"(D0),          \
                   "=&{" x0 "}"(X0), "=&{" d1 "}"(D1), "=&{" x1 "}"(X1)                           \
                 : "{" m "}"(M), "{v24}"(base), [K] "i"(n), [KD] "i"(n + 1), [R] "i"(R),        \
                   [Q] "i"(1), [P] "i"(R), [PD] "i"(R + 1), [MV] "i"(R), [recs] "s"(recs), [r0] "s"(r0), [r1] "s"(r1),          \
                   [slots] "s"(slots)                                                             \
                 : "s72", "s73", "s74", "s75", "s76", "s77", "s78", "s79", "s80", "s82", "s83",   \
                   "s84", "s85", "s86", "s88", "s89", "s90", "vcc", "scc", "memory");             \
  }
  if constexpr (R <= 4) {
    LPF_WALK(4, Words4, "v[28:31]", "v[32:35]", "v[36:39]", "v[40:43]", "v[44:47]", "v[48:49]",
             "v[50:53]", "v[54:55]")
  } else if constexpr (R <= 8) {
    LPF_WALK(8, Words8, "v[28:35]", "v[36:43]", "v[44:51]", "v[52:59]", "v[60:67]", "v[68:69]",
             "v[70:77]", "v[78:79]")
  } else {
    LPF_WALK(16, Words16, "v[28:43]", "v[44:59]", "v[60:75]", "v[76:91]", "v[92:107]",
             "v[108:109]", "v[110:125]", "v[126:127]")
  }
#undef LPF_WALK
#endif
}

// Count of vector `idx` = (dx, dy) for phase slot p, in the image's output layout (the GRID
// layout also fills -v, eq. (symmetry)); ADD: a part of it (several workgroups per group), added
// to entries that are zero before the launch.
template <bool ADD>
__device__ __forceinline__ void put_count(const CoverImg &I, uint32_t *__restrict__ out, int p,
                                          const MemDesc &v, uint32_t c) {
  auto put = [&](size_t i) {
    if constexpr (ADD) {
      if (c) atomicAdd(out + i, c);
    } else {
      out[i] = c;
    }
  };
  if (I.layout == 0) {
    put((size_t)p * I.nv + v.idx);
  } else {
    const int gw = 2 * I.cx + 1;
    const size_t g = (size_t)gw * (2 * I.cy + 1);
    const size_t i = (size_t)p * g + (size_t)(v.dy + I.cy) * gw + (v.dx + I.cx);
    const size_t j = (size_t)p * g + (size_t)(I.cy - v.dy) * gw + (I.cx - v.dx);
    put(i);
    if (j != i) put(j);
  }
}

// One mask of C consecutive dwords per lane and item: item i is chunk i / rows of row i mod rows,
// so that a wave's lanes read consecutive rows (distinct banks), C + 1 dwords for C funnel
// shifts.  The last chunk of a row is moved back to end with the row (its overlap is written
// twice with the same values).  (Four steps at a time, their reads under way together, with the
// steps of a mask padded to a multiple of four, were slower: 1 024 x 1 024, cutoff 512: 5.9
// against 5.6 ms.)
template <int C>
__device__ __forceinline__ void build_mask(const LPF_CONST CoverGroup &g, const LPF_CONST uint32_t *bops,
                                           int b0, int b1, uint32_t *__restrict__ lds,
                                           uint32_t *__restrict__ dst) {
  const int items = cover_mask_items<C>(g.wid, g.rows);
  for (int i = threadIdx.x; i < items; i += blockDim.x) {
    const int at = cover_mask_item<C>(g, i);
    uint32_t v[C];
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] = 0xffffffffu;
    for (int b = b0; b < b1; ++b) {
      const uint32_t op = bops[b];
      const uint32_t *q = lds + at + (op & 0xffffu);
      const uint32_t sh = (op >> 16) & 31u;
      uint32_t t[C + 1];
#pragma unroll
      for (int c = 0; c <= C; ++c) t[c] = q[c];
#pragma unroll
      for (int c = 0; c < C; ++c) v[c] &= funnel(t[c + 1], t[c], (int)sh);
    }
#pragma unroll
    for (int c = 0; c < C; ++c) dst[at + c] = v[c];
  }
}

// One group of one phase over the tiles split, split + nsplit, ... of the image (one workgroup).
// phase 1 counts set pixels, phase 0 clear ones; p: the phase's place in the output.
template <int R, bool SAMPLE>
__device__ __forceinline__ void cover_group(const CoverImg &I, int gi, int phase, int p, int split,
                                            const uint64_t *__restrict__ bits,
                                            const uint32_t *__restrict__ sample,
                                            uint32_t *__restrict__ out,
                                            uint32_t *__restrict__ lds) {
  const LPF_CONST CoverGroup &g = constant(I.groups)[gi];
  const LPF_CONST int32_t *piece_off = constant(I.piece_off) + g.piece0;
  const LPF_CONST uint32_t *bops = constant(I.bops);
  const int ntiles = g.ntiles * I.nct;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rpw = 64 / I.S;
  const int strip = lane / rpw, r_in = lane - strip * rpw;
  const int SR = I.S * R;
  uint32_t *slots = lds + (1 + g.nw) * g.asz + kCoverPad;
  for (int t = tid; t < g.nmem; t += nt) slots[t] = 0u;
  const int wpr = 2 * ((I.W + 63) >> 6);
  const int swd = (I.W + 31) >> 5;
  const uint32_t *rows = reinterpret_cast<const uint32_t *>(bits);
  const uint32_t flip = phase ? 0u : 0xffffffffu;
  const bool mirror = g.mirror != 0;
  const int nwb = g.nwb;
  const int piece = wave / nwb, bw = wave - piece * nwb;
  const int r0 = piece_off[piece], r1 = piece_off[piece + 1];
  const int cells = g.rows * g.wid;
  for (int tile = split; tile < ntiles; tile += I.nsplit) {
    const int ct = tile / g.ntiles;
    const int e0 = ct * SR;
    const int Y0 = (tile - ct * g.ntiles) * g.tile;
    __syncthreads();  // every wave is done with the previous tile
    // rows Y0 .. Y0 + rows - 1 (mod H): a word per lane, so that a wave reads along the rows
    for (int i = tid; i < cells; i += nt) {
      int y, e;
      cover_cell(g, i, y, e);
      int r = Y0 + y;
      if (r >= I.H) r -= I.H;
      if (r >= I.H) r %= I.H;
      const uint32_t v = periodic32(rows + (size_t)r * wpr, I.W, word_start(I.W, e0 + e, mirror));
      lds[y * g.rst + e] = flip ^ (mirror ? bit_reverse(v) : v);
    }
    for (int a = 1; a <= g.nw; ++a) {
      __syncthreads();
      build_mask<cover_mask_words(R)>(g, bops, g.bop[a - 1], g.bop[a], lds, lds + a * g.asz);
    }
    __syncthreads();
    const int rows_here = min(g.tile, I.H - Y0);
    if (r0 < r1) {
      for (int row0 = bw * rpw; row0 < rows_here; row0 += nwb * rpw) {
        const int row = row0 + r_in;
        const bool row_ok = row < rows_here;
        const uint32_t *srow =
            SAMPLE ? sample + (size_t)((mirror ? I.H : 0) + Y0 + (row_ok ? row : 0)) * swd : nullptr;
        uint32_t st[R];
        start_pixels<R, SAMPLE>(st, e0 + strip * R, I.W, row_ok, srow);
        walk<R>(I.recs, r0, r1, lds_address(lds + row * g.rst + strip * R), st, lds_address(slots));
      }
    }
  }
  __syncthreads();
  if (I.nsplit == 1) {
    for (int t = tid; t < g.nmem; t += nt) put_count<false>(I, out, p, I.mems[g.mem0 + t], slots[t]);
  } else {
    for (int t = tid; t < g.nmem; t += nt) put_count<true>(I, out, p, I.mems[g.mem0 + t], slots[t]);
  }
}

__global__ void k_cover_zero(uint32_t *__restrict__ out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = 0u;
}

// The counts that several workgroups add to, zeroed in one launch for a whole batch: image
// blockIdx.y's, when its groups are split.
__global__ void k_cover_zero_batch(const CoverImg *__restrict__ imgs,
                                   const int64_t *__restrict__ counts_off, int nph,
                                   uint32_t *__restrict__ counts) {
  const CoverImg &I = imgs[blockIdx.y];
  if (I.nsplit <= 1) return;
  const int64_t n = (int64_t)nph * (I.layout == 0 ? (int64_t)I.nv
                                                  : (int64_t)(2 * I.cx + 1) * (2 * I.cy + 1));
  uint32_t *out = counts + counts_off[blockIdx.y];
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = 0u;
}

// Start pixels of a Monte-Carlo position set as mask words: [0] rows as they are, [1] rows
// reversed (for the mirrored groups); bits past W clear.
__global__ void k_start_sets(const uint32_t *__restrict__ src, int W, int H, int swd, int wpr,
                             uint32_t *__restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 2 * H * swd) return;
  const int r = i / swd, e = i - r * swd;
  const bool mirror = r >= H;
  const uint32_t *row = src + (size_t)(mirror ? r - H : r) * wpr;
  const int left = W - 32 * e;
  uint32_t v = periodic32(row, W, word_start(W, e, mirror));
  if (mirror) v = bit_reverse(v);
  out[i] = v & (left >= 32 ? 0xffffffffu : (1u << left) - 1u);
}

// Workgroups go to the eight XCDs in turn.  The phases of an image differ in work (a zero count
// ends a walk), so both phases of an item go to the same XCD: eight items of one phase, then the
// same eight of the other.  (With the phase in the lowest bit, one phase was counted on
// the even XCDs and the other on the odd ones: 512^2, cutoff 128: 0.27 against 0.15 ms.)
template <int R, bool SAMPLE>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4)))
k_cover(CoverImg I, const int2 *__restrict__ items, int n_items, unsigned phase_mask,
        const uint64_t *__restrict__ bits, const uint32_t *__restrict__ sample,
        uint32_t *__restrict__ out) {
  extern __shared__ uint32_t lds[];
  const bool both = phase_mask == 3u;
  const int b = blockIdx.x;
  const int p = both ? (b >> 3) & 1 : 0;
  const int i = both ? (b >> 4) * 8 + (b & 7) : b;
  if (i >= n_items) return;
  const int2 it = items[i];
  cover_group<R, SAMPLE>(I, it.x, both ? p : (int)(phase_mask >> 1), p, it.y, bits, sample, out, lds);
}

__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4)))
k_cover_batch(const CoverImg *__restrict__ imgs, const int64_t *__restrict__ bits_off,
              const int64_t *__restrict__ counts_off, const int4 *__restrict__ items,
              unsigned phase_mask, const uint64_t *__restrict__ pool,
              uint32_t *__restrict__ counts) {
  extern __shared__ uint32_t lds[];
  const int4 it = items[blockIdx.x];
  const CoverImg &I = imgs[it.x];
  const uint64_t *bits = pool + bits_off[it.x];
  uint32_t *out = counts + counts_off[it.x];
  const int phase = it.z, p = phase_mask == 3u ? phase : 0;
  switch (I.R) {
#define LPF_R(r) \
  case r: cover_group<r, false>(I, it.y, phase, p, it.w, bits, nullptr, out, lds); break;
    LPF_R(1) LPF_R(2) LPF_R(3) LPF_R(4) LPF_R(5) LPF_R(6) LPF_R(7) LPF_R(8)
    LPF_R(9) LPF_R(10) LPF_R(11) LPF_R(12) LPF_R(13) LPF_R(14) LPF_R(15) LPF_R(16)
#undef LPF_R
  }
}

using CoverKernel = void (*)(CoverImg, const int2 *, int, unsigned, const uint64_t *,
                             const uint32_t *, uint32_t *);
CoverKernel cover_kernel(int R, bool sample) {
  switch (R) {
#define LPF_R(r) \
  case r: return sample ? k_cover<r, true> : k_cover<r, false>;
    LPF_R(1) LPF_R(2) LPF_R(3) LPF_R(4) LPF_R(5) LPF_R(6) LPF_R(7) LPF_R(8)
    LPF_R(9) LPF_R(10) LPF_R(11) LPF_R(12) LPF_R(13) LPF_R(14) LPF_R(15) LPF_R(16)
#undef LPF_R
  }
  return nullptr;
}

}  // namespace

hipError_t launch_cover(const CoverImg &I, const CoverShape &sh, const int2 *items, int n_items,
                        size_t lds_bytes, unsigned phase_mask, const uint64_t *bits,
                        const uint32_t *sample, uint32_t *out, hipStream_t stream) {
  const CoverKernel k = cover_kernel(I.R, sample != nullptr);
  if (!k || I.R != sh.R || I.S != sh.S || sh.wpg < 1 || sh.wpg > 16 || 64 % I.S)
    return hipErrorInvalidValue;
  const int nph = phase_mask == 3u ? 2 : 1;
  if (I.nsplit > 1) {
    const int64_t n = (int64_t)nph * (I.layout == 0 ? (int64_t)I.nv
                                                    : (int64_t)(2 * I.cx + 1) * (2 * I.cy + 1));
    hipLaunchKernelGGL(k_cover_zero, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)),
                       dim3(256), 0, stream, out, n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int blocks = nph == 2 ? (n_items + 7) / 8 * 16 : n_items;
  hipLaunchKernelGGL(k, dim3(blocks), dim3(64 * sh.wpg), lds_bytes, stream, I, items, n_items,
                     phase_mask, bits, sample, out);
  return hipGetLastError();
}

hipError_t launch_start_sets(const uint64_t *sample, int W, int H, uint32_t *out,
                             hipStream_t stream) {
  const int swd = (W + 31) / 32, n = 2 * H * swd;
  hipLaunchKernelGGL(k_start_sets, dim3((n + 255) / 256), dim3(256), 0, stream,
                     reinterpret_cast<const uint32_t *>(sample), W, H, swd, 2 * ((W + 63) / 64), out);
  return hipGetLastError();
}

hipError_t launch_cover_zero(const CoverImg *imgs, const int64_t *counts_off, int n_images,
                             unsigned phase_mask, uint32_t *counts, hipStream_t stream) {
  hipLaunchKernelGGL(k_cover_zero_batch, dim3(64, n_images), dim3(256), 0, stream, imgs,
                     counts_off, phase_mask == 3u ? 2 : 1, counts);
  return hipGetLastError();
}

hipError_t launch_cover_batch(const CoverImg *imgs, const int64_t *bits_off,
                              const int64_t *counts_off, const int4 *items, int n_items, int wpg,
                              size_t lds_bytes, unsigned phase_mask, const uint64_t *pool,
                              uint32_t *counts, hipStream_t stream) {
  hipLaunchKernelGGL(k_cover_batch, dim3(n_items), dim3(64 * wpg), lds_bytes, stream, imgs,
                     bits_off, counts_off, items, phase_mask, pool, counts);
  return hipGetLastError();
}

hipError_t prepare_cover_kernels(int max_lds_bytes) {
  hipError_t e = hipFuncSetAttribute((const void *)k_cover_batch,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, max_lds_bytes);
  for (int R = 1; R <= 16; ++R)
    for (int s = 0; s < 2; ++s) {
      hipError_t r = hipFuncSetAttribute((const void *)cover_kernel(R, s),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, max_lds_bytes);
      if (r != hipSuccess) e = r;
    }
  return e;
}

}  // namespace lpf
