// Lineal path function of a periodic 3-D volume (the extension of Sec. 2; with cz = 0 it is the
// sum over the xy-cuts of their 2-D functions, the ensemble of cuts of Sec. 6.3): segments as a
// prefix tree (plan_cover3.hip).
//
// 32 start voxels of one x-row share a word; a lane owns P words of Q rows.  A workgroup stages a
// slab (zb start planes and the cz planes and cy rows behind them, reversed for dx < 0) and its
// waves walk their pieces of the group's tree over the slab's rows.  In the staged slab a voxel of
// a segment is a constant offset from the start row, so the walk is that of the 2-D evaluation
// (walk_dev.h), with several rows per lane, because a record costs about 30 scalar and 12 vector
// instructions beside those per word, and, for both phases, both products: a step's dwords are
// read and shifted once (one phase per workgroup: 1366 us against 587).
//
// 100 x 100 x 100, cutoff 16, both phases: 555 us, vector work 400 and LDS 300 of them; with every
// voxel of every segment walked (k_lpf3_slab: 14 per vector, here 6.2 steps) 880.
#include <algorithm>

#include "cover3.h"
#include "lpf_internal.h"
#include "row_dev.h"
#include "walk_dev.h"

namespace lpf {

namespace {

typedef uint32_t Bases __attribute__((ext_vector_type(4)));
typedef uint32_t Start4 __attribute__((ext_vector_type(4)));
typedef uint32_t Start8 __attribute__((ext_vector_type(8)));
typedef uint32_t Start12 __attribute__((ext_vector_type(12)));
typedef uint32_t Start16 __attribute__((ext_vector_type(16)));
static_assert(kCover3Slots * 4 == 4096, "the offset in LPF_WALK_BOTH below");

// The records [r0, r1) for Q rows of P words per lane; BOTH: the start words of phase 1, then those
// of phase 0.
template <int P, int Q, bool BOTH>
__device__ __forceinline__ void walk3(const int4 *recs, int r0, int r1, const uint32_t (&base)[Q],
                                      const uint32_t (&st)[Q * P * (BOTH ? 2 : 1)], uint32_t slots) {
#if __HIP_DEVICE_COMPILE__
  constexpr int K = Q * P * (BOTH ? 2 : 1), PD = (P + 2) / 2 * 2;
  Bases B = 0u;
  for (int q = 0; q < Q; ++q) B[q] = base[q];
// (the registers above the start words are the walk's)
#define LPF_V10(t) "v" t "0", "v" t "1", "v" t "2", "v" t "3", "v" t "4", "v" t "5", "v" t "6", "v" t "7", "v" t "8", "v" t "9"
#define LPF_WALK3(StartK, m, text, ...)                                                           \
  {                                                                                               \
    StartK M = 0u;                                                                                \
    for (int i = 0; i < K; ++i) M[i] = st[i];                                                     \
    asm volatile(text                                                                             \
                 :                                                                                \
                 : "{" m "}"(M), "{v[24:27]}"(B), [K] "i"(K), [KD] "i"(Q * PD + 1),               \
                   [R] "i"(Q * P), [Q] "i"(Q), [P] "i"(P), [PD] "i"(PD), [MV] "i"(K),             \
                   [recs] "s"(recs), [r0] "s"(r0), [r1] "s"(r1), [slots] "s"(slots)               \
                 : "s72", "s73", "s74", "s75", "s76", "s77", "s78", "s79", "s80", "s82", "s83",   \
                   "s84", "s85", "s86", "s88", "s89", "s90", "vcc", "scc", "memory", __VA_ARGS__); \
  }
#define LPF_WALK3_ANY(StartK, m, ...)                                                             \
  {                                                                                               \
    if constexpr (BOTH)                                                                           \
      LPF_WALK3(StartK, m, LPF_WALK_BOTH("4096"), __VA_ARGS__)                                    \
    else                                                                                          \
      LPF_WALK3(StartK, m, LPF_WALK_ASM, __VA_ARGS__)                                             \
  }
  // last register: 28 + 4 K + 2 (Q PD + 1) + 2
  static_assert(28 + 4 * K + 2 * (Q * PD + 1) + 2 <= 121, "registers");
  if constexpr (K <= 4) {
    static_assert(28 + 4 * K + 2 * (Q * PD + 1) + 2 <= 69 || K > 4, "registers");
    LPF_WALK3_ANY(Start4, "v[28:31]", "v32", "v33", "v34", "v35", "v36", "v37", "v38", "v39",
                  LPF_V10("4"), LPF_V10("5"), LPF_V10("6"))
  } else if constexpr (K <= 8) {
    static_assert(28 + 4 * K + 2 * (Q * PD + 1) + 2 <= 99 || K > 8, "registers");
    LPF_WALK3_ANY(Start8, "v[28:35]", "v36", "v37", "v38", "v39", LPF_V10("4"), LPF_V10("5"),
                  LPF_V10("6"), LPF_V10("7"), LPF_V10("8"), LPF_V10("9"))
  } else if constexpr (K <= 12) {
    LPF_WALK3_ANY(Start12, "v[28:39]", LPF_V10("4"), LPF_V10("5"), LPF_V10("6"), LPF_V10("7"),
                  LPF_V10("8"), LPF_V10("9"), LPF_V10("10"), LPF_V10("11"), "v120", "v121")
  } else {
    LPF_WALK3_ANY(Start16, "v[28:43]", "v44", "v45", "v46", "v47", "v48", "v49", LPF_V10("5"),
                  LPF_V10("6"), LPF_V10("7"), LPF_V10("8"), LPF_V10("9"), LPF_V10("10"),
                  LPF_V10("11"), "v120", "v121")
  }
#undef LPF_WALK3_ANY
#undef LPF_WALK3
#undef LPF_V10
#endif
}

template <int P, bool BOTH>
__global__ void __launch_bounds__(64 * kCover3Waves) __attribute__((amdgpu_waves_per_eu(4)))
k_cover3(Cover3Shape g, const Cover3Group *__restrict__ groups,
         const int32_t *__restrict__ piece_off, const int4 *__restrict__ recs,
         const int32_t *__restrict__ mems, int ngroups, int nv, const uint32_t *__restrict__ bits,
         unsigned phase_mask, uint32_t *__restrict__ counts) {
  extern __shared__ uint32_t lds[];
  constexpr int Q = cover3_rows(P, BOTH);
  const int slab = blockIdx.x / ngroups, gi = blockIdx.x - slab * ngroups;
  const Cover3Group gr = groups[gi];
  const uint32_t flip = phase_mask == 1u ? 0xffffffffu : 0u;
  const int Z0 = slab * g.zb, planes = min(g.zb, g.D - Z0);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t *slots = lds + (g.zb + g.cz) * g.ps + kCoverPad;
  for (int t = tid; t < 2 * kCover3Slots; t += 64 * kCover3Waves) slots[t] = 0u;
  const int HH = g.H + g.cy, wpr = 2 * ((g.W + 63) >> 6);
  const int total = (planes + g.cz) * HH;
  for (Cover3Cell c(tid, g.wid, HH); c.pr < total; c.next(g.wid, HH)) {
    const uint32_t v = periodic32(bits + c.row(g, gr.down != 0, Z0) * wpr, g.W,
                                  word_start(g.W, c.e, gr.mirror != 0));
    lds[c.pl * g.ps + c.yh * g.rst + c.e] = flip ^ (gr.mirror ? bit_reverse(v) : v);
  }
  __syncthreads();
  const int nwb = kCover3Waves / g.npieces, piece = wave / nwb, bw = wave - piece * nwb;
  const int r0 = __builtin_amdgcn_readfirstlane(piece_off[gr.piece0 + piece]);
  const int r1 = __builtin_amdgcn_readfirstlane(piece_off[gr.piece0 + piece + 1]);
  if (r0 < r1) {
    const int rpw = 64 / g.S, strip = lane / rpw, r_in = lane - strip * rpw;
    const int rows = planes * g.H, down = gr.down ? g.cy * g.rst : 0;
    for (int row0 = bw * rpw * Q; row0 < rows; row0 += nwb * rpw * Q) {
      uint32_t base[Q], st[Q * P * (BOTH ? 2 : 1)];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int r = row0 + q * rpw + r_in, row = r < rows ? r : 0;
        const int z = row / g.H;
        const uint32_t *at = lds + z * g.ps + (row - z * g.H) * g.rst + strip * P;
        base[q] = lds_address(at);
#pragma unroll
        for (int i = 0; i < P; ++i) {
          const int left = g.W - 32 * (strip * P + i);  // voxels of the row from this word on
          const uint32_t m = left >= 32 ? 0xffffffffu : left > 0 ? (1u << left) - 1u : 0u;
          const uint32_t own = at[down + i], some = r < rows ? m : 0u;
          st[q * P + i] = own & some;
          if constexpr (BOTH) st[(Q + q) * P + i] = ~own & some;
        }
      }
      walk3<P, Q, BOTH>(recs, r0, r1, base, st, lds_address(slots));
    }
  }
  __syncthreads();
  for (int t = tid; t < gr.nmem; t += 64 * kCover3Waves) {
    uint32_t *out = counts + mems[gr.mem0 + t];
    const uint32_t c = slots[t], c0 = slots[kCover3Slots + t];
    if constexpr (BOTH) {  // phase 0 first
      if (c0) atomicAdd(out, c0);
      out += nv;
    }
    if (c) atomicAdd(out, c);
  }
}

__global__ void k_cover3_zero(uint32_t *__restrict__ counts, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) counts[i] = 0;
}

using Cover3Kernel = void (*)(Cover3Shape, const Cover3Group *, const int32_t *, const int4 *,
                              const int32_t *, int, int, const uint32_t *, unsigned, uint32_t *);
Cover3Kernel cover3_kernel(int P, bool both) {
  switch (P) {
    case 1: return both ? k_cover3<1, true> : k_cover3<1, false>;
    case 2: return both ? k_cover3<2, true> : k_cover3<2, false>;
    case 3: return both ? k_cover3<3, true> : k_cover3<3, false>;
    default: return both ? k_cover3<4, true> : k_cover3<4, false>;
  }
}

}  // namespace

hipError_t launch_cover3(const Cover3Launch &L, hipStream_t stream) {
  const int nph = L.phase_mask == 3u ? 2 : 1;
  const int64_t n = (int64_t)nph * L.nv;
  hipLaunchKernelGGL(k_cover3_zero, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream,
                     L.counts, n);
  hipLaunchKernelGGL(cover3_kernel(L.sh.P, nph == 2), dim3((unsigned)(L.ngroups * L.sh.nslab)), dim3(64 * kCover3Waves),
                     L.lds_bytes, stream, L.sh, L.groups, L.piece_off, L.recs, L.mems, L.ngroups,
                     L.nv, reinterpret_cast<const uint32_t *>(L.bits), L.phase_mask, L.counts);
  return hipGetLastError();
}

hipError_t prepare_cover3_kernels(int max_lds_bytes) {
  hipError_t e = hipSuccess;
  for (int i = 0; i < 8; ++i) {
    const hipError_t r = hipFuncSetAttribute((const void *)cover3_kernel(i / 2 + 1, i & 1),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, max_lds_bytes);
    if (r != hipSuccess) e = r;
  }
  return e;
}

}  // namespace lpf
