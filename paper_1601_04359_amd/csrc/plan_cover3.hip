// Launch plans of the volume evaluation (host code): segments as a prefix tree.
//
// The digitised segments of neighbouring directions start alike: at cutoff 16 the 14 voxels of a
// segment in the mean are 4.5 nodes of the tree of all segments with the same signs and major
// axis.  The tree is walked in depth-first order; a product is saved at up to two branches above
// the current path, from which the paths below go on, and a segment that another one extends is
// counted on the way (the records are those of the 2-D walk, cover.h).
#include <algorithm>
#include <climits>
#include <cstdlib>
#include <cstring>
#include <exception>

#include "../../include/lpf.h"
#include "cover3.h"
#include "lpf_internal.h"
#include "parallel.h"
#include "row_dev.h"

namespace lpf {

namespace {

// A segment: n steps, each moving the major axis by one and minor axis a (bit 0) or b (bit 1) or
// both; step k in bits 63 - 2 k, 62 - 2 k, so that words of one class sort in depth-first order.
struct Seg {
  uint64_t key;
  int n, idx;
  int cls;  // mirror | down << 1, then the major axis
  // steps, then length: a number that sorts like the two
  uint64_t order() const {
    static_assert(kCover3Cut <= 24, "steps in the upper 48 bits of the key");
    return key | (uint64_t)n;
  }
};

int class_of(const int16_t *v) {
  const int a = std::abs(v[0]), b = std::abs(v[1]), c = std::abs(v[2]);
  const int maj = a >= b && a >= c ? 0 : (b >= c ? 1 : 2);
  return ((v[0] < 0) | (v[1] < 0) << 1) * 4 + maj;
}

Seg segment_of(const int16_t *v, int idx, int cls) {
  const int a[3] = {std::abs(v[0]), std::abs(v[1]), std::abs(v[2])};
  const int maj = cls & 3, n = a[maj];
  const int ma = maj == 0 ? a[1] : a[0], mb = maj == 2 ? a[1] : a[2];
  Seg s{0, n, idx, cls};
  int ea = n, eb = n;  // the rounding of the 2-D segments per minor axis
  for (int k = 0; k < n; ++k) {
    uint64_t st = 0;
    ea += 2 * ma;
    eb += 2 * mb;
    if (ea >= 2 * n) {
      ea -= 2 * n;
      st |= 1;
    }
    if (eb >= 2 * n) {
      eb -= 2 * n;
      st |= 2;
    }
    s.key |= st << (62 - 2 * k);
  }
  return s;
}

int common_steps(const Seg &a, const Seg &b) {
  if (a.cls != b.cls) return -1;  // not even the first voxel's step code means the same
  const int m = std::min(a.n, b.n);
  const uint64_t d = a.key ^ b.key;
  return d ? std::min(m, __builtin_clzll(d) / 2) : m;
}

// The records of a group's pieces.
class Walker {
 public:
  explicit Walker(const Cover3Shape &sh) : sh_(sh) {}
  // The records of segments s[0 .. n) (sorted, one mirror and down), slots from slot0 on.
  void piece(const Seg *s, int n, int slot0, std::vector<int4> &recs) {
    out_ = &recs;
    s_ = s;
    slot0_ = slot0;
    lcp_.resize(n);
    for (int i = 0; i + 1 < n; ++i) lcp_[i] = common_steps(s[i], s[i + 1]);
    int a = 0;
    for (int i = 0; i < n; ++i)
      if (i + 1 == n || lcp_[i] < 0) {
        nodes_.clear();
        stride_ = 0;
        for (int j = a; j <= i; ++j) stride_ = std::max(stride_, s_[j].n + 1);
        const int root = tree(a, i + 1);
        memo_.assign(nodes_.size() * 3 * stride_, kUnset);
        emit(root, 0, 0);
        a = i + 1;
      }
  }

 private:
  struct Node {
    int a, b, m;           // segments a .. b - 1 share their first m steps
    int kid = -1, next = -1;  // first child; next child of the same parent
  };
  const Seg *s_ = nullptr;
  const Cover3Shape &sh_;
  int slot0_ = 0;
  std::vector<int4> *out_ = nullptr;
  std::vector<int> lcp_;
  // costs by node, saves left and depth; at most kCover3Slots (kCover3Cut + 2) < 2^15
  std::vector<uint16_t> memo_;
  static constexpr uint16_t kUnset = 0xffff;
  int stride_ = 0;
  std::vector<Node> nodes_;

  int tree(int a, int b) {
    Node t{a, b, s_[a].n};
    for (int i = a; i + 1 < b; ++i) t.m = std::min(t.m, lcp_[i]);
    if (b - a > 1) {
      int c = s_[a].n == t.m ? a + 1 : a;  // a segment that ends here is counted at this node
      int last = -1;
      for (int i = c; i < b; ++i)
        if (i + 1 == b || lcp_[i] == t.m) {
          const int u = tree(c, i + 1);
          (last < 0 ? t.kid : nodes_[last].next) = u;
          last = u;
          c = i + 1;
        }
    }
    nodes_.push_back(t);
    return (int)nodes_.size() - 1;
  }
  // Steps (a save or a restore: one) of the walks below node v from a product of the first d
  // steps, k saves left.
  static constexpr int kCopy = 1;
  int cost(int v, int d, int k) {
    const Node &t = nodes_[v];
    if (t.kid < 0) return t.m - d + kCopy;
    uint16_t &c = memo_[((size_t)v * 3 + k) * stride_ + d];
    if (c != kUnset) return c;
    int x = unsaved(v, d, k);
    if (k > 0) x = std::min(x, saved(v, d, k));
    return c = (uint16_t)x;
  }
  int own(const Node &t, int d) const { return s_[t.a].n == t.m ? t.m - d + kCopy : 0; }
  int unsaved(int v, int d, int k) {
    const Node &t = nodes_[v];
    int c = own(t, d);
    for (int u = t.kid; u >= 0; u = nodes_[u].next) c += cost(u, d, k);
    return c;
  }
  int saved(int v, int d, int k) {
    const Node &t = nodes_[v];
    if (t.m == d) return INT_MAX;
    int c = t.m - d + 2 * kCopy;
    for (int u = t.kid; u >= 0; u = nodes_[u].next) c += cost(u, t.m, k - 1);
    return c;
  }
  // Step 0 of a record: voxel k of segment i (the lane's own voxel is in the start pixels).
  uint32_t code(int i, int k) const {
    const Seg &s = s_[i];
    const uint64_t steps = k ? s.key >> (64 - 2 * k) : 0;
    const int qa = __builtin_popcountll(steps & 0x5555555555555555ull);
    const int qb = __builtin_popcountll(steps & 0xaaaaaaaaaaaaaaaaull);
    const int maj = s.cls & 3, down = (s.cls >> 3) & 1;
    const int x = maj == 0 ? k : qa, y = maj == 1 ? k : (maj == 0 ? qa : qb), z = maj == 2 ? k : qb;
    return (uint32_t)(z * sh_.ps + (down ? sh_.cy - y : y) * sh_.rst + (x >> 5)) |
           (uint32_t)(x & 31) << 16;
  }
  // The walk of segment i from step d (saved at `level`, 0: the start) to step m; counted or not.
  void walk(int i, int d, int m, int level, bool count) {
    for (int k = d + 1, first = 1; k <= m || first; k += 2, first = 0) {
      // (the segment of one voxel: its own voxel again)
      int4 r = make_int4((int)code(i, std::min(k, m)), 0, 0, 0);
      if (k + 1 <= m) {
        r.y = (int)code(i, k + 1);
        r.x |= (int)kRecTwo;
      }
      if (first) r.x |= (level + 1) << kRecRestore;
      if (count && k + 2 > m) {
        r.x |= (int)kRecCount;
        r.z = slot0_ + i;
      }
      out_->push_back(r);
    }
  }
  void emit(int v, int d, int level) {
    const Node t = nodes_[v];
    std::vector<int4> &recs = *out_;
    const int k = 2 - level;
    if (t.kid < 0) {
      walk(t.a, d, t.m, level, true);
      recs.back().w = (int)recs.size();
      return;
    }
    const bool ends = s_[t.a].n == t.m;
    const size_t r0 = recs.size();
    if (k > 0 && t.m > d && saved(v, d, k) < unsaved(v, d, k)) {
      walk(t.a, d, t.m, level, ends);
      const size_t at = recs.size() - 1;
      recs[at].x |= (level + 1) << kRecSave;
      for (int u = t.kid; u >= 0; u = nodes_[u].next) emit(u, t.m, level + 1);
      recs[at].w = (int)recs.size();  // a zero count here: nothing below counts
    } else {
      if (ends) walk(t.a, d, t.m, level, true);
      const size_t at = recs.size() - 1;
      for (int u = t.kid; u >= 0; u = nodes_[u].next) emit(u, d, level);
      if (ends && recs.size() > r0) recs[at].w = (int)recs.size();
    }
  }
};

}  // namespace

bool plan_cover3(int W, int H, int D, int cx, int cy, int cz, const int16_t *vec, int64_t nv,
                 int lds, int cus, Cover3Host &p) {
  const int swd = (W + 31) / 32;
  if (std::max(cx, std::max(cy, cz)) > kCover3Cut || swd > 16) return false;
  p = Cover3Host{};
  Cover3Shape &sh = p.sh;
  sh.W = W;
  sh.H = H;
  sh.D = D;
  sh.cx = cx;
  sh.cy = cy;
  sh.cz = cz;
  sh.S = 1;
  while (4 * sh.S < swd) sh.S *= 2;
  sh.P = (swd + sh.S - 1) / sh.S;
  sh.wid = sh.P * sh.S + (cx >> 5) + 1;
  // rows an odd number of dwords apart and planes such that rows on both sides of a plane's end
  // keep the banks of consecutive rows
  sh.rst = sh.wid | 1;
  sh.ps = (H + cy) * sh.rst;
  sh.ps += (64 - cy * sh.rst % 64) % 64;
  const int avail = lds / 4 - 2 * kCover3Slots - kCoverPad;
  if ((int64_t)(cz + 1) * sh.ps > std::min(avail, 65535)) return false;
  const int zmax = std::min(D, avail / sh.ps - cz);
  sh.nslab = (D + zmax - 1) / zmax;
  sh.zb = (D + sh.nslab - 1) / sh.nslab;
  sh.nslab = (D + sh.zb - 1) / sh.zb;
  p.lds_bytes = (size_t)4 * ((size_t)(sh.zb + cz) * sh.ps + kCoverPad + 2 * kCover3Slots);
  // Waves that share a piece: as many as there are bands for.  A piece starts from nothing, so that
  // many pieces share little (60^3, cutoff 8: 37, 31 and 28 us with at most 4, 8 and 16 waves).
  const int band = 64 / sh.S * cover3_rows(sh.P, true), bands = (sh.zb * H + band - 1) / band;
  int nwb = 1;
  while (nwb < kCover3Waves && 2 * nwb <= bands) nwb *= 2;
  sh.npieces = kCover3Waves / nwb;

  // the segments class by class, sorted in each; a thread for about 3 000 of them
  std::vector<Seg> seg((size_t)nv);
  {
    constexpr int kClasses = 16;
    int64_t at[kClasses + 1] = {}, fill[kClasses];
    std::vector<uint8_t> cls((size_t)nv);
    for (int64_t i = 0; i < nv; ++i) ++at[(cls[i] = (uint8_t)class_of(vec + 3 * i)) + 1];
    for (int c = 0; c < kClasses; ++c) fill[c] = at[c + 1] += at[c];
    std::vector<int> by((size_t)nv);
    for (int64_t i = nv; i-- > 0;) by[--fill[cls[i]]] = (int)i;
    parallel(kClasses, (int)std::min<int64_t>(6, 1 + nv / 3000), [&](int c) {
      const int64_t a = at[c], n = at[c + 1] - a;
      std::vector<std::pair<uint64_t, int>> order((size_t)n);
      std::vector<Seg> own((size_t)n);
      for (int64_t i = 0; i < n; ++i) {
        own[i] = segment_of(vec + 3 * by[a + i], by[a + i], c);
        order[i] = {own[i].order(), (int)i};
      }
      std::sort(order.begin(), order.end());
      for (int64_t i = 0; i < n; ++i) seg[a + i] = own[order[i].second];
    });
  }
  // groups of about equal work (steps not shared with the segment before, and a count), cut where
  // the signs change; one workgroup per compute unit, since each stages its slab and starts its
  // trees anew (60^3, cutoff 8: 28 us, with two 41, with four 66; 100^3, cutoff 16: 555, 563, 597)
  std::vector<int64_t> work((size_t)nv + 1, 0);
  for (int64_t i = 0; i < nv; ++i) {
    const int shared = i ? std::max(0, common_steps(seg[i - 1], seg[i])) : 0;
    work[i + 1] = work[i] + 3 + (seg[i].n - shared);
  }
  const int want = std::max(1, cus / sh.nslab);
  int ncls = 1;  // signs of dx and dy that occur
  for (int64_t i = 1; i < nv; ++i) ncls += seg[i].cls / 4 != seg[i - 1].cls / 4;
  std::vector<std::pair<int64_t, int64_t>> cut;
  for (int64_t a = 0; a < nv;) {
    int64_t e = a;
    while (e < nv && seg[e].cls / 4 == seg[a].cls / 4) ++e;  // one mirror and down
    const int64_t w = work[e] - work[a];
    const int ng = (int)std::max<int64_t>(1 + w * std::max(0, want - ncls) / work[nv],
                                             (e - a + kCover3Slots - 1) / kCover3Slots);
    int64_t s = a;
    for (int g = 0; g < ng; ++g) {
      int64_t t = s;
      const int64_t to = work[a] + w * (g + 1) / ng;
      while (t < e && (g + 1 == ng || work[t + 1] <= to) && t - s < kCover3Slots) ++t;
      if (t > s) cut.push_back({s, t});
      s = t;
    }
    while (s < e) {  // what the slots left over
      const int64_t t = std::min<int64_t>(e, s + kCover3Slots);
      cut.push_back({s, t});
      s = t;
    }
    a = e;
  }
  const int ng = (int)cut.size();
  std::vector<std::vector<int4>> recs((size_t)ng);
  std::vector<std::vector<int32_t>> off((size_t)ng);
  // A thread for about 1 000 segments (starting one takes as long as planning 200 of them), a few
  // runs of groups each.
  const int threads = (int)std::min<int64_t>(16, 1 + nv / 1000), runs = std::min(ng, 8 * threads);
  parallel(runs, threads, [&](int run) {
    Walker w(sh);
    for (int g = (int)((int64_t)ng * run / runs); g < (int)((int64_t)ng * (run + 1) / runs); ++g) {
      const int64_t a = cut[g].first, e = cut[g].second;
      recs[g].reserve((size_t)(4 * (e - a)));
      off[g].reserve((size_t)sh.npieces + 1);
      int64_t s = a;
      for (int k = 0; k < sh.npieces; ++k) {
        off[g].push_back((int32_t)recs[g].size());
        const int64_t to = work[a] + (work[e] - work[a]) * (k + 1) / sh.npieces;
        int64_t t = s;
        while (t < e && (k + 1 == sh.npieces || work[t + 1] <= to)) ++t;
        if (t > s) w.piece(seg.data() + s, (int)(t - s), (int)(s - a), recs[g]);
        s = t;
      }
      off[g].push_back((int32_t)recs[g].size());
    }
  });
  size_t nrec = 2;
  for (const auto &r : recs) nrec += r.size();
  p.recs.reserve(nrec);
  for (int g = 0; g < ng; ++g) {
    const Seg &s = seg[cut[g].first];
    const int32_t base = (int32_t)p.recs.size();
    Cover3Group G{};
    G.piece0 = (int32_t)p.piece_off.size();
    G.mem0 = (int32_t)p.mems.size();
    G.nmem = (int32_t)(cut[g].second - cut[g].first);
    G.mirror = (s.cls >> 2) & 1;
    G.down = (s.cls >> 3) & 1;
    p.groups.push_back(G);
    for (int32_t o : off[g]) p.piece_off.push_back(base + o);
    for (int4 r : recs[g]) {
      if (r.x & (int)kRecCount) r.w += base;
      p.recs.push_back(r);
    }
    for (int64_t i = cut[g].first; i < cut[g].second; ++i) p.mems.push_back(seg[i].idx);
  }
  p.recs.push_back(make_int4(0, 0, 0, 0));  // records are read up to two past a piece
  p.recs.push_back(make_int4(0, 0, 0, 0));
  return true;
}

namespace {

// The plan run on the host for one phase, every access checked.  False when one is out of bounds.
bool run_cover3(const Cover3Host &p, const uint8_t *vol, int phase, uint32_t *counts) {
  const Cover3Shape &s = p.sh;
  const int rpw = 64 / s.S, SP = s.S * s.P, Q = cover3_rows(s.P, false), wpr = 2 * ((s.W + 63) / 64);
  const std::vector<uint32_t> rows = packed_rows(vol, s.W, s.D * s.H, wpr);
  std::vector<uint32_t> lds(p.lds_bytes / 4);
  const size_t rows_end = lds.size() - 2 * kCover3Slots;
  for (const Cover3Group &g : p.groups) {
    for (int slab = 0; slab < s.nslab; ++slab) {
      const int Z0 = slab * s.zb, planes = std::min(s.zb, s.D - Z0);
      std::fill(lds.begin(), lds.end(), 0x5a5a5a5au);  // cells that are not staged: any value
      const int hh = s.H + s.cy, total = (planes + s.cz) * hh;
      for (int t = 0; t < 64 * kCover3Waves; ++t)
        for (Cover3Cell c(t, s.wid, hh); c.pr < total; c.next(s.wid, hh)) {
          const size_t at = (size_t)c.pl * s.ps + (size_t)c.yh * s.rst + c.e;
          const size_t row = c.row(s, g.down != 0, Z0);
          if (at >= rows_end || row >= (size_t)s.D * s.H) return false;
          const uint32_t v = periodic32(rows.data() + row * wpr, s.W, word_start(s.W, c.e, g.mirror != 0));
          lds[at] = (phase ? 0u : ~0u) ^ (g.mirror ? bit_reverse(v) : v);
        }
      for (int pc = 0; pc < s.npieces; ++pc) {
        const int r0 = p.piece_off[g.piece0 + pc], r1 = p.piece_off[g.piece0 + pc + 1];
        const int nrows = planes * s.H, bands = (nrows + rpw * Q - 1) / (rpw * Q);
        for (int band = 0; band < bands; ++band) {
          const int nw = 64 * Q * s.P;
          std::vector<uint32_t> st((size_t)nw, 0), A, S1, S2;
          std::vector<size_t> base((size_t)nw);
          for (int l = 0; l < 64; ++l)
            for (int q = 0; q < Q; ++q)
              for (int i = 0; i < s.P; ++i) {
                const int r = (band * Q + q) * rpw + l % rpw, w = l / rpw * s.P + i;
                const int row = r < nrows ? r : 0;
                const int j = (l * Q + q) * s.P + i;
                base[j] = (size_t)(row / s.H) * s.ps + (size_t)(row % s.H) * s.rst + w;
                const size_t own = base[j] + (g.down ? (size_t)s.cy * s.rst : 0);
                if (own >= rows_end || w >= SP) return false;
                const int left = s.W - 32 * w;
                st[j] = r < nrows && left > 0 ? lds[own] & (left >= 32 ? ~0u : (1u << left) - 1) : 0;
              }
          for (int r = r0; r < r1;) {
            const int4 rec = p.recs.at(r);
            switch (((uint32_t)rec.x >> kRecRestore) & 3) {
              case 1: A = st; break;
              case 2: A = S1; break;
              case 3: A = S2; break;
            }
            if (A.size() != st.size()) return false;
            for (int t = 0; t < ((uint32_t)rec.x & kRecTwo ? 2 : 1); ++t) {
              const uint32_t c = (uint32_t)(t ? rec.y : rec.x);
              for (int j = 0; j < nw; ++j) {
                const size_t at = base[j] + (c & 0xffff);
                if (at + 1 >= rows_end) return false;
                const uint64_t v = (uint64_t)lds[at] | (uint64_t)lds[at + 1] << 32;
                A[j] &= (uint32_t)(v >> ((c >> 16) & 31));
              }
            }
            const int save = ((uint32_t)rec.x >> kRecSave) & 3;
            if (save == 1) S1 = A;
            if (save == 2) S2 = A;
            ++r;
            if ((uint32_t)rec.x & kRecCount) {
              if (rec.z < 0 || rec.z >= g.nmem || rec.w < r || rec.w > r1) return false;
              uint32_t n = 0;
              for (uint32_t a : A) n += (uint32_t)__builtin_popcount(a);
              counts[p.mems[g.mem0 + rec.z]] += n;
              if (!n) r = rec.w;
            }
          }
        }
      }
    }
  }
  return true;
}

}  // namespace
}  // namespace lpf

extern "C" lpf_status lpf_cover3_counts(const uint8_t *vol, int W, int H, int D, int cx, int cy,
                                        int cz, int phase, uint32_t *counts) {
  if (!vol || !counts || W < 1 || H < 1 || D < 1 || W > 1024 || H > 1024 || D > 1024 || cx < 0 ||
      cy < 0 || cz < 0 || cx >= W || cy >= H || cz >= D || phase < 0 || phase > 1)
    return LPF_E_INVAL;
  try {
    const int64_t nv = lpf_num_vectors3(cx, cy, cz);
    std::vector<int16_t> vec((size_t)3 * nv);
    if (lpf_vectors3(cx, cy, cz, vec.data()) != LPF_OK) return LPF_E_INVAL;
    lpf::Cover3Host p;
    if (!lpf::plan_cover3(W, H, D, cx, cy, cz, vec.data(), nv, 160 * 1024, 256, p))
      return LPF_E_UNSUPPORTED;
    std::vector<int> seen((size_t)nv, 0);
    for (int32_t m : p.mems) ++seen[m];
    for (int t : seen)
      if (t != 1) return LPF_E_INVAL;
    std::fill(counts, counts + nv, 0u);
    if (!lpf::run_cover3(p, vol, phase, counts)) return LPF_E_INVAL;
  } catch (const std::exception &) {
    return LPF_E_NOMEM;
  }
  return LPF_OK;
}
