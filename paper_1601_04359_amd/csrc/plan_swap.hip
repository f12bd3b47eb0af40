// Launch plans of the interchange delta (host code): placements from shared segments.
//
// The change of a vector's count under an interchange is a sum over the placements of its path
// through either changed pixel (k_swap.hip): path pixel k on the changed pixel, k = 0 .. n.  All
// placements of all vectors lie in one window around the pixel, and neighbouring slopes and
// placements run through the same short digitised segments.  A segment is a first pixel and its
// steps; the plan lists the distinct ones of 1, 2, 4 and 8 pixels, each the AND of two of half its
// length, and each placement as the AND of the segments of 8 pixels that cover it (the last one
// overlapping).  At cutoff 48 a placement of 34 pixels in the mean is then 4.7 reads, and its share
// of the segments 0.8 more.  Segments of 16 pixels would halve the reads, but they are about as many
// as the placements (22 000 of 40 000 in an octant), and fewer vectors fit in LDS: 4096 candidates
// at cutoff 48 take 123 us with 8 pixels, 135 with 6, 157 with 4, 174 with 16.
//
// A sector is a range of directions whose pixels and segments fit in the LDS of a workgroup.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <exception>
#include <stdexcept>

#include "../../include/lpf.h"
#include "lpf_internal.h"
#include "parallel.h"
#include "row_dev.h"
#include "swap.h"

namespace lpf {

namespace {

// Distinct keys in the order of their first use.
class Interner {
 public:
  Interner() : table_(1024, -1) {}
  int find_or_add(uint64_t key, bool &fresh) {
    if (2 * (keys_.size() + 1) > table_.size()) grow();
    size_t h = hash(key);
    while (table_[h] >= 0) {
      if (keys_[table_[h]] == key) {
        fresh = false;
        return table_[h];
      }
      h = (h + 1) & (table_.size() - 1);
    }
    fresh = true;
    table_[h] = (int)keys_.size();
    keys_.push_back(key);
    return table_[h];
  }
  const std::vector<uint64_t> &keys() const { return keys_; }

 private:
  size_t hash(uint64_t k) const {
    return (size_t)((k * 0x9E3779B97F4A7C15ull) >> 32) & (table_.size() - 1);
  }
  void grow() {
    std::vector<int>(table_.size() * 2, -1).swap(table_);
    for (size_t i = 0; i < keys_.size(); ++i) {
      size_t h = hash(keys_[i]);
      while (table_[h] >= 0) h = (h + 1) & (table_.size() - 1);
      table_[h] = (int)i;
    }
  }
  std::vector<int> table_;
  std::vector<uint64_t> keys_;
};

struct Vec {
  int idx, dx, dy;
  int rank = 0;  // among its sector's vectors in canonical order
  int n() const { return std::max(std::abs(dx), dy); }
};

// The segments of one sector: level l has 2^l pixels.
struct Builder {
  int cx, cy;
  Interner lev[kSwapLevels];
  std::vector<std::pair<int, int>> parts[kSwapLevels];
  std::vector<SwapTile> tiles;
  std::vector<int32_t> rank;
  std::vector<std::pair<int, int>> reads;  // (level, segment) of every tile, in the order of ents
  // the current vector: its pixels and the steps from each pixel on (bit t: the minor coordinate
  // moves between pixels st + t and st + t + 1)
  int oct = 0, n = 0;
  std::vector<int> px, py;
  std::vector<uint64_t> steps;

  Builder(int cx_, int cy_) : cx(cx_), cy(cy_) {}

  void set(const Vec &v) {
    const int ax = std::abs(v.dx);
    const bool flat = ax >= v.dy;
    n = flat ? ax : v.dy;
    const int m = flat ? v.dy : ax;
    oct = (flat ? 0 : 1) | (v.dx < 0 ? 2 : 0);
    px.resize(n + 1);
    py.resize(n + 1);
    steps.assign(n + 2, 0);
    for (int k = 0; k <= n; ++k) {
      const int y = n ? (int)((2LL * k * m + n) / (2LL * n)) : 0;  // eq. (segments)
      px[k] = (v.dx < 0 ? -1 : 1) * (flat ? k : y);
      py[k] = flat ? y : k;
    }
    for (int k = n - 1; k >= 0; --k) {
      const bool s = flat ? py[k + 1] != py[k] : px[k + 1] != px[k];
      steps[k] = (steps[k + 1] << 1) | (s ? 1 : 0);
    }
  }
  // Segment of level l from path pixel st, of the placement with pixel k on the changed pixel.
  int segment(int l, int st, int k) {
    const int len = 1 << l;
    const uint64_t at = (uint64_t)(py[st] - py[k] + cy) * (2 * cx + 1) + (px[st] - px[k] + cx);
    const uint64_t key = len == 1 ? at << 34
                                  : (at << 34) | (uint64_t)oct << 32 |
                                        (steps[st] & (((uint64_t)1 << (len - 1)) - 1));
    bool fresh;
    const int s = lev[l].find_or_add(key, fresh);
    if (fresh) {
      if (l == 0) {
        parts[0].push_back({0, 0});
      } else {
        const int a = segment(l - 1, st, k), b = segment(l - 1, st + len / 2, k);
        parts[l].push_back({a, b});
      }
    }
    return s;
  }
  // The placements of vectors v[0 .. nv) as one tile.
  void tile(const Vec *v, int nv) {
    SwapTile t{};
    t.nvec = nv;
    int nk = 1, r = 1;
    for (int i = 0; i < nv; ++i) {
      const int p = v[i].n() + 1;
      nk = std::max(nk, p);
      r = std::max(r, p >= kSwapLen ? (p + kSwapLen - 1) / kSwapLen : 2);
    }
    t.nk = (nk + 3) / 4 * 4;
    t.r2 = (r + 1) / 2;
    const size_t base = reads.size();
    reads.resize(base + (size_t)t.nk * t.r2 * 2 * 64, {-1, 0});
    for (int i = 0; i < nv; ++i) {
      set(v[i]);
      const int p = n + 1;
      int l = kSwapLevels - 1;
      while ((1 << l) > p) --l;
      const int len = 1 << l, nr = (p + len - 1) / len;
      for (int k = 0; k <= n; ++k)
        for (int j = 0; j < 2 * t.r2; ++j) {
          const int st = std::min(std::min(j, nr - 1) * len, p - len);
          reads[base + (((size_t)k * t.r2 + j / 2) * 64 + i) * 2 + (j & 1)] = {l, segment(l, st, k)};
        }
    }
    for (int i = 0; i < 64; ++i) rank.push_back(i < nv ? v[i].rank : 0);
    tiles.push_back(t);
  }
  int slots() const {
    size_t s = 1;
    for (int l = 0; l < kSwapLevels; ++l) s += lev[l].keys().size();
    return (int)std::min<size_t>(s, 1 << 30);
  }
};

// A sector's tables with slots assigned: within a level by position, then steps, so that lanes
// (neighbouring vectors or segments) read neighbouring slots.
struct SectorTables {
  SwapSector s;
  std::vector<uint32_t> pix, segs, ents;
  std::vector<SwapTile> tiles;
  std::vector<int32_t> rank, idx;
  int slots = 0;
};

void finish(Builder &b, SectorTables &o) {
  std::vector<int> slot[kSwapLevels];
  int base = 1;
  o.s = SwapSector{};
  for (int l = 0; l < kSwapLevels; ++l) {
    const std::vector<uint64_t> &keys = b.lev[l].keys();
    std::vector<std::pair<uint64_t, int>> ord(keys.size());
    for (size_t i = 0; i < keys.size(); ++i) ord[i] = {keys[i], (int)i};
    std::sort(ord.begin(), ord.end());
    slot[l].resize(keys.size());
    for (size_t i = 0; i < ord.size(); ++i) slot[l][ord[i].second] = base + (int)i;
    if (l == 0) {
      o.s.npix = (int)keys.size();
      for (const auto &e : ord) o.pix.push_back((uint32_t)(e.first >> 34));
    } else {
      o.s.off[l] = (int32_t)o.segs.size();
      o.s.cnt[l] = (int32_t)keys.size();
      for (const auto &e : ord) {
        const std::pair<int, int> &p = b.parts[l][e.second];
        o.segs.push_back((uint32_t)slot[l - 1][p.first] * 8 |
                         (uint32_t)slot[l - 1][p.second] * 8 << 16);
      }
    }
    base += (int)keys.size();
  }
  o.slots = base;
  o.ents.resize(b.reads.size() / 2);
  auto at = [&](const std::pair<int, int> &r) {
    return r.first < 0 ? 0u : (uint32_t)slot[r.first][r.second] * 8;
  };
  for (size_t i = 0; i < o.ents.size(); ++i)
    o.ents[i] = at(b.reads[2 * i]) | at(b.reads[2 * i + 1]) << 16;
  int off = 0;
  for (SwapTile &t : b.tiles) {
    t.off = off;
    off += t.nk * t.r2 * 64;
  }
  o.tiles = std::move(b.tiles);
  o.rank = std::move(b.rank);
}

}  // namespace

bool plan_swap(int cx, int cy, size_t max_bytes, SwapHost &p) {
  const int c = std::max(cx, cy);
  if (c > kSwapMaxCut) return false;
  const int64_t nv = lpf_num_vectors(cx, cy);
  {
    // placements, at most c + 1 of c + 1 pixels per vector
    const double ents = (double)nv * (c + 1) * ((c + 1 + 2 * kSwapLen - 1) / (2 * kSwapLen));
    if (ents * sizeof(uint32_t) > (double)max_bytes) return false;
  }
  std::vector<int16_t> can((size_t)2 * nv);
  if (lpf_vectors(cx, cy, can.data()) != LPF_OK) return false;
  std::vector<Vec> v((size_t)nv);
  std::vector<double> ang((size_t)nv);
  for (int64_t i = 0; i < nv; ++i) {
    v[i] = Vec{(int)i, can[2 * i], can[2 * i + 1]};
    ang[i] = std::atan2((double)v[i].dy, (double)v[i].dx);
  }
  std::vector<int> by((size_t)nv);
  for (int64_t i = 0; i < nv; ++i) by[i] = (int)i;
  std::sort(by.begin(), by.end(),
            [&](int a, int b) { return ang[a] != ang[b] ? ang[a] < ang[b] : a < b; });
  // sectors of equally many vectors, 64 per wave at most; halved when one does not fit in LDS
  int want = (int)((nv + 64 * kSwapTiles - 1) / (64 * kSwapTiles));
  std::vector<SectorTables> out;
  for (;; want *= 2) {
    out.assign((size_t)want, SectorTables{});
    std::vector<char> bad((size_t)want, 0);
    parallel(want, 16, [&](int s) {
      const int64_t i0 = nv * s / want, i1 = nv * (s + 1) / want;
      std::vector<Vec> mine;
      for (int64_t i = i0; i < i1; ++i) mine.push_back(v[by[i]]);
      std::sort(mine.begin(), mine.end(), [](const Vec &a, const Vec &b) { return a.idx < b.idx; });
      for (size_t i = 0; i < mine.size(); ++i) {
        mine[i].rank = (int)i;
        out[s].idx.push_back(mine[i].idx);
      }
      // by length: the lanes of a tile read about as many placements and segments
      std::sort(mine.begin(), mine.end(), [](const Vec &a, const Vec &b) {
        return a.n() != b.n() ? a.n() < b.n() : a.idx < b.idx;
      });
      Builder b(cx, cy);
      const int m = (int)mine.size(), nt = std::max(1, (m + 63) / 64);
      for (int t = 0; t < nt; ++t) {
        const int t0 = m * t / nt, t1 = m * (t + 1) / nt;
        if (t1 > t0) b.tile(mine.data() + t0, t1 - t0);
      }
      if (b.slots() > kSwapSlots)
        bad[s] = 1;
      else
        finish(b, out[s]);
    });
    if (std::find(bad.begin(), bad.end(), 1) == bad.end()) break;
    if (want > nv) return false;
  }
  p = SwapHost{};
  p.cx = cx;
  p.cy = cy;
  for (SectorTables &o : out) {
    o.s.pix0 = (int32_t)p.pix.size();
    for (int l = 1; l < kSwapLevels; ++l) o.s.off[l] += (int32_t)p.segs.size();
    o.s.tile0 = (int32_t)p.tiles.size();
    o.s.ntiles = (int32_t)o.tiles.size();
    o.s.idx0 = (int32_t)p.idx.size();
    o.s.nvec = (int32_t)o.idx.size();
    for (SwapTile &t : o.tiles) t.off += (int32_t)p.ents.size();
    p.pix.insert(p.pix.end(), o.pix.begin(), o.pix.end());
    p.segs.insert(p.segs.end(), o.segs.begin(), o.segs.end());
    p.ents.insert(p.ents.end(), o.ents.begin(), o.ents.end());
    p.tiles.insert(p.tiles.end(), o.tiles.begin(), o.tiles.end());
    p.rank.insert(p.rank.end(), o.rank.begin(), o.rank.end());
    p.idx.insert(p.idx.end(), o.idx.begin(), o.idx.end());
    p.sectors.push_back(o.s);
    p.slots = std::max(p.slots, o.slots);
  }
  return true;
}

namespace {

// The plan run on the host, one interchange (a the phase-1 pixel) at a time, every table entry
// checked against its array.  False when an entry is out of range or reads a slot that is not
// written yet.
bool run_swap(const SwapHost &p, const uint8_t *img, int W, int H, int a, int b, int64_t nv,
              int32_t *d0, int32_t *d1) {
  const int w = 2 * p.cx + 1, h = 2 * p.cy + 1, nd = 2 * ((W + 63) / 64);
  const std::vector<uint32_t> rows = packed_rows(img, W, H, nd);
  // the window around a and around b per phase, in words of 32 columns as k_swap_near writes them
  std::vector<uint8_t> win[2][2];
  for (int side = 0; side < 2; ++side) {
    const int sx = (side ? b : a) % W, sy = (side ? b : a) / W;
    for (auto &v : win[side]) v.resize((size_t)w * h);
    for (int r = 0; r < h; ++r) {
      const int y = (sy + r - p.cy + H) % H;
      int x = (sx - p.cx + W) % W;
      for (int w0 = 0; w0 < w; w0 += 32, x = (x + 32) % W) {
        const uint32_t v = row_word(rows.data() + (size_t)y * nd, nd, W, x);
        const uint32_t v1 = v | (y == b / W ? every((b % W - x + W) % W, W) : 0u);
        const uint32_t v0 = ~v | (y == a / W ? every((a % W - x + W) % W, W) : 0u);
        for (int t = 0; t < 32 && w0 + t < w; ++t) {
          win[side][1][(size_t)r * w + w0 + t] = v1 >> t & 1;
          win[side][0][(size_t)r * w + w0 + t] = v0 >> t & 1;
        }
      }
    }
  }
  std::vector<int> seen((size_t)nv, 0);
  std::vector<uint8_t> val((size_t)p.slots);
  for (const SwapSector &s : p.sectors) {
    std::vector<int> cnt((size_t)4 * 64 * s.ntiles, 0);
    for (int side = 0; side < 2; ++side)
      for (int ph = 0; ph < 2; ++ph) {
        int slot = 0;
        val[slot++] = 0;
        for (int i = 0; i < s.npix; ++i) {
          const uint32_t at = p.pix[s.pix0 + i];
          if (at >= (uint32_t)(w * h) || slot >= p.slots) return false;
          val[slot++] = win[side][ph][at];
        }
        for (int l = 1; l < kSwapLevels; ++l) {
          const int done = slot;
          for (int i = 0; i < s.cnt[l]; ++i) {
            const uint32_t e = p.segs[s.off[l] + i];
            const int u = (int)(e & 0xffff), t = (int)(e >> 16);
            if (u % 8 || t % 8 || u / 8 >= done || t / 8 >= done || slot >= p.slots) return false;
            val[slot++] = val[u / 8] & val[t / 8];
          }
        }
        for (int t = 0; t < s.ntiles; ++t) {
          const SwapTile &T = p.tiles[s.tile0 + t];
          if (T.nvec < 1 || T.nvec > 64 || T.nk % 4 || T.r2 < 1 || T.r2 > kSwapReads / 2 || T.nk > kSwapMaxCut + 4) return false;
          for (int k = 0; k < T.nk; ++k)
            for (int i = 0; i < 64; ++i) {
              int v = 1;
              for (int j = 0; j < T.r2; ++j) {
                const uint32_t e = p.ents.at((size_t)T.off + ((size_t)k * T.r2 + j) * 64 + i);
                const int u = (int)(e & 0xffff), q = (int)(e >> 16);
                if (u % 8 || q % 8 || u / 8 >= slot || q / 8 >= slot) return false;
                v &= val[u / 8] & val[q / 8];
              }
              cnt[((size_t)t * 64 + i) * 4 + 2 * ph + side] += v;
            }
        }
      }
    for (int t = 0; t < s.ntiles; ++t)
      for (int i = 0; i < 64; ++i) {
        const int *n = &cnt[((size_t)t * 64 + i) * 4];
        if (i >= p.tiles[s.tile0 + t].nvec) {
          if (n[0] | n[1] | n[2] | n[3]) return false;
          continue;
        }
        const int rank = p.rank[(size_t)(s.tile0 + t) * 64 + i];
        if (rank < 0 || rank >= s.nvec || s.nvec > 64 * kSwapTiles) return false;
        const int ix = p.idx[s.idx0 + rank];
        if (ix < 0 || ix >= nv || seen[ix]++) return false;
        d0[ix] = n[0] - n[1];
        d1[ix] = n[3] - n[2];
      }
  }
  return std::find(seen.begin(), seen.end(), 0) == seen.end();
}

}  // namespace
}  // namespace lpf

extern "C" lpf_status lpf_swap_plan_delta(const uint8_t *img, int W, int H, int cx, int cy, int a,
                                          int b, int32_t *delta) {
  if (!img || !delta || W < 1 || H < 1 || W > 4096 || H > 4096 || cx < 0 || cy < 0 || cx >= W ||
      cy >= H || a < 0 || b < 0 || a >= W * H || b >= W * H || !img[a] || img[b])
    return LPF_E_INVAL;
  try {
    lpf::SwapHost p;
    if (!lpf::plan_swap(cx, cy, SIZE_MAX, p)) return LPF_E_UNSUPPORTED;
    const int64_t nv = lpf_num_vectors(cx, cy);
    if (!lpf::run_swap(p, img, W, H, a, b, nv, delta, delta + nv)) return LPF_E_INVAL;
  } catch (const std::exception &) {
    return LPF_E_NOMEM;
  }
  return LPF_OK;
}
