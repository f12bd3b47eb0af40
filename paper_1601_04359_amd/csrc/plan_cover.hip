// Launch plans of the full evaluation (host code): paths covered by shared words.
//
// Counting one vector means AND-ing the image, shifted to each pixel of the vector's digitised
// path.  Two facts make most of these pixels free:
//  * Paths of neighbouring slopes start alike.  The walked paths of one octant, in the order of
//    their slopes, form a prefix tree; a product taken at a branch is kept in registers and every
//    path below the branch goes on from it.  A shorter vector whose path is a prefix of a longer
//    one (Sec. 3.2) is a node on the way and is counted there.
//  * An AND may take a pixel twice.  A digitised line of a narrow range of slopes repeats a few
//    pixel patterns (words) all along, so with the product of a word kept for every pixel of the
//    staged rows (one mask array in LDS), a step takes the whole word at once, and overlapping
//    words cover a path exactly: greedily, the step that reaches furthest without passing the
//    next count.
// At cutoff 128 both together leave 2.6 steps per vector (86 without them, 38 with prefixes
// shared by whole chains only).
//
// A group is a range of slopes of one octant with up to kCoverWords words, walked by one
// workgroup; a piece is the part of it that one wave walks.  Vectors with dx < 0 are walked on the
// mirrored image, so every offset is >= 0, with the words and records of the group of dx >= 0.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdlib>
#include <exception>

#include "../../include/lpf.h"
#include "cover.h"
#include "parallel.h"
#include "row_dev.h"

namespace lpf {

namespace {

// A walked path: the first len + 1 pixels of the line of slope m / n (minor over major), and the
// members counted on it.
struct Path {
  int n, m, len, m0, nm;
  int q(int k) const { return n ? (int)((2ll * k * m + n) / (2ll * n)) : 0; }
};

// The vectors of an octant with dx < 0 lie on the same paths on the mirrored image, but for the
// axis, the first `axis` paths: it holds no vector with dx < 0 (the longest one takes all of it).
struct Octant {
  bool xm = true;
  std::vector<Path> paths;   // by slope, then length
  std::vector<MemDesc> mems;
  int axis = 0;
};

// Canonical index of (dx, dy): [0,cx] x [0,cy] row by row, then [-cx,-1] x [1,cy].
int64_t index_of(int cx, int cy, int dx, int dy) {
  if (dx >= 0) return (int64_t)dy * (cx + 1) + dx;
  return (int64_t)(cx + 1) * (cy + 1) + (int64_t)(dy - 1) * cx + (dx + cx);
}

// The vectors of one octant as walked paths: longest first, each with the vectors not yet taken
// whose paths are its prefixes (u = pixel k of the walk, a prefix when u's slope lies in the
// interval of slopes that digitise to pixels 0..k; see plan_full.hip).  The octant owns the
// vectors dx >= 0 with dx >= dy (xm) or dx < dy, so that octants are independent.
void build_octant(int cx, int cy, bool xm, Octant &o) {
  o.xm = xm;
  const int N = xm ? cx : cy, M = xm ? cy : cx;
  auto put = [&](int k, int q) {
    const int dx = xm ? k : q, dy = xm ? q : k;
    o.mems.push_back(MemDesc{(int32_t)index_of(cx, cy, dx, dy), (int16_t)dx, (int16_t)dy, k});
  };
  const bool zero = xm ? (cx > 0 || cy == 0) : (cx == 0 && cy > 0);
  if (zero && N == 0) {  // the 1 x 1 domain: the zero vector alone
    o.paths.push_back(Path{0, 0, 0, 0, 1});
    put(0, 0);
    o.axis = 1;
    return;
  }
  bool zero_done = !zero;
  std::vector<char> placed((size_t)(N + 1) * (M + 1), 0);
  for (int n = N; n >= 1; --n) {
    const int mhi = std::min(xm ? n : n - 1, M);
    for (int m = 0; m <= mhi; ++m) {
      if (placed[(size_t)n * (M + 1) + m]) continue;
      Path p{n, m, n, (int)o.mems.size(), 0};
      if (!zero_done) {
        put(0, 0);
        zero_done = true;
      }
      // slopes that digitise to the pixels so far: [lp / lq, hp / hq)
      int64_t lp = -1, lq = 1, hp = (int64_t)1 << 30, hq = 1;
      int err = n, q = 0;
      for (int k = 1; k < n; ++k) {
        err += 2 * m;
        if (err >= 2 * n) {
          err -= 2 * n;
          ++q;
        }
        if ((xm || q < k) && !(q * lq < lp * k) && q * hq < hp * k) {
          char &t = placed[(size_t)k * (M + 1) + q];
          if (!t) {
            t = 1;
            put(k, q);
          }
        }
        if (lp * 2 * k < (2 * q - 1) * lq) {
          lp = 2 * q - 1;
          lq = 2 * k;
        }
        if ((2 * q + 1) * hq < hp * 2 * k) {
          hp = 2 * q + 1;
          hq = 2 * k;
        }
      }
      put(n, m);
      p.nm = (int)o.mems.size() - p.m0;
      // paths with many members (axes, diagonals: one per pixel) are cut into several walks
      constexpr int kCut = kCoverSlots / 4;
      for (int j0 = 0; j0 < p.nm; j0 += kCut) {
        Path c = p;
        c.m0 = p.m0 + j0;
        c.nm = std::min(kCut, p.nm - j0);
        c.len = o.mems[c.m0 + c.nm - 1].l;
        o.paths.push_back(c);
      }
    }
  }
  std::sort(o.paths.begin(), o.paths.end(), [](const Path &a, const Path &b) {
    const int64_t x = (int64_t)a.m * b.n, y = (int64_t)b.m * a.n;
    return x != y ? x < y : a.len < b.len;
  });
  while (o.axis < (int)o.paths.size() && o.paths[o.axis].m == 0) ++o.axis;
}

// Steps of a path along the minor axis, bit k - 1 = q_k - q_{k-1}; bit_words(len) words.
inline int bit_words(int len) { return (len >> 6) + 2; }
void letters(const Path &p, int len, uint64_t *b) {
  std::fill(b, b + bit_words(len), 0);
  int err = p.n;
  for (int k = 0; k < len; ++k) {
    err += 2 * p.m;
    if (err >= 2 * p.n) {
      err -= 2 * p.n;
      b[k >> 6] |= 1ull << (k & 63);
    }
  }
}
inline uint64_t bits64(const uint64_t *b, int j) {
  const int w = j >> 6, s = j & 63;
  return s ? (b[w] >> s) | (b[w + 1] << (64 - s)) : b[w];
}
int common(const uint64_t *a, const uint64_t *b, int len) {
  for (int w = 0; w * 64 < len; ++w) {
    const uint64_t d = a[w] ^ b[w];
    if (d) return std::min(len, w * 64 + __builtin_ctzll(d));
  }
  return len;
}

// A word: L steps (L + 1 pixels).
struct Word {
  int L = 0;
  const uint64_t *b = nullptr;
};
// Letters j .. j + L - 1 of b as a word in `at`, bit_words(L) words.
Word sub_word(const uint64_t *b, int j, int L, uint64_t *at) {
  std::fill(at, at + bit_words(L), 0);
  for (int k = 0; k < L; k += 64) {
    uint64_t v = bits64(b, j + k);
    if (L - k < 64) v &= (1ull << (L - k)) - 1;
    at[k >> 6] = v;
  }
  return Word{L, at};
}
// Where a word starts on a path: bit j of occ (words of 64 pixels, occ_words(len) of them).
inline int occ_words(int len) { return (len >> 6) + 1; }
void find_word(const uint64_t *b, int len, const Word &w, uint64_t *occ) {
  const int top = len - w.L;  // the last pixel where the word fits
  for (int x = 0; x < occ_words(len); ++x) {
    uint64_t o = 0;
    if (64 * x <= top) {
      o = top - 64 * x >= 63 ? ~0ull : (2ull << (top - 64 * x)) - 1;
      // (64 x + t <= len, so the reads end in the path's spare word)
      for (int t = 0; t < w.L && o; ++t) {
        const uint64_t l = bits64(b, 64 * x + t);
        o &= (w.b[t >> 6] >> (t & 63)) & 1 ? l : ~l;
      }
    }
    occ[x] = o;
  }
}
// The last start at pixel <= at, -1 when there is none from pixel `from` on (or before).
inline int last_start(const uint64_t *occ, int at, int from) {
  int w = at >> 6;
  uint64_t x = occ[w] & (~0ull >> (63 - (at & 63)));
  const int w0 = std::max(from, 0) >> 6;
  while (!x && w > w0) x = occ[--w];
  return x ? 64 * w + 63 - __builtin_clzll(x) : -1;
}

// The furthest step from a path covered below pixel c that does not pass pixel `to`: array (0 the
// image: one pixel) and the pixel it starts at; returns the last pixel it reaches.
struct Step {
  int arr, j;
};
// (occ: the words' starts, `width` words each).
int best_step(const Word *words, int nw, const uint64_t *occ, int width, int c, int to, Step &s) {
  int end = c;
  s = Step{0, c};
  for (int w = 0; w < nw; ++w) {
    const int L = words[w].L, at = std::min(c, to - L);
    if (at < 0) continue;
    const int j = last_start(occ + (size_t)w * width, at, end - L + 1);
    if (j >= 0 && j + L > end) {
      end = j + L;
      s = Step{w + 1, j};
    }
  }
  return end;
}

struct GroupOut {
  CoverGroup g{};
  int nw = 0;  // words, at most
  size_t lds_dw = 0;
  std::vector<int32_t> piece_off;  // within recs
  std::vector<int4> recs;
  std::vector<uint32_t> bops;
  std::vector<MemDesc> mems;
  int64_t cost = 0, steps = 0, counts = 0, bsteps = 0;
};

// LDS rows of a group: the window of the image that its paths reach from a tile's start pixels.
// Row y (0 = the tile's first row) is staged from dword xs(y) on; rows are rst dwords apart, so
// the address of (row, dword) is linear and the window of a steep group, which shifts to the
// right row by row, is held without the rest of its bounding box.
struct Geometry {
  const Octant *o;
  int SR, maxpy;
  std::vector<int> lo, hi;  // first and last pixel offset in x at each row offset
  Geometry(const Octant &oct, const Path &first, const Path &last, int len, int sr) : o(&oct), SR(sr) {
    maxpy = oct.xm ? last.q(len) : len;
    lo.assign(maxpy + 1, INT_MAX);
    hi.assign(maxpy + 1, 0);
    for (int k = 0; k <= len; ++k) {
      const int a = first.q(k), b = last.q(k);
      if (oct.xm) {
        for (int y = a; y <= b; ++y) {
          lo[y] = std::min(lo[y], k);
          hi[y] = std::max(hi[y], k);
        }
      } else {
        lo[k] = a;
        hi[k] = b;
      }
    }
    // monotone bounds (rows that only some paths reach)
    for (int y = maxpy - 1; y >= 0; --y) lo[y] = std::min(lo[y], lo[y + 1]);
    for (int y = 1; y <= maxpy; ++y) hi[y] = std::max(hi[y], hi[y - 1]);
    slope = 0;
    if (maxpy > 0) {
      const double s = oct.xm ? (double)last.n / std::max(last.m, 1) : (double)first.m / first.n;
      if (s <= 16.0) slope = (int)std::floor(s / 32.0 * 65536.0);
    }
  }
  int slope;
  void set(int tile, int S, int R, CoverGroup &g) const {
    g.tile = tile;
    g.rows = std::max(2, tile + maxpy);  // one row, H = 1: rows_magic would not fit 32 bits
    g.sh_a = slope;
    int64_t b = 0;
    for (int d = 0; d <= maxpy; ++d)
      b = std::max<int64_t>(b, (int64_t)slope * d - (int64_t)(lo[d] >> 5) * 65536);
    g.sh_b = (int)b;
    auto xs = [&](int y) {
      const int d = std::max(0, y - tile + 1);
      return std::max(0, (int)(((int64_t)d * g.sh_a - g.sh_b) >> 16));
    };
    // (rows before the tile's last one start at dword 0, and hi does not fall)
    int wid = 0;
    for (int y = tile - 1; y < g.rows; ++y)
      wid = std::max(wid, SR + (hi[std::min(y, maxpy)] >> 5) - xs(y) + 1);
    g.wid = wid;
    g.wid_magic = (uint32_t)((((uint64_t)1 << 32) + wid - 1) / wid);
    g.rows_magic = (uint32_t)((((uint64_t)1 << 32) + g.rows - 1) / g.rows);
    // lanes of a wave on distinct banks: an odd row stride for one lane per row, else the stride
    // with the fewest lanes per bank
    int best = wid, worst = INT_MAX;
    for (int r = wid; r < wid + 16 && worst > 1; ++r) {
      int cnt[64] = {}, w = 0;
      const int rpw = 64 / S;
      for (int l = 0; l < 64; ++l) w = std::max(w, ++cnt[((l % rpw) * r + (l / rpw) * R) & 63]);
      if (w < worst) {
        worst = w;
        best = r;
      }
    }
    g.rst = best;
    g.asz = (g.rows - 1) * g.rst + xs(g.rows - 1) + wid;
  }
};

// Prefix tree of a piece's paths: the leaves are paths, an inner node the pixels 0..m that the
// paths a..b-1 share.
struct Node {
  int a, b, m;
  int kid = -1, next = -1;  // first child; next child of the same parent
  int memo = -1;            // its entries in memo_
};

class GroupBuilder {
 public:
  GroupBuilder(int H, const CoverShape &sh) : H_(H), sh_(sh) {}

  // The group of paths a .. b - 1 of an octant: tile and LDS layout; false when its rows do not fit.
  bool fit(const Octant &o, int a, int b, GroupOut &out) {
    set(o, a, b);
    int len = 0, nmem = 0;
    for (int i = a_; i < b_; ++i) {
      len = std::max(len, o_->paths[i].len);
      nmem += o_->paths[i].nm;
    }
    const int rpw = 64 / sh_.S;
    const int bands = (H_ + rpw - 1) / rpw;
    Geometry geo(*o_, o_->paths[a_], o_->paths[b_ - 1], len, sh_.S * sh_.R);
    CoverGroup &g = out.g;
    g.nmem = nmem;
    const int avail = sh_.lds / 4 - nmem - kCoverPad;
    // Words, waves per chain and tile by estimated work: steps per member by the number of words
    // (measured means over the groups of cutoffs 128 to 512; longer paths take more), a count per
    // member, and the masks' steps over the staged rows.
    const double len_f = std::min(2.0, std::max(0.5, len / 256.0));
    static const double kSteps[] = {20, 8, 4.6, 3.4, 3.0};
    double best = 1e300;
    CoverGroup pick = g;
    for (int nwb = sh_.nwb; nwb >= 1; nwb /= 2) {
      if (nwb > bands) continue;
      // sixteen pieces share too little (1 024 x 1 024, cutoff 512: 6.9 against 5.6 ms)
      if (nwb == 1 && sh_.wpg > 8 && best < 1e300) continue;
      for (int w = kCoverWords; w >= 1; --w) {
        int prev = -1;
        for (int nt = 1; nt <= bands; ++nt) {
          int per = (bands + nt - 1) / nt;
          per = (per + nwb - 1) / nwb * nwb;
          if (per == prev) continue;
          prev = per;
          // (rows alone beyond the budget: no need for the exact window)
          if ((int64_t)per * rpw <= 16384 &&
              (int64_t)(1 + w) * (per * rpw + geo.maxpy) * sh_.S * sh_.R <= avail) {
            CoverGroup t = g;
            geo.set(per * rpw, sh_.S, sh_.R, t);
            if ((int64_t)(1 + w) * t.asz <= std::min(avail, 65535)) {
              const double SR = sh_.S * sh_.R;
              const double walk = nmem * (kSteps[w] * len_f * (1.5 * sh_.R + 6) + sh_.R + 12) *
                                  (1.0 + 0.04 * (sh_.wpg / nwb - 1));
              const double build = (6 + 5 * w) * 2.5 * sh_.R * t.rows * t.wid / (t.tile * SR);
              if (walk + build < best) {
                best = walk + build;
                pick = t;
                pick.nwb = nwb;
                out.nw = w;
              }
              break;
            }
          }
          if (per == nwb) break;
        }
      }
    }
    g = pick;
    return best < 1e300;
  }

  // Its words and records, in the layout that fit() chose.
  void build(const Octant &o, int a, int b, GroupOut &out) {
    set(o, a, b);
    words_.clear();
    slot0_.clear();
    CoverGroup &g = out.g;
    const int nmem = g.nmem;
    g.ntiles = (H_ + g.tile - 1) / g.tile;
    int len = 0;
    for (int i = a_; i < b_; ++i) len = std::max(len, o_->paths[i].len);
    width_ = occ_words(len);
    bits_.resize((size_t)(b_ - a_) * bit_words(len));
    for (int i = a_; i < b_; ++i) letters(o_->paths[i], o_->paths[i].len, let(i - a_));
    out.mems.reserve(nmem);
    choose_words(out.nw, out);
    g.nw = (int)words_.size();
    out.lds_dw = (size_t)(1 + g.nw) * g.asz + kCoverPad + nmem;
    // members: slots in path order
    for (int i = a_; i < b_; ++i) {
      const Path &p = o_->paths[i];
      slot0_.push_back((int)out.mems.size());
      out.mems.insert(out.mems.end(), o_->mems.begin() + p.m0, o_->mems.begin() + p.m0 + p.nm);
    }
    pieces(out);
    out.counts = nmem;
  }

 private:
  const int H_;
  const CoverShape sh_;
  // the group, and what is kept of one for the next is the memory only
  const Octant *o_ = nullptr;
  int a_ = 0, b_ = 0;
  void set(const Octant &o, int a, int b) {
    o_ = &o;
    a_ = a;
    b_ = b;
  }
  int width_ = 0;               // words of the longest path's pixels
  std::vector<uint64_t> bits_;  // the paths' letters
  uint64_t *let(int i) { return bits_.data() + (size_t)i * (width_ + 1); }
  std::vector<int> slot0_;
  std::vector<Word> words_;
  std::vector<uint64_t> cand_bits_;  // letters of the words tried

  uint32_t encode(const CoverGroup &g, int arr, int x, int y) const {
    return (uint32_t)(arr * g.asz + y * g.rst + (x >> 5)) | ((uint32_t)(x & 31) << 16);
  }

  // The words: greedily, from the beginnings and ends of the middle path, the one that saves most
  // steps (sampled paths, their last two thirds: what comes before is mostly shared), as long as
  // it saves more than building its mask costs.
  void choose_words(int nw, GroupOut &out) {
    CoverGroup &g = out.g;
    const int np = b_ - a_;
    std::vector<int> smp;
    const bool quick = np < 40;  // small groups: their plans are most of a first call
    const int ns = std::min(np, quick ? 3 : 5);
    for (int s = 0; s < ns; ++s) smp.push_back((int)((2ll * s + 1) * np / (2 * ns)));
    int mid = np / 2;
    for (int i = 0; i < np; ++i)  // the longest path near the middle
      if (std::abs(i - np / 2) <= np / 4 && o_->paths[a_ + i].len > o_->paths[a_ + mid].len) mid = i;
    const int ml = o_->paths[a_ + mid].len;
    auto longer = [&](int L) { return L + std::max(1, quick ? L / 2 : L / 3); };
    int most_cand = 0;
    for (int L = 1; L <= ml; L = longer(L)) most_cand += 2;
    const int wb = bit_words(ml);
    cand_bits_.resize((size_t)most_cand * wb);
    std::vector<Word> cand;
    cand.reserve(most_cand);
    for (int L = 1; L <= ml; L = longer(L)) {
      for (int j : {0, ml - L}) {
        const Word w = sub_word(let(mid), j, L, &cand_bits_[cand.size() * wb]);
        // (the two words of a length follow each other)
        const bool seen = !cand.empty() && cand.back().L == L &&
                          std::equal(w.b, w.b + bit_words(L), cand.back().b);
        if (!seen) cand.push_back(w);
      }
    }
    const int nc = (int)cand.size();
    // starts of every candidate on every sample
    std::vector<std::vector<uint64_t>> occ(ns);
    std::vector<int> width(ns);
    for (int s = 0; s < ns; ++s) {
      const int len = o_->paths[a_ + smp[s]].len;
      width[s] = occ_words(len);
      occ[s].resize((size_t)nc * width[s]);
      for (int c = 0; c < nc; ++c)
        find_word(let(smp[s]), len, cand[c], &occ[s][(size_t)c * width[s]]);
    }
    const double scale = (double)np / ns;
    const double ratio = 1.5 * (double)g.rows * g.wid / ((double)g.tile * sh_.S * sh_.R);
    std::vector<int> sel;
    // cost of the words sel[0..k), given up once it passes `most`
    auto steps = [&](const int *ws, int k, double most) {
      double bc = 0;
      for (int x = 0; x < k; ++x) {
        int sub = 0;
        const int L = cand[ws[x]].L;
        for (int y = 0; y < k; ++y)
          if (cand[ws[y]].L < L) sub = std::max(sub, cand[ws[y]].L);
        bc += sub ? (double)L / (sub + 1) + 2 : L + 1;
      }
      bc *= ratio;
      if (bc >= most) return most;
      const int64_t limit = most < 1e200 ? (int64_t)((most - bc) / scale) + 1 : INT64_MAX;
      int64_t n = 0;
      for (int s = 0; s < ns; ++s) {
        const Path &p = o_->paths[a_ + smp[s]];
        const uint64_t *oc = occ[s].data();
        int c = p.len / 3;
        for (int t = 0; t < p.nm; ++t) {
          const int l = o_->mems[p.m0 + t].l;
          while (c <= l) {
            int end = c;
            for (int x = 0; x < k; ++x) {
              const int L = cand[ws[x]].L, at = std::min(c, l - L);
              if (at < 0) continue;
              const int j = last_start(oc + (size_t)ws[x] * width[s], at, end - L + 1);
              if (j >= 0) end = std::max(end, j + L);
            }
            c = end + 1;
            if (++n > limit) return most;
          }
        }
      }
      return n * scale + bc;
    };
    int ws[kCoverWords] = {};
    double cur = steps(ws, 0, 1e300);
    auto better = [&](int at, int k) {  // the best candidate for word `at` of k; -1 when none helps
      int best = -1;
      for (int c = 0; c < nc; ++c) {
        ws[at] = c;
        const double v = steps(ws, k, cur - 0.5);
        if (v < cur - 0.5) {
          cur = v;
          best = c;
        }
      }
      return best;
    };
    int k = 0;
    while (k < nw) {
      const int best = better(k, k + 1);
      if (best < 0) break;
      ws[k++] = best;
    }
    // the first word was chosen alone: once more, given the others
    if (k > 1 && !quick) {
      const int old = ws[0], best = better(0, k);
      ws[0] = best < 0 ? old : best;
    }
    sel.assign(ws, ws + k);
    std::sort(sel.begin(), sel.end(), [&](int x, int y) { return cand[x].L < cand[y].L; });
    sel.erase(std::unique(sel.begin(), sel.end()), sel.end());
    for (int w : sel) words_.push_back(cand[w]);
    // each mask from the image and the shorter masks
    g.bop[0] = 0;
    for (size_t w = 0; w < words_.size(); ++w) {
      const Word &wd = words_[w];
      const int wd_words = occ_words(wd.L);
      std::vector<uint64_t> oc(w * wd_words);
      for (size_t v = 0; v < w; ++v) find_word(wd.b, wd.L, words_[v], &oc[v * wd_words]);
      int c = 0;
      while (c <= wd.L) {
        Step s;
        c = best_step(words_.data(), (int)w, oc.data(), wd_words, c, wd.L, s) + 1;
        int q = 0;
        for (int k = 0; k < s.j; ++k) q += (int)((wd.b[k >> 6] >> (k & 63)) & 1);
        out.bops.push_back(o_->xm ? encode(g, s.arr, s.j, q) : encode(g, s.arr, q, s.j));
      }
      g.bop[w + 1] = (int)out.bops.size();
    }
    for (int w = (int)words_.size(); w < kCoverWords; ++w) g.bop[w + 1] = (int)out.bops.size();
    out.bsteps = (int64_t)out.bops.size();
  }

  // ---- the walks of one piece ----
  struct Memo {
    int s, k, cost;
    bool save;
    int next;
  };
  std::vector<Node> nodes_;
  std::vector<Memo> memo_;
  std::vector<int> lcp_;
  std::vector<uint64_t> occ_;  // the words' starts on each path, width_ words each
  const uint64_t *occ(int i) const { return occ_.data() + (size_t)i * words_.size() * width_; }

  int tree(int a, int b) {
    Node t{a, b, 0};
    if (b - a == 1) {
      t.m = o_->paths[a].len;
    } else {
      int m = INT_MAX;
      for (int i = a; i + 1 < b; ++i) m = std::min(m, lcp_[i - a_]);
      t.m = m;
      int s = a, last = -1;
      for (int i = a; i < b; ++i)
        if (i + 1 == b || lcp_[i - a_] == m) {
          const int u = tree(s, i + 1);
          (last < 0 ? t.kid : nodes_[last].next) = u;
          last = u;
          s = i + 1;
        }
    }
    nodes_.push_back(t);
    return (int)nodes_.size() - 1;
  }

  // Least cost, in pixels, of the walks below node v from a product saved at depth s with k saves
  // left, and whether to save at v's depth.  A save or a restore copies the product: about 6.
  std::pair<int, bool> best_save(int v, int s, int k) {
    for (int e = nodes_[v].memo; e >= 0; e = memo_[e].next)
      if (memo_[e].s == s && memo_[e].k == k) return std::make_pair(memo_[e].cost, memo_[e].save);
    std::pair<int, bool> r(0, false);
    const Node t = nodes_[v];
    if (t.kid < 0) {
      r.first = t.m - s + 6;
    } else {
      for (int u = t.kid; u >= 0; u = nodes_[u].next) r.first += best_save(u, s, k).first;
      if (k > 0 && t.m - s >= 6) {
        int c = t.m - s + 12;
        for (int u = t.kid; u >= 0; u = nodes_[u].next) c += best_save(u, t.m, k - 1).first;
        if (c < r.first) r = std::make_pair(c, true);
      }
    }
    memo_.push_back(Memo{s, k, r.first, r.second, nodes_[v].memo});
    nodes_[v].memo = (int)memo_.size() - 1;
    return r;
  }

  // The pieces: about equal work for each wave.  The work of a path shows only once its records
  // are there (what it shares with its neighbours is walked once), so the group is cut by members
  // first and cut again by the work that each path's records took (slowest against mean piece at
  // cutoff 512: 1.5 and 1.13; an estimate from the unshared lengths gave 1.5 as well).
  void pieces(GroupOut &out) {
    const int np = b_ - a_;
    lcp_.assign(np, 0);
    for (int i = 0; i + 1 < np; ++i)
      lcp_[i] = common(let(i), let(i + 1),
                       std::min(o_->paths[a_ + i].len, o_->paths[a_ + i + 1].len));
    occ_.resize((size_t)np * words_.size() * width_);
    for (int i = 0; i < np; ++i)
      for (size_t w = 0; w < words_.size(); ++w)
        find_word(let(i), o_->paths[a_ + i].len, words_[w], &occ_[(i * words_.size() + w) * width_]);
    out.recs.reserve((size_t)4 * out.g.nmem);
    const int nsub = sh_.wpg / out.g.nwb;
    work_.resize(np);
    for (int i = 0; i < np; ++i) work_[i] = 4 + 3 * o_->paths[a_ + i].nm;
    for (int pass = 0; pass < (nsub > 1 ? 2 : 1); ++pass) {
      const std::vector<int> w = work_;
      int64_t total = 0;
      for (int x : w) total += x;
      std::fill(work_.begin(), work_.end(), 0);
      out.recs.clear();
      out.piece_off.clear();
      out.steps = 0;
      int i = 0;
      int64_t acc = 0;
      for (int p = 0; p < nsub; ++p) {
        out.piece_off.push_back((int32_t)out.recs.size());
        const int s = i;
        while (i < np && (p + 1 == nsub || (acc + w[i] / 2) * nsub < total * (p + 1))) acc += w[i++];
        if (i == s) continue;
        nodes_.clear();
        const int root = tree(a_ + s, a_ + i);
        memo_.clear();
        in_acc_ = -1;
        emit(out, root, -1, 0, 0, 2);
      }
      out.piece_off.push_back((int32_t)out.recs.size());
    }
    out.cost = 0;
    for (int x : work_) out.cost += x;
  }
  std::vector<int> work_;  // vector instructions of each path's records

  int in_acc_ = -1;  // level of the saved product that the accumulators hold, -1 none

  // Records for `steps` on path i; the last one carries the count.
  void put(GroupOut &out, int i, const std::vector<Step> &steps, int level, int slot) {
    const Path &p = o_->paths[i];
    auto code = [&](const Step &s) {
      const int q = p.q(s.j);
      return o_->xm ? encode(out.g, s.arr, s.j, q) : encode(out.g, s.arr, q, s.j);
    };
    for (size_t t = 0; t < steps.size(); t += 2) {
      int4 r = make_int4((int)code(steps[t]), 0, 0, 0);
      if (t + 1 < steps.size()) {
        r.y = (int)code(steps[t + 1]);
        r.x |= (int)kRecTwo;
      }
      if (!(in_acc_ == level && level > 0)) {
        if (!started_) r.x |= (level + 1) << kRecRestore;
      }
      started_ = true;
      in_acc_ = -1;
      if (slot >= 0 && t + 2 >= steps.size()) {
        r.x |= (int)kRecCount;
        r.z = slot;
      }
      out.recs.push_back(r);
    }
    out.steps += (int64_t)steps.size();
    work_[i - a_] += (int)(steps.size() * (3 * sh_.R / 2 + 6)) + (slot >= 0 ? sh_.R + 12 : 0);
  }
  bool started_ = false;
  // of one call of emit, before it goes on to the nodes below
  std::vector<std::pair<int, int>> ends_;
  std::vector<Step> st_;

  // Walks below node v; products covered below pixel c are saved at `level` (depth s).
  void emit(GroupOut &out, int v, int s, int c, int level, int k) {
    const Node t = nodes_[v];
    const bool leaf = t.kid < 0;
    if (!leaf && !(level < 2 && best_save(v, std::max(s, 0), k).second)) {
      for (int u = t.kid; u >= 0; u = nodes_[u].next) emit(out, u, s, c, level, k);
      return;
    }
    // counts on the shared pixels s < l <= m of the paths below: (l, slot)
    ends_.clear();
    for (int i = t.a; i < t.b; ++i)
      for (int x = 0; x < o_->paths[i].nm; ++x) {
        const int l = o_->mems[o_->paths[i].m0 + x].l;
        if (l > s && l <= t.m) ends_.push_back({l, slot0_[i - a_] + x});
      }
    std::sort(ends_.begin(), ends_.end());
    const uint64_t *oc = occ(t.a - a_);
    const int nw = (int)words_.size();
    int cv = c;
    const size_t rec0 = out.recs.size();
    started_ = false;
    for (const auto &e : ends_) {
      st_.clear();
      while (cv <= e.first) {
        Step x;
        cv = best_step(words_.data(), nw, oc, width_, cv, e.first, x) + 1;
        st_.push_back(x);
      }
      put(out, t.a, st_, level, e.second);
    }
    size_t rec1 = out.recs.size();  // the records up to here: counts of this node
    if (!leaf) {
      // on towards the branch, while steps are worth it
      st_.clear();
      for (;;) {
        if (cv > t.m) break;
        Step x;
        const int end = best_step(words_.data(), nw, oc, width_, cv, t.m, x);
        if (end - cv < 3) break;
        cv = end + 1;
        st_.push_back(x);
      }
      if (!st_.empty()) put(out, t.a, st_, level, -1);
      if (out.recs.size() > rec0) {
        out.recs.back().x |= (level + 1) << kRecSave;
        in_acc_ = level + 1;
        for (int u = t.kid; u >= 0; u = nodes_[u].next) emit(out, u, t.m, cv, level + 1, k - 1);
      } else {
        for (int u = t.kid; u >= 0; u = nodes_[u].next) emit(out, u, s, c, level, k);
      }
    }
    for (size_t r = rec0; r < rec1; ++r)
      if (out.recs[r].x & (int)kRecCount) out.recs[r].w = (int)out.recs.size();
  }
};

}  // namespace

void cover_lanes(int W, int H, int *R, int *S) {
  // words times lanes that a band walks, plus the work per record that does not depend on R
  // (about four words' worth)
  const int swd = (W + 31) / 32;
  int64_t best = INT64_MAX;
  for (int s = 1; s <= 64; s *= 2)
    for (int r = 16; r >= 1; --r) {
      const int nct = (swd + r * s - 1) / (r * s);
      if (s > 1 && (s / 2) * r >= swd) continue;
      const int bands = (H + 64 / s - 1) / (64 / s);
      const int64_t cost = (int64_t)nct * bands * (r + 4);
      if (cost < best) {
        best = cost;
        *R = r;
        *S = s;
      }
    }
}

namespace {

// The plan for given octants and shape; false when some group's rows do not fit sh.lds.
bool build_cover(const std::vector<Octant> &oct, int W, int H, int cx, int cy, const CoverShape &sh,
                 int groups_want, CoverHost &out, std::vector<int64_t> &tile_cost) {
  out = CoverHost();
  out.sh = sh;
  const int swd = (W + 31) / 32;
  out.nct = (swd + sh.R * sh.S - 1) / (sh.R * sh.S);
  // groups of about equal cost
  auto cost = [](const Path &p) { return 4 + 3 * (int64_t)p.nm; };
  int64_t total = 0;
  for (auto &o : oct)
    for (int p = 0; p < (int)o.paths.size(); ++p) total += (p < o.axis ? 1 : 2) * cost(o.paths[p]);
  // Groups of dx >= 0 and, right after them, the same of dx < 0: a group without an axis path has its
  // mirrored image's words and records (src); only the first ones are planned apart.
  struct Range {
    int o, a, b;
    bool mirror;
    int src;
  };
  std::vector<Range> ranges;
  for (int i = 0; i < 2; ++i) {
    const Octant &o = oct[i];
    if (o.paths.empty()) continue;
    int64_t oc = 0, om = 0, ac = 0, am = 0;  // cost and members; the axis's
    for (int p = 0; p < (int)o.paths.size(); ++p) {
      oc += cost(o.paths[p]);
      om += o.paths[p].nm;
      if (p < o.axis) {
        ac += cost(o.paths[p]);
        am += o.paths[p].nm;
      }
    }
    // Both signs of dx together get their share of the groups: `want` with the axis and as many without
    // the groups that are axis only.  (One group more than groups_want can mean one more round of
    // workgroups: 512 x 512, cutoff 128: 128 groups 147 us, 130 158.)
    const double share = (double)groups_want * (2 * oc - ac) / total;
    const int64_t alone = (int64_t)(ac * share / (2 * oc - ac));
    int want = std::max(1, (int)std::llround((share + alone) / 2));
    // Groups full of members would leave remnants between them.  Where that sets their number, an axis
    // that fills a third of one has a group of its own (1024 x 1024, cutoff 512: 8.05 ms, with others in
    // its group 8.2); a shorter one does not (512 x 512, cutoff 255: 2 412 mask steps, apart 2 626).
    const int np = (int)o.paths.size(), first = (int)ranges.size();
    auto full = [](int64_t m) { return (int)((m * 5 / 4 + kCoverSlots - 1) / kCoverSlots); };
    const bool apart = full(om - am / 2) > want && am * 3 > kCoverSlots && o.axis < np;
    const int start = apart ? o.axis : 0;
    want = std::max(want, full(apart ? om - am : om - am / 2));
    if (apart) oc -= ac;
    int a = start;
    int64_t acc = 0;
    int mem = 0, k = 1;
    for (int p = a; p < np; ++p) {
      const Path &pt = o.paths[p];
      if (p > a && (mem + pt.nm > kCoverSlots || (acc + cost(pt) / 2) * want >= oc * k)) {
        ranges.push_back({i, a, p, false, -1});
        a = p;
        mem = 0;
        while ((acc + cost(pt) / 2) * want >= oc * k) ++k;
      }
      acc += cost(pt);
      mem += pt.nm;
    }
    ranges.push_back({i, a, np, false, -1});
    for (int r = first, e = (int)ranges.size(); r < e; ++r) {
      const Range g = ranges[r];
      if (g.b > o.axis)
        ranges.push_back({i, std::max(g.a, o.axis), g.b, true, g.a >= o.axis ? r : -1});
    }
    if (start) ranges.push_back({i, 0, start, false, -1});
  }
  const int ng = (int)ranges.size();
  std::vector<GroupOut> go(ng);
  std::atomic<bool> fits(true);
  // A thread for about 300 vectors (their plan takes some 200 us, starting a thread 30), a few runs
  // of groups each; fit() tries tiles of as many heights as there are bands.
  int64_t members = 0;
  for (const Octant &o : oct) members += (int64_t)o.mems.size();
  const int threads = (int)std::min<int64_t>(16, std::min<int64_t>(ng / 4, 1 + members / 300));
  const int bands = (H + 64 / sh.S - 1) / (64 / sh.S);
  const int runs = std::min(ng, 8 * std::max(1, threads));
  auto groups = [&](int thr, auto &&f) {
    parallel(runs, thr, [&](int run) {
      GroupBuilder gb(H, sh);
      for (int i = (int)((int64_t)ng * run / runs); i < (int)((int64_t)ng * (run + 1) / runs); ++i)
        if (ranges[i].src < 0) f(gb, oct[ranges[i].o], ranges[i].a, ranges[i].b, go[i]);
    });
  };
  groups((int64_t)ng * bands > 256 ? threads : 1,
         [&](GroupBuilder &gb, const Octant &o, int a, int b, GroupOut &x) {
           if (fits && !gb.fit(o, a, b, x)) fits = false;
         });
  if (!fits) return false;
  groups(threads, [&](GroupBuilder &gb, const Octant &o, int a, int b, GroupOut &x) {
    gb.build(o, a, b, x);
  });
  size_t nrec = 64, dw = 0;
  for (auto &x : go) nrec += x.recs.size();
  out.recs.reserve(nrec);
  out.mems.reserve((size_t)(cx + 1) * (cy + 1) + (size_t)cx * cy);
  tile_cost.clear();
  for (int i = 0; i < ng; ++i) {
    const Range &rg = ranges[i];
    const GroupOut &x = go[rg.src < 0 ? i : rg.src];
    CoverGroup g = rg.src < 0 ? x.g : out.groups[rg.src];  // (records and words: the source's)
    if (rg.src < 0) {
      g.piece0 = (int32_t)out.piece_off.size();
      const int r0 = (int)out.recs.size(), b0 = (int)out.bops.size();
      for (int &b : g.bop) b += b0;
      for (int32_t p : x.piece_off) out.piece_off.push_back(p + r0);
      out.recs.insert(out.recs.end(), x.recs.begin(), x.recs.end());
      for (size_t r = r0; r < out.recs.size(); ++r) out.recs[r].w += r0;
      out.bops.insert(out.bops.end(), x.bops.begin(), x.bops.end());
    }
    g.mirror = rg.mirror ? 1 : 0;
    g.mem0 = (int32_t)out.mems.size();
    out.mems.insert(out.mems.end(), x.mems.begin(), x.mems.end());
    if (rg.mirror)
      for (size_t m = g.mem0; m < out.mems.size(); ++m) {
        MemDesc &v = out.mems[m];
        v.dx = (int16_t)-v.dx;
        v.idx = (int32_t)index_of(cx, cy, v.dx, v.dy);
      }
    // vector instructions of a tile: its masks (8 dwords a lane, about 40 instructions a step with
    // the waits between them), its rows, the walks of its bands
    const int bands = g.tile / (64 / sh.S);
    tile_cost.push_back(x.cost * bands + (x.bsteps * 5 + 60) * g.rows * g.wid / 64);
    out.steps += x.steps;
    out.counts += x.counts;
    out.bsteps += x.bsteps;
    dw = std::max(dw, x.lds_dw);
    out.groups.push_back(g);
  }
  out.recs.resize(out.recs.size() + 48, make_int4(0, 0, 0, 0));  // read ahead of the last record
  out.lds_bytes = dw * 4;
  return true;
}

}  // namespace

bool plan_cover(int W, int H, int cx, int cy, int fR, int fS, int fW, int fL, int cus,
                CoverHost &out) {
  int R = 0, S = 0;
  cover_lanes(W, H, &R, &S);
  if (fR) R = fR;
  if (fS || fR) {
    const int swd = (W + 31) / 32;
    S = 1;
    while (S < 64 && S * R < swd) S *= 2;
    if (fS) S = fS;
  }
  const int64_t nv = (int64_t)(cx + 1) * (cy + 1) + (int64_t)cx * cy;
  std::vector<Octant> oct(2);
  parallel(2, nv > 3000 ? 2 : 1, [&](int i) { build_octant(cx, cy, i == 0, oct[i]); });
  for (;; R = R / 2) {
    for (int big = 0; big < 2; ++big) {
      if (fL && big) break;
      CoverShape sh;
      sh.R = R;
      sh.S = S;
      sh.lds = fL ? fL : (big ? 160 : 80) * 1024;
      sh.wpg = fW ? fW : (sh.lds > 80 * 1024 ? 16 : 8);
      sh.nwb = sh.wpg % 2 ? 1 : 2;
      // Groups: one item (group, phase, tile) per resident workgroup and phase, at least 64 groups
      // (512 x 512, cutoff 128, one tile per item: 64 groups 0.20 ms, 128 0.144, 160 0.141, 256
      // 0.167: fewer groups have wider slopes and poorer words, more build more masks), fewer
      // when a piece would get less than about three paths (128 x 128, cutoff 32: 12.3 against
      // 13.5 us with six).
      const int nsub = sh.wpg / sh.nwb;
      const int64_t paths = nv / 3 + 1;
      const int64_t slots = (int64_t)cus * (sh.lds > 80 * 1024 ? 1 : 2);
      const int nct = ((W + 31) / 32 + R * S - 1) / (R * S);
      const int rpw = 64 / S;
      const int bands = (H + rpw - 1) / rpw;
      int per = bands;  // bands of a tile, at a guess: the widest rows of a group, three masks
      while (per > 2 && (int64_t)(per * rpw + cy) * (R * S + 4) * 16 > sh.lds) --per;
      const int64_t tiles = (int64_t)((bands + per - 1) / per) * nct;
      int64_t g = std::max<int64_t>(slots / tiles, 64);
      g = std::max<int64_t>(4, std::min<int64_t>(g, paths / (3 * nsub)));
      std::vector<int64_t> tile_cost;
      if (!build_cover(oct, W, H, cx, cy, sh, (int)g, out, tile_cost)) continue;
      int64_t most = 1;
      for (const CoverGroup &x : out.groups) most = std::max<int64_t>(most, x.ntiles * out.nct);
      // up to eight items per CU and phase, so that the last ones are short (1 024 x 1 024, cutoff
      // 512: 5.6 ms against 6.1 with two)
      const int64_t items = 8 * (int64_t)cus;
      const int64_t want = std::min(most, std::max<int64_t>(1, items / (int64_t)out.groups.size()));
      const int64_t each = (most + want - 1) / want;
      out.nsplit = (int)((most + each - 1) / each);
      std::vector<std::pair<int64_t, int2>> list;
      for (int x = 0; x < (int)out.groups.size(); ++x) {
        const int tiles_x = out.groups[x].ntiles * out.nct;
        for (int t = 0; t < std::min(out.nsplit, tiles_x); ++t)
          list.push_back({tile_cost[x] * ((tiles_x - t + out.nsplit - 1) / out.nsplit), make_int2(x, t)});
      }
      std::stable_sort(list.begin(), list.end(),
                       [](const auto &a, const auto &b) { return a.first > b.first; });
      for (auto &x : list) {
        out.items.push_back(x.second);
        out.cost.push_back(x.first);
      }
      return true;
    }
    if (fR || R == 1) return false;
  }
}

namespace {

// The masks of a group as the kernel builds them, C dwords per item; false when an access leaves
// its array.
template <int C>
bool run_masks(const CoverHost &p, const CoverGroup &g, int64_t top, std::vector<uint32_t> &lds) {
  const int items = cover_mask_items<C>(g.wid, g.rows);
  for (int a = 1; a <= g.nw; ++a)
    for (int i = 0; i < items; ++i) {
      const int at = cover_mask_item<C>(g, i);
      if (at < 0 || at + C > g.asz) return false;
      uint32_t v[C];
      std::fill(v, v + C, ~0u);
      for (int b = g.bop[a - 1]; b < g.bop[a]; ++b) {
        const int64_t q = at + (int64_t)(p.bops[b] & 0xffff);
        if (q + C >= top) return false;
        for (int c = 0; c < C; ++c) v[c] &= funnel(lds[q + c + 1], lds[q + c], (p.bops[b] >> 16) & 31);
      }
      for (int c = 0; c < C; ++c) lds[(size_t)a * g.asz + at + c] = v[c];
    }
  return true;
}
bool run_masks(int C, const CoverHost &p, const CoverGroup &g, int64_t top,
               std::vector<uint32_t> &lds) {
  switch (C) {
    case 2: return run_masks<2>(p, g, top, lds);
    case 3: return run_masks<3>(p, g, top, lds);
    case 4: return run_masks<4>(p, g, top, lds);
    case 5: return run_masks<5>(p, g, top, lds);
    case 6: return run_masks<6>(p, g, top, lds);
    case 7: return run_masks<7>(p, g, top, lds);
    default: return run_masks<8>(p, g, top, lds);
  }
}

}  // namespace

bool run_cover(const CoverHost &p, const uint8_t *img, int W, int H, int phase, int64_t *counts) {
  const int S = p.sh.S, R = p.sh.R, rpw = 64 / S, SR = S * R, wpr = 2 * ((W + 63) / 64);
  const std::vector<uint32_t> rows = packed_rows(img, W, H, wpr);
  std::vector<uint32_t> lds(p.lds_bytes / 4 + 64);
  for (const CoverGroup &g : p.groups) {
    const int64_t top = (int64_t)(1 + g.nw) * g.asz + kCoverPad;
    if (top + g.nmem > (int64_t)p.lds_bytes / 4) return false;
    std::vector<int64_t> slot(g.nmem, 0);
    for (int ct = 0; ct < p.nct; ++ct)
      for (int rt = 0; rt < g.ntiles; ++rt) {
        uint32_t junk = 12345u + ct * 7 + rt;
        for (auto &d : lds) d = junk = junk * 1664525u + 1013904223u;
        for (int i = 0; i < g.rows * g.wid; ++i) {
          int y, e;
          cover_cell(g, i, y, e);
          const int64_t at = (int64_t)y * g.rst + e;
          if (y < 0 || y >= g.rows || at < 0 || at >= g.asz) return false;
          const uint32_t *row = rows.data() + (size_t)((rt * g.tile + y) % H) * wpr;
          const uint32_t v = periodic32(row, W, word_start(W, ct * SR + e, g.mirror != 0));
          lds[at] = (phase ? 0u : ~0u) ^ (g.mirror ? bit_reverse(v) : v);
        }
        if (!run_masks(cover_mask_words(R), p, g, top, lds)) return false;
        const int rows_here = std::min(g.tile, H - rt * g.tile);
        const int nsub = p.sh.wpg / g.nwb;
        for (int pc = 0; pc < nsub; ++pc)
          for (int row = 0; row < g.tile; ++row)
            for (int strip = 0; strip < S; ++strip) {
              std::vector<uint32_t> init(R), A(R), sv[2] = {std::vector<uint32_t>(R), std::vector<uint32_t>(R)};
              for (int i = 0; i < R; ++i) {
                const int64_t w0 = ct * SR + strip * R + i;
                for (int b = 0; b < 32; ++b)
                  if (row < rows_here && 32 * w0 + b < W) init[i] |= 1u << b;
              }
              for (int r = p.piece_off[g.piece0 + pc]; r < p.piece_off[g.piece0 + pc + 1]; ++r) {
                const int4 q = p.recs[r];
                const int rs = (q.x >> kRecRestore) & 3, sa = (q.x >> kRecSave) & 3;
                if (rs) A = rs == 1 ? init : sv[rs - 2];
                for (int t = 0; t < (q.x & (int)kRecTwo ? 2 : 1); ++t) {
                  const int c = t ? q.y : q.x;
                  const int64_t at = (int64_t)row * g.rst + strip * R + (c & 0xffff);
                  const int sh = (c >> 16) & 31;
                  if (at + R >= top) return false;
                  for (int i = 0; i < R; ++i)
                    A[i] &= (uint32_t)((((uint64_t)lds[at + i + 1] << 32) | lds[at + i]) >> sh);
                }
                if (sa) sv[sa - 1] = A;
                if (q.x & (int)kRecCount) {
                  int64_t n = 0;
                  for (int i = 0; i < R; ++i) n += __builtin_popcount(A[i]);
                  if (q.z < 0 || q.z >= g.nmem) return false;
                  slot[q.z] += n;
                  if (q.w <= r) return false;
                  if (n == 0) r = q.w - 1;  // the kernel tests a whole wave's count
                }
              }
            }
      }
    for (int t = 0; t < g.nmem; ++t) counts[p.mems[g.mem0 + t].idx] += slot[t];
  }
  (void)rpw;
  return true;
}

}  // namespace lpf

// Host run of the launch plan of lpf_full (include/lpf.h).
extern "C" lpf_status lpf_cover_counts(const uint8_t *img, int W, int H, int cx, int cy, int phase,
                                       int R, int S, int waves, int lds_bytes, uint32_t *counts) {
  auto pow2 = [](int v, int hi) { return v == 0 || (v >= 1 && v <= hi && (v & (v - 1)) == 0); };
  if (!img || !counts || W < 1 || H < 1 || W > 4096 || H > 4096 || cx < 0 || cy < 0 || cx >= W ||
      cy >= H || phase < 0 || phase > 1 || !pow2(R, 16) || !pow2(S, 64) || waves < 0 ||
      waves > 16 || lds_bytes < 0 || lds_bytes > 160 * 1024)
    return LPF_E_INVAL;
  try {
    lpf::CoverHost p;
    if (!lpf::plan_cover(W, H, cx, cy, R, S, waves, lds_bytes, 256, p)) return LPF_E_UNSUPPORTED;
    std::vector<int64_t> n((size_t)lpf_num_vectors(cx, cy), -1);
    std::vector<int> seen(n.size(), 0);
    for (const lpf::MemDesc &m : p.mems) {
      n[m.idx] = 0;
      ++seen[m.idx];
    }
    for (int t : seen)
      if (t != 1) return LPF_E_INVAL;
    if (!lpf::run_cover(p, img, W, H, phase, n.data())) return LPF_E_INVAL;
    for (size_t i = 0; i < n.size(); ++i) counts[i] = (uint32_t)n[i];
  } catch (const std::exception &) {
    return LPF_E_NOMEM;
  }
  return LPF_OK;
}
