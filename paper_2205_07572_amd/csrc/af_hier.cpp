// af_hier.cpp -- host quadtree of equal-size patches (Sec. 3).
//
// A hierarchy is a leaf set of the forest of quadtrees rooted at the
// n0x x n0y level-0 patches of a periodic rectangle.  Patch (l, ix, iy) of
// level l covers cells [ix m, (ix+1) m) x [iy m, (iy+1) m) of level l; its
// children are (l+1, 2ix+qx, 2iy+qy).  Lookups go through dense per-level
// tables (leaf id or -1), so every query is O(levels).
#include <algorithm>
#include <cstdio>
#include <string>
#include <vector>

#include "af_hier.h"

namespace af {

namespace {
// v modulo n; one step outside [0, n), as a neighbour is, without a division
inline long long wrapi(long long v, long long n) {
  if (v < 0) v += n;
  else if (v >= n) v -= n;
  return v >= 0 && v < n ? v : ((v % n) + n) % n;
}
}  // namespace
int Hier::find(int l, long long px, long long py) const {
  if (l < 0 || l > lmax) return -1;
  const long long nx = npx(l), ny = npy(l);
  px = wrapi(px, nx);
  py = wrapi(py, ny);
  return lut[size_t(lut_off[l] + py * nx + px)];
}

// Leaf covering patch position (l, px, py): the position itself or an
// ancestor; returns its id and level, or -1 if the position is subdivided.
int Hier::cover(int l, long long px, long long py, int* lev) const {
  for (int k = l; k >= 0; --k) {
    const int id = find(k, px >> (l - k), py >> (l - k));
    if (id >= 0) {
      *lev = k;
      return id;
    }
    // positions are wrapped per level inside find; shifting a wrapped value
    // stays consistent because every level's extent is a multiple of 2
  }
  return -1;
}

std::string Hier::build(const std::vector<Leaf>& in) {
  leaves = in;
  const int n = int(leaves.size());
  if (n == 0) return "empty leaf set";
  lut_off.assign(lmax + 2, 0);
  long long total = 0;
  for (int l = 0; l <= lmax; ++l) {
    lut_off[l] = int(total);
    total += (long long)npx(l) * npy(l);
  }
  lut_off[lmax + 1] = int(total);
  if (total > (1LL << 28)) return "lookup tables too large (lmax too high)";
  lut.assign(size_t(total), -1);
  level_first.assign(lmax + 2, -1);
  level_count.assign(lmax + 2, 0);
  int prev_level = -1;
  for (int k = 0; k < n; ++k) {
    const Leaf& L = leaves[k];
    if (L.level < 0 || L.level > lmax) return "leaf level out of range";
    if (L.ix < 0 || L.ix >= npx(L.level) || L.iy < 0 || L.iy >= npy(L.level)) return "leaf index out of range";
    if (L.level < prev_level) return "leaves must be sorted by level";
    prev_level = L.level;
    int& slot = lut[size_t(lut_off[L.level] + (long long)L.iy * npx(L.level) + L.ix)];
    if (slot >= 0) return "duplicate leaf";
    slot = k;
    if (level_first[L.level] < 0) level_first[L.level] = k;
    level_count[L.level]++;
  }
  // exact tiling: no leaf has a leaf ancestor, and the areas add up
  long long area = 0;
  for (const Leaf& L : leaves) {
    area += 1LL << (2 * (lmax - L.level));
    for (int k = L.level - 1; k >= 0; --k)
      if (find(k, L.ix >> (L.level - k), L.iy >> (L.level - k)) >= 0) return "leaf overlaps an ancestor leaf";
  }
  if (area != (long long)n0x * n0y << (2 * lmax)) return "leaves do not cover the domain";
  // 2:1 balance across edges and corners (periodic): the level-l positions
  // around every leaf must be covered by leaves of level >= l-1.  A leaf is
  // pure if all eight are leaves of its own level.
  pure.assign(n, 1);
  for (int k = 0; k < n; ++k) {
    const Leaf& L = leaves[k];
    for (int dy = -1; dy <= 1; ++dy)
      for (int dx = -1; dx <= 1; ++dx) {
        if ((!dx && !dy) || find(L.level, L.ix + dx, L.iy + dy) >= 0) continue;
        pure[k] = 0;
        int lev;
        if (cover(L.level - 1, (L.ix + dx) >> 1, (L.iy + dy) >> 1, &lev) >= 0 && lev < L.level - 1)
          return "hierarchy is not 2:1 balanced";
      }
  }
  // side relations
  rel.assign(size_t(n) * 4, 0);
  side_mask.assign(n, 0);
  static const int sdx[4] = {-1, 1, 0, 0}, sdy[4] = {0, 0, -1, 1};
  for (int k = 0; k < n; ++k) {
    if (pure[k]) continue;
    const Leaf& L = leaves[k];
    for (int s = 0; s < 4; ++s) {
      const long long px = L.ix + sdx[s], py = L.iy + sdy[s];
      int r;
      if (find(L.level, px, py) >= 0) r = 0;
      else if (L.level > 0 && find(L.level - 1, wrapi(px, npx(L.level)) >> 1, wrapi(py, npy(L.level)) >> 1) >= 0) r = -1;
      else r = 1;
      rel[size_t(k) * 4 + s] = int8_t(r);
      if (r != 0) side_mask[k] |= uint8_t(1 << s);
    }
  }
  // coarse-fine faces per coarse level, in the order (coarse leaf, cell row,
  // cell column, side)
  faces.assign(lmax + 1, {});
  for (int k = 0; k < n; ++k) {
    if (pure[k]) continue;
    const Leaf& C = leaves[k];
    int fine[4][2];  // the two leaves facing side s
    bool any = false;
    for (int s = 0; s < 4; ++s) {
      if (rel[size_t(k) * 4 + s] != 1) continue;
      any = true;
      for (int q = 0; q < 2; ++q) {
        const long long fx = s == 0 ? 2LL * C.ix - 1 : s == 1 ? 2LL * C.ix + 2 : 2LL * C.ix + q;
        const long long fy = s == 2 ? 2LL * C.iy - 1 : s == 3 ? 2LL * C.iy + 2 : 2LL * C.iy + q;
        if ((fine[s][q] = find(C.level + 1, fx, fy)) < 0) return "internal: missing fine neighbour";
      }
    }
    if (!any) continue;
    for (int cj = 0; cj < m; ++cj)
      for (int ci = 0; ci < m; ci += (cj == 0 || cj == m - 1) ? 1 : m - 1)
        for (int s = 0; s < 4; ++s) {
          const bool on = s == 0 ? ci == 0 : s == 1 ? ci == m - 1 : s == 2 ? cj == 0 : cj == m - 1;
          if (!on || rel[size_t(k) * 4 + s] != 1) continue;
          CFFace F;
          F.coarse = k;
          F.side = s;
          F.k = s < 2 ? cj : ci;
          // the two fine faces facing coarse face F.k: 2 F.k and the next,
          // m of them on each fine leaf
          const int q = 2 * F.k >= m ? 1 : 0;
          F.fine = fine[s][q];
          F.fk = 2 * F.k - q * m;
          faces[C.level].push_back(F);
        }
  }
  finest = 0;
  for (const Leaf& L : leaves) finest = std::max(finest, L.level);
  return "";
}

// Regrid (Sec. 3): refine tagged leaves, close under 2:1 corner balance,
// coarsen qualifying families, sort by (level, iy, ix).
std::vector<Leaf> Hier::regrid(const int8_t* tags) const {
  // the candidate leaf set as dense per-level flags, indexed like the lookup
  // table; scanning them level by level, row by row gives the (level, iy, ix)
  // order of the result
  const size_t total = lut.size();
  auto at = [&](int l, int px, int py) { return size_t(lut_off[l]) + size_t(py) * size_t(npx(l)) + size_t(px); };
  std::vector<uint8_t> cur(total, 0), was(total, 0);
  std::vector<int8_t> old_tag(total, 0);
  for (size_t k = 0; k < leaves.size(); ++k) {
    const Leaf& L = leaves[k];
    const size_t e = at(L.level, L.ix, L.iy);
    was[e] = 1;
    old_tag[e] = tags[k];
    if (tags[k] == 1 && L.level < lmax) {
      for (int q = 0; q < 4; ++q) cur[at(L.level + 1, 2 * L.ix + (q & 1), 2 * L.iy + (q >> 1))] = 1;
    } else {
      cur[e] = 1;
    }
  }
  // level of the leaf of the set covering position (l, px, py) inside the
  // domain, itself or an ancestor; -1 if the position is subdivided
  auto covering = [&](int l, int px, int py) {
    for (int k = l; k >= 0; --k)
      if (cur[at(k, px >> (l - k), py >> (l - k))]) return k;
    return -1;
  };
  // every leaf of the set, in (level, iy, ix) order
  auto for_each = [&](auto&& f) {
    for (int l = 0; l <= lmax; ++l)
      for (int iy = 0; iy < npy(l); ++iy) {
        const uint8_t* row = &cur[at(l, 0, iy)];
        for (int ix = 0; ix < npx(l); ++ix)
          if (row[ix]) f(l, ix, iy);
      }
  };
  // balance closure: a leaf two levels coarser than a touching leaf splits,
  // and its children are looked at in their turn (the closure does not depend
  // on the order; a leaf once in balance stays so, since others only split)
  std::vector<Leaf> todo;
  for_each([&](int l, int ix, int iy) {
    if (l >= 2) todo.push_back({l, ix, iy});
  });
  while (!todo.empty()) {
    const Leaf L = todo.back();
    todo.pop_back();
    if (!cur[at(L.level, L.ix, L.iy)]) continue;  // split meanwhile
    for (int dy = -1; dy <= 1; ++dy)
      for (int dx = -1; dx <= 1; ++dx) {
        if (!dx && !dy) continue;
        const int px = int(wrapi(L.ix + dx, npx(L.level))), py = int(wrapi(L.iy + dy, npy(L.level)));
        int lev;
        while ((lev = covering(L.level, px, py)) >= 0 && lev <= L.level - 2) {
          const int sx = px >> (L.level - lev), sy = py >> (L.level - lev);
          cur[at(lev, sx, sy)] = 0;
          for (int q = 0; q < 4; ++q) {
            const Leaf C{lev + 1, 2 * sx + (q & 1), 2 * sy + (q >> 1)};
            cur[at(C.level, C.ix, C.iy)] = 1;
            if (C.level >= 2) todo.push_back(C);
          }
        }
      }
  }
  // families: all four siblings are leaves tagged -1, and no sibling has a
  // subdivided level-l neighbour position outside the family
  std::vector<Leaf> parents;
  for_each([&](int l, int ix, int iy) {
    if (l == 0 || (ix & 1) || (iy & 1)) return;
    bool ok = true;
    for (int q = 0; q < 4 && ok; ++q) {
      const size_t e = at(l, ix + (q & 1), iy + (q >> 1));
      if (!cur[e] || !was[e] || old_tag[e] != -1) ok = false;
    }
    for (int q = 0; q < 4 && ok; ++q) {
      const int sx = ix + (q & 1), sy = iy + (q >> 1);
      for (int dy = -1; dy <= 1 && ok; ++dy)
        for (int dx = -1; dx <= 1 && ok; ++dx) {
          if (!dx && !dy) continue;
          // finer leaves touch the parent
          if (covering(l, int(wrapi(sx + dx, npx(l))), int(wrapi(sy + dy, npy(l)))) < 0) ok = false;
        }
    }
    if (ok) parents.push_back({l - 1, ix >> 1, iy >> 1});
  });
  for (const Leaf& P : parents) {
    for (int q = 0; q < 4; ++q) cur[at(P.level + 1, 2 * P.ix + (q & 1), 2 * P.iy + (q >> 1))] = 0;
    cur[at(P.level, P.ix, P.iy)] = 1;
  }
  std::vector<Leaf> out;
  for_each([&](int l, int ix, int iy) { out.push_back({l, ix, iy}); });
  return out;
}

}  // namespace af
