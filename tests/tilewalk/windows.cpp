// windows.cpp -- host replay of the copy kernels' window walk (copy_geom.hpp):
// rows of every length and start, each element in exactly one window or piece
// of one, a full window on a 16-byte boundary of the target; a row of few
// elements in no more windows than elements.  Test code.
#include <cstdio>
#include <vector>
#include "copy_geom.hpp"
using namespace etc;

static int check(uint32_t nc, int es, uint64_t to, uint32_t group) {
  const int vw = 16 / es;
  std::vector<int> hits(nc, 0);
  if (nc > 1 && group == window_group(nc, es) && windows_per_row(nc, es, group) > nc) return 7;
  for (uint32_t w = 0; w < windows_per_row(nc, es, group); ++w) {
    const Window x = row_window(w, nc, to, es, group);
    if (x.hi <= x.lo) continue;
    if (x.lo < 0 || x.hi > int32_t(nc) || x.hi - x.lo > vw) return 1;
    if (x.hi - x.lo == vw && (to + uint64_t(x.lo) * es) % 16) return 2;
    // a smaller window touches one 16-byte unit only
    if ((to + uint64_t(x.lo) * es) / 16 != (to + uint64_t(x.hi) * es - 1) / 16) return 3;
    if (x.hi - x.lo == vw) {
      for (int32_t e = x.lo; e < x.hi; ++e) ++hits[size_t(e)];
      continue;
    }
    const uint64_t at = to + uint64_t(x.lo) * es;
    const Pieces p = window_pieces(x.hi - x.lo, uint32_t(at % 16) / es, es);
    const bool inside = at % 16 && (at + uint64_t(x.hi - x.lo) * es) % 16;
    const struct { bool is; int32_t e, n; } pieces[3] = {{p.p4, p.e4, 4}, {p.p2, p.e2, 2}, {p.p1, p.e1, 1}};
    for (const auto& q : pieces) {
      if (!q.is) continue;
      if (x.lo + q.e < 0 || x.lo + q.e + q.n > int32_t(nc)) return 5;
      if (!inside && (at + uint64_t(q.e) * es) % (uint64_t(q.n) * es)) return 6;  // a store off its boundary
      for (int32_t e = q.e; e < q.e + q.n; ++e) ++hits[size_t(x.lo + e)];
    }
  }
  for (uint32_t e = 0; e < nc; ++e)
    if (hits[e] != 1) return 4;
  return 0;
}

// The walk over a tile's windows: each of nr rows' windows once, by the
// workgroups of an all-kinds launch (in index order or in XCD runs) and of a
// one-kind launch.
static int check_tile(uint32_t nr, uint32_t nc, int es) {
  const uint32_t vw = 16u / uint32_t(es), lap = kTileElems / vw;
  const TileGeom g{0, 0, nr, nc, true};
  const uint32_t used = sub_used(g);
  for (int order = 0; order < 3; ++order) {
    const uint32_t n = nr * windows_per_row(nc, es, order < 2 ? window_group(nc, es) : kind_window_group(g, es));
    std::vector<int> hits(n, 0);
    const uint32_t per = (order < 2 ? kSubElems : kind_sub_elems(es)) / vw;
    if (per > kSubThreads) return 1;
    for (uint32_t j = 0; j < lap / per; ++j) {
      if (order < 2 && j >= used) continue;
      const uint32_t q = order == 1 ? xcd_run(j, used) : j;
      for (uint32_t lane = 0; lane < per; ++lane)
        for (uint32_t i = q * per + lane; i < n; i += lap) ++hits[i];
    }
    for (uint32_t i = 0; i < n; ++i)
      if (hits[i] != 1) return 2 + order;
  }
  return 0;
}

int main() {
  std::vector<uint32_t> widths;
  for (uint32_t nc = 1; nc <= 600; ++nc) widths.push_back(nc);
  for (uint32_t nc : {1023u, 1024u, 1194u, 1791u, 4097u, 16377u, 16383u, 16384u}) widths.push_back(nc);
  for (int es : {2, 4})
    for (uint32_t nc : widths)
      for (uint64_t m = 0; m < 256; m += uint64_t(es))
        for (uint32_t group : {16u, kSectorBytes})
          if (int e = check(nc, es, 0x7f0000001000ull + m, group)) {
            std::printf("row of %u elements of %d bytes at %llu: error %d\n", nc, es, (unsigned long long)m, e);
            return 1;
          }
  for (int es : {2, 4})
    for (uint32_t nc : widths)
      for (uint32_t nr : {1u, 2u, 3u, kTileElems / nc / 2, kTileElems / nc})
        if (nr && (nr == 1 || nr * nc <= kTileElems))
          if (int e = check_tile(nr, nc, es)) {
            std::printf("tile of %u x %u elements of %d bytes: error %d\n", nr, nc, es, e);
            return 1;
          }
  // the XCD order is a permutation of the sub-chunks in use
  for (uint32_t used = 1; used <= kSubPerTile; ++used) {
    std::vector<int> hits(used, 0);
    for (uint32_t j = 0; j < used; ++j) {
      if (xcd_run(j, used) >= used) return 1;
      ++hits[xcd_run(j, used)];
    }
    for (int h : hits)
      if (h != 1) return 1;
  }
  std::printf("ok\n");
  return 0;
}
