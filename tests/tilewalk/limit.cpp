// limit.cpp -- the grid limit of a copy launch, on the host: a rank of odd
// widths whose tiles by elements just fit a launch, and whose lower tiles by
// windows do not, has the former.  Prints "ok".  Test code.
#include <cstdio>
#include <vector>
#include "copy_geom.hpp"
#include "plan.hpp"
using namespace etc;

// Old rank 0's pack table when a GPT of hidden 1194 goes from TP1 to TP2: the
// attention output is split into 597-wide halves.
static std::vector<CopyBox> table(int layers) {
  etc_plan_t P;
  P.model = {};
  P.model.arch = ETC_ARCH_GPT;
  P.model.num_layers = layers;
  P.model.hidden = 1194;
  P.model.num_heads = P.model.num_kv_heads = 2;
  P.model.ffn_hidden = 1194;
  P.model.vocab = 2;
  P.model.flags = ETC_F_LAYERS_ONLY;
  P.src = Grid{1, 1, 1};
  P.dst = Grid{2, 1, 1};
  P.home = {-1, -1};
  build_host_plan(P);
  std::vector<int32_t> peers;
  return build_pack_boxes(P, 0, &peers, nullptr);
}

static uint64_t by_elems(const std::vector<CopyBox>& v) {
  uint64_t n = 0;
  for (size_t i = 0; i + 1 < v.size(); ++i) {
    const uint64_t rows = v[i].tc == v[i].cols && v[i].rows > 1 ? kTileElems / v[i].cols : v[i].tr;
    n += (v[i].rows + rows - 1) / rows * v[i].ntc;
  }
  return n;
}

int main() {
  const uint64_t limit = uint64_t(INT32_MAX) / kSubPerTile;
  const std::vector<CopyBox> one = table(1);
  const uint64_t few = by_elems(one), many = one.back().tile0;
  const int layers = int(limit / few);
  if (many <= few || many * uint64_t(layers) <= limit) return std::printf("the shape does not reach the limit\n"), 1;
  const std::vector<CopyBox> v = table(layers);
  if (v.back().tile0 != few * uint64_t(layers)) return std::printf("%u tiles, not by elements\n", v.back().tile0), 1;
  for (size_t i = 0; i + 1 < v.size(); ++i) {
    const TileGeom g = tile_geom(v[i], v[i + 1].tile0 - 1, v[i + 1].tile0);
    if (v[i + 1].tile0 <= v[i].tile0 || g.r0 + g.nr != v[i].rows || g.c0 + g.nc != v[i].cols)
      return std::printf("box %zu is not covered\n", i), 1;
  }
  std::printf("ok\n");
  return 0;
}
