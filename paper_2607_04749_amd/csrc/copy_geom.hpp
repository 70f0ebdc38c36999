// copy_geom.hpp -- tile geometry of the copy engine: which box a tile belongs
// to, and the rows and columns of a tile.
// Host and device share it, so the planner's bounds checks and the kernel
// walk the same tiles.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "copy_desc.hpp"

namespace etc {

// Index of the box holding tile t: the last box with tile0 <= t.
__host__ __device__ inline uint32_t box_of_tile(const CopyBox* boxes, uint32_t nbox, uint32_t t) {
  uint32_t lo = 0, hi = nbox;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (boxes[mid].tile0 <= t) lo = mid;
    else hi = mid;
  }
  return lo;
}

struct TileGeom {
  uint32_t r0, c0, nr, nc;  // tile rows [r0, r0+nr), columns [c0, c0+nc) of the box
  bool last;                // last tile of its box
};

// Geometry of tile t of box b (next0 = first tile of the next box).
__host__ __device__ inline TileGeom tile_geom(const CopyBox& b, uint32_t t, uint32_t next0) {
  TileGeom g;
  const uint32_t j = t - b.tile0;
  const uint32_t band = j / b.ntc, tcol = j - band * b.ntc;
  g.r0 = band * b.tr;
  g.c0 = tcol * b.tc;
  g.nr = b.tr < b.rows - g.r0 ? b.tr : b.rows - g.r0;
  g.nc = b.tc < b.cols - g.c0 ? b.tc : b.cols - g.c0;
  g.last = t + 1 == next0;
  return g;
}

// Element offsets of a tile's first element on each side.
__host__ __device__ inline uint64_t tile_arena_elem(const CopyBox& b, const TileGeom& g) {
  return b.a_off + uint64_t(g.r0) * b.a_ld + g.c0;
}
__host__ __device__ inline uint64_t tile_msg_elem(const CopyBox& b, const TileGeom& g) {
  return b.m_off + uint64_t(g.r0) * b.m_ld + g.c0;
}

// Sub-chunks: a tile splits into kSubPerTile sub-chunks, copied by
// workgroups of kSubThreads threads (one wavefront); a launch of all four
// kinds gives workgroup kSubPerTile * t + j sub-chunk j of tile t.  For each
// kind, sub-chunk j covers the tile's vectors [j * kSubElems / vw,
// (j + 1) * kSubElems / vw) when the kind moves in 16-byte vectors of vw
// elements (one vector per lane at most), in row-major order over the tile and
// clipped to its size; else the windows of as many vectors, and those a whole
// tile of vectors further on.
// A launch of one kind cuts a tile of that kind into kind_sub_elems(es)-element
// sub-chunks instead and gives each workgroup kind_group(es) consecutive
// ones of one tile.
constexpr uint32_t kSubThreads = 64;
constexpr uint32_t kSubPerTile = 64;
constexpr uint32_t kSubElems = kTileElems / kSubPerTile;  // 256
static_assert(kSubElems / 4 <= kSubThreads, "a 4-byte kind's sub-chunk must fit one vector per lane");

// One-kind launches, for a kind of es bytes per element: elements per
// sub-chunk (one 16-byte vector per lane of the wavefront: 256 of a 4-byte
// kind, 512 of bf16), sub-chunks per workgroup (8 KB per workgroup for
// every kind), and workgroups per tile.
__host__ __device__ constexpr uint32_t kind_sub_elems(int es) { return kSubThreads * 16u / uint32_t(es); }
__host__ __device__ constexpr uint32_t kind_group(int /*es*/) { return 8u; }
__host__ __device__ constexpr uint32_t kind_wg_per_tile(int es) {
  return kTileElems / kind_sub_elems(es) / kind_group(es);
}
static_assert(kTileElems % (kind_sub_elems(2) * kind_group(2)) == 0 &&
                  kTileElems % (kind_sub_elems(4) * kind_group(4)) == 0,
              "whole groups per tile");
static_assert(kind_sub_elems(2) / 8 <= kSubThreads && kind_sub_elems(4) / 4 <= kSubThreads,
              "a one-kind sub-chunk must fit one vector per lane");

// The workgroups of a one-kind launch walk the tile list in windows, one
// per XCD at a time: the list is cut into kXcds * kKindWindows equal windows
// of consecutive tiles, and the workgroups of XCD x (the hardware deals
// workgroup w to XCD w % kXcds) copy window x, then window x + kXcds, ...,
// each in tile order.  A launch of one kind has one read and one write
// stream; eight fronts far apart in each, every one fed by one XCD, kept
// them faster than one compact front on MI355X (the all-kinds launches,
// with four streams each way, stay compact).  Two windows per XCD rather
// than one keep the XCDs' shares of strided and contiguous tiles even.
constexpr uint32_t kXcds = 8;
constexpr uint32_t kKindWindows = 2;
__host__ __device__ inline uint32_t kind_window_tiles(uint32_t ntiles) {
  return (ntiles + kXcds * kKindWindows - 1) / (kXcds * kKindWindows);
}
// workgroups in a one-kind launch over ntiles tiles (a few past the last
// tile, when the windows overhang it, find no tile)
__host__ __device__ inline uint64_t kind_grid(uint32_t ntiles, int es) {
  return uint64_t(kXcds) * kKindWindows * kind_window_tiles(ntiles) * kind_wg_per_tile(es);
}
// Tile t and group q (sub-chunks [q * kind_group, (q + 1) * kind_group)) of
// workgroup w of a one-kind launch; false for a workgroup past the last tile.
__host__ __device__ inline bool kind_wg_tile(uint32_t w, uint32_t ntiles, int es, uint32_t* t, uint32_t* q) {
  const uint32_t gpt = kind_wg_per_tile(es), per = kind_window_tiles(ntiles);
  const uint32_t x = w % kXcds, k = w / kXcds, s = k / gpt, m = s / per;
  *t = (m * kXcds + x) * per + s % per;
  *q = k % gpt;
  return m < kKindWindows && *t < ntiles;
}

// Whether the kind of element size es moves a tile in 16-byte vectors: the
// box is vector-aligned for that size and every row of the tile is whole
// vectors (other tiles move in windows, below).
__host__ __device__ inline bool sub_vectors(const CopyBox& b, const TileGeom& g, int es) {
  return ((b.vec >> (es == 2 ? 0 : 1)) & 1) && g.nc % (16u / uint32_t(es)) == 0;
}

// Index range [lo, hi) of sub-chunk j over n items, per items per sub-chunk.
__host__ __device__ inline void sub_range(uint32_t j, uint32_t per, uint32_t n, uint32_t* lo, uint32_t* hi) {
  const uint32_t a = j * per;
  *lo = a < n ? a : n;
  *hi = a + per < n ? a + per : n;
}

// Tiles that cannot move in aligned 16-byte vectors are cut into windows: the
// 16-byte units of the target side that a row of the tile touches, in groups
// of 64 bytes, so that no 64-byte sector is shared by two workgroups but at the
// ends of a row.  A window that lies inside the row moves as one vector (its
// load may be unaligned, its store is not), the first and last of a row in
// smaller pieces.  Every row has windows_per_row of them, a few before its
// start and past its end empty.  Groups of 16 and of 128 bytes measured up to
// 3 % slower (rows of 1443 to 3813 elements) and 4 % slower (597 elements).
// All-kinds launches, which have workgroups in plenty, go without the grouping
// for rows of less than 512 bytes: most of their windows would be empty (a row
// of 3 elements has 2 windows, or 8 in a group).  Packs and unpacks with rows
// of 7 to 113 elements took 1 to 15 % less time that way, 1 to 4 % less than
// with the line at 128 bytes and as much as at 256.
constexpr uint32_t kSectorBytes = 64, kNarrowBytes = 512;
__host__ __device__ inline uint32_t window_group(uint32_t nc, int es) {
  return nc * uint32_t(es) < kNarrowBytes ? 16u : kSectorBytes;
}
__host__ __device__ inline uint32_t windows_per_row(uint32_t nc, int es, uint32_t group) {
  return (nc * uint32_t(es) + 2 * group - 1 - uint32_t(es)) / group * (group / 16u);
}
// Whether an all-kinds launch copies a tile that moves in windows one element per lane.
__host__ __device__ inline bool tile_few(const TileGeom& g) { return g.nr * g.nc <= kSubThreads; }
// Windows in one pass of a tile's sub-chunks.  Tiles of several rows hold no
// more (tiles.hip); a one-row tile may, and the first sub-chunks then take
// the rest in a second pass.
__host__ __device__ constexpr uint32_t lap_windows(int es) { return kTileElems / (16u / uint32_t(es)); }
// One-kind launches group such rows too where the tile's windows fit a pass all
// the same: the eight sub-chunks of a workgroup follow each other, and fewer
// windows mean fewer workgroups at work.  Boxes of 5, 7 and 9 columns one kind at
// a time: 131, 141 and 120 us, without the grouping 141, 156 and 126.
__host__ __device__ inline uint32_t kind_window_group(const TileGeom& g, int es) {
  return g.nr * windows_per_row(g.nc, es, kSectorBytes) <= lap_windows(es) ? kSectorBytes : window_group(g.nc, es);
}
// Sub-chunks of an all-kinds launch past this many of a tile hold nothing of
// any kind, in windows or (fewer) in vectors.
__host__ __device__ inline uint32_t sub_used(const TileGeom& g) {
  const uint32_t w4 = windows_per_row(g.nc, 4, window_group(g.nc, 4));
  const uint32_t w2 = 2 * windows_per_row(g.nc, 2, window_group(g.nc, 2));
  const uint32_t n = (g.nr * (w4 > w2 ? w4 : w2) + kSubThreads - 1) / kSubThreads;
  return n < kSubPerTile ? n : kSubPerTile;
}
// Elements [lo, hi) of a row of nc elements in its window w, where the row
// starts at address `to` on the target side; empty when hi <= lo.
struct Window {
  int32_t lo, hi;
};
__host__ __device__ inline Window row_window(uint32_t w, uint32_t nc, uint64_t to, int es, uint32_t group) {
  const int32_t vw = 16 / es, at = int32_t(w) * vw - int32_t(uint32_t(to) & (group - 1)) / es;
  return Window{at > 0 ? at : 0, at + vw < int32_t(nc) ? at + vw : int32_t(nc)};
}

// The pieces of 4, 2 and 1 elements that a window of m < 16 / es elements moves
// in (p: whether there is one, e: its first element), where the window starts
// `at` elements into its 16-byte unit of the target side.  The last window of
// a row starts its unit and the first one ends it: big pieces lie towards that
// end, so each is aligned on the target side.  Those of a row inside one unit
// need not be.
struct Pieces {
  bool p4, p2, p1;
  int32_t e4, e2, e1;
};
__host__ __device__ inline Pieces window_pieces(int32_t m, uint32_t at, int es) {
  const bool first = at != 0 && at + uint32_t(m) == 16u / uint32_t(es);
  return Pieces{es == 2 && (m & 4) != 0, (m & 2) != 0, (m & 1) != 0,
                first ? m & 3 : 0, first ? m & 1 : m & 4, first ? 0 : m & 6};
}

// The hardware deals workgroup w to XCD w % kXcds.  Where a tile's rows do not
// start on 128-byte lines, neighbouring sub-chunks share lines, and the L2 of
// one XCD should see both: an order of the tile's sub-chunks in which each XCD
// takes four consecutive ones out of every 4 * kXcds.  Sub-chunks past the
// last 4 * kXcds that are all in use stay in place, or a tile of few
// would keep some XCDs idle.
__host__ __device__ inline uint32_t xcd_run(uint32_t j, uint32_t used) {
  constexpr uint32_t m = 4 * kXcds - 1;
  return (j | m) < used ? (j & ~m) | ((j & (kXcds - 1)) * 4) | ((j & m) / kXcds) : j;
}

// Byte offset of kind k's section inside a message of npad elements per section.
__host__ __device__ inline uint64_t section_byte(uint64_t npad, int k) {
  return npad * (k == 0 ? 0 : (k == 1 ? 2 : (k == 2 ? 6 : 10)));
}

}  // namespace etc
