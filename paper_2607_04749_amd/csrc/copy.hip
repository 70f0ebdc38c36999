// copy.hip -- the pack / unpack copy engine for gfx950 (MI355X).
//
// Pure data movement, HBM bound: each launch copies a list of routed boxes
// between a rank's four state arenas (strided rows) and message sections
// (contiguous rows), for all four state kinds, or (Refer) straight from a
// source rank's arenas into a target rank's.  Boxes are pre-cut on the host
// into uniform tiles of up to kTileElems elements per kind.
//
// Launch shape: short-lived one-wavefront workgroups (kSubThreads threads)
// over sub-chunks of the tiles, kSubElems elements of a kind each (1 KB of an
// fp32 kind, one 16-byte vector per lane; 512 B of bf16).  A launch of all
// four kinds (pack, unpack, Refer) gives each workgroup one sub-chunk of
// every kind, copied kind after kind; a launch of one kind (state chunking)
// gives each workgroup kind_group consecutive sub-chunks of that kind, each a
// full wavefront of vectors (kind_sub_elems: 1 KB, 512 bf16 elements or 256
// fp32 ones), 8 KB per workgroup, and walks the tiles in one window per XCD
// at a time (kind_wg_tile).
// Either way a workgroup finds its tile's descriptor once (a binary search of
// the tile table, scalar loads) and then moves a few KB.  The hardware
// dispatches the workgroups in index order, so the whole GPU advances
// through each buffer as one compact front; all-kinds and large one-kind launches reserve
// LDS so that at most 25 of their workgroups share a CU (kSubLdsBytes).  On MI355X this ran 5-14 %
// faster than a persistent grid of one deep-batched workgroup per CU for all
// four kinds, and up to 9 % faster for one kind, and it holds its rate where
// the persistent grid lost about 10 % to an unfavourable relative placement
// of the source and target buffers.  Loads and stores are non-temporal since
// nothing is reused.
//
// Rows that are not whole aligned vectors (widths that no power of two
// divides, or an odd tensor ahead of a box in its message) move in windows of
// the target's 16-byte units (copy_window): unaligned vector loads, aligned
// vector stores.  A copy of four streams with one 16-byte vector per lane ran
// at 6.5 TB/s where both sides start on 128-byte lines, 6.0 where the source
// does not, 5.4 where the target does not start on 64 bytes and 5.1 where
// neither does: a line that two workgroups share is fetched, or merged into
// memory, twice, as neighbouring workgroups lie on different XCDs.  With four
// consecutive KB per XCD (xcd_run) these became 6.25, 5.85 and 5.7, so boxes
// off the lines take their sub-chunks in that order; boxes on them do not,
// which would cost 1.7 %.  Against element-by-element copies on the same
// buffers, GPU time: a 1.9 B GPT from TP4 to TP6 (rows of 597 elements) 915 ->
// 797 us; a 6-layer Llama from TP3 to TP2 (rows of 681 and 454) 69.4 -> 63.2;
// unpacks from TP8 to TP6 with boxes of 7, 27 and 101 columns 66 -> 53, 35 ->
// 30 and 141 -> 124, and the same steps one kind at a time 239 -> 142, 200 ->
// 94 and 415 -> 274.
#include <hip/hip_runtime.h>

#include "copy_desc.hpp"
#include "copy_geom.hpp"
#include "etc.h"

namespace etc {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));  // any element's address

struct CopyArgs {
  const CopyBox* boxes;  // nbox boxes + 1 sentinel (tile0 = ntiles)
  uint32_t nbox;
  uint32_t ntiles;
  int32_t kind;        // the kind to copy (one-kind launches)
  uint32_t mode;       // MsgMode: what peer[] points at
  char* arena[4];
  char* peer[ETC_MAX_PEERS];  // start of each peer's message (kMsgArenas: source arena of kind k)
};

// One kind of one tile: where the copy reads and writes, and the row pitches.
template <bool kPack, int kEs>
struct KindTile {
  using E = typename std::conditional<kEs == 2, uint16_t, uint32_t>::type;
  char* Mb;  // this kind's section of the message, or (Refer) the source arena of this kind
  const char* src;
  char* dst;
  uint64_t sld, dld;  // row pitches in bytes
  __device__ __forceinline__ KindTile(const CopyArgs& a, const CopyBox& b, char* mbase, const TileGeom& g, int kind) {
    char* A = a.arena[kind] + tile_arena_elem(b, g) * kEs;
    Mb = a.mode == kMsgArenas ? a.peer[kind]
                              : mbase + (a.mode == kMsgSections ? section_byte(b.msg_npad, kind) : 0);
    char* M = Mb + tile_msg_elem(b, g) * kEs;
    src = kPack ? A : M;
    dst = kPack ? M : A;
    sld = (kPack ? uint64_t(b.a_ld) : b.m_ld) * kEs;
    dld = (kPack ? b.m_ld : uint64_t(b.a_ld)) * kEs;
  }
  __device__ __forceinline__ const E* from(uint32_t r, uint32_t c) const {
    return reinterpret_cast<const E*>(src + r * sld) + c;
  }
  __device__ __forceinline__ E* to(uint32_t r, uint32_t c) const { return reinterpret_cast<E*>(dst + r * dld) + c; }
  // zero the padding that rounds the box up to a multiple of 8 elements
  __device__ __forceinline__ void zero_pad(const CopyBox& b) const {
    E* tail = reinterpret_cast<E*>(Mb + (b.m_off + uint64_t(b.rows) * b.cols) * kEs);
    if (threadIdx.x < b.pad) tail[threadIdx.x] = 0;
  }
};

// Window w of a row of nc elements, as one vector or up to three pieces.  All
// of a wavefront's loads of a kind are issued before any store of that kind:
// most wavefronts hold an end of some row, and a second load after the first
// store would double their time.  (Rows inside one 16-byte unit went element by element, a load and a
// store in turn: tiny boxes of 5-wide rows 4 to 5 % slower than in pieces.)
template <int kEs>
__device__ __forceinline__ void copy_window(const char* src, char* dst, uint32_t w, uint32_t nc, uint32_t group) {
  using E1 = typename std::conditional<kEs == 2, uint16_t, uint32_t>::type;
  using E2 = typename std::conditional<kEs == 2, uint32_t, uint64_t>::type;
  constexpr int32_t vw = 16 / kEs;
  const Window x = row_window(w, nc, reinterpret_cast<uint64_t>(dst), kEs, group);
  const int32_t m = x.hi > x.lo ? x.hi - x.lo : 0;
  src += int64_t(x.lo) * kEs;
  dst += int64_t(x.lo) * kEs;
  const Pieces p = window_pieces(m, uint32_t(reinterpret_cast<uint64_t>(dst)) % 16u / kEs, kEs);
  u32x4 v;  // each is stored only where it was loaded
  uint64_t v4;
  E2 v2;
  E1 v1;
  if (m == vw) v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(src));
  if (m < vw) {
    if (kEs == 2 && p.p4) __builtin_memcpy(&v4, src + p.e4 * kEs, 8);
    if (p.p2) __builtin_memcpy(&v2, src + p.e2 * kEs, 2 * kEs);
    if (p.p1) __builtin_memcpy(&v1, src + p.e1 * kEs, kEs);
  }
  // one wait for all of them: vmcnt counts stores too, so waits of their own
  // would wait for stores (as this one does for those of the kind before)
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt 0
  if (m == vw) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst));
  if (m < vw) {
    if (kEs == 2 && p.p4) __builtin_memcpy(dst + p.e4 * kEs, &v4, 8);
    if (p.p2) __builtin_memcpy(dst + p.e2 * kEs, &v2, 2 * kEs);
    if (p.p1) __builtin_memcpy(dst + p.e1 * kEs, &v1, kEs);
  }
}

// ---------------------------------------------------------------------------
// All four kinds: one sub-chunk of each kind per workgroup.

// The tile's 16-byte vectors of sub-chunk j, one per lane at most.
template <bool kPack, int kEs, uint32_t kSub>
__device__ __forceinline__ void copy_sub_vectors(const KindTile<kPack, kEs>& k, const TileGeom& g, uint32_t j) {
  constexpr uint32_t vw = 16 / kEs;
  static_assert(kSub / vw <= kSubThreads, "at most one vector per lane");
  const uint32_t vpr = g.nc / vw;
  uint32_t lo, hi;
  sub_range(j, kSub / vw, g.nr * vpr, &lo, &hi);
  const uint32_t i = lo + threadIdx.x;
  if (i < hi) {
    const uint32_t r = g.nr == 1 ? 0 : i / vpr;
    const uint32_t c = i - r * vpr;
    __builtin_nontemporal_store(
        __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(k.src + r * k.sld + uint64_t(c) * 16)),
        reinterpret_cast<u32x4*>(k.dst + r * k.dld + uint64_t(c) * 16));
  }
}

// Sub-chunk j (kSub elements) of one kind of a tile that moves in vectors.
template <bool kPack, int kEs, uint32_t kSub>
__device__ __forceinline__ void copy_sub(const CopyArgs& a, const CopyBox& b, char* mbase, const TileGeom& g,
                                         uint32_t j, int kind) {
  copy_sub_vectors<kPack, kEs, kSub>(KindTile<kPack, kEs>(a, b, mbase, g, kind), g, j);
}

// Sub-chunk j of one kind of a tile of any box, or, where the tile's rows do
// not start on 128-byte lines, sub-chunk `run` in its place.
template <bool kPack, int kEs, uint32_t kSub>
__device__ __forceinline__ void copy_sub_any(const KindTile<kPack, kEs>& k, const CopyBox& b, const TileGeom& g,
                                             uint32_t j, uint32_t run, uint32_t group) {
  if (kPack && j == 0 && g.last && b.pad) k.zero_pad(b);
  const uint64_t bases = reinterpret_cast<uint64_t>(k.dst) | reinterpret_cast<uint64_t>(k.src);
  if ((bases | (g.nr == 1 ? 0 : k.dld | k.sld)) % kLineBytes != 0) j = run;
  if (sub_vectors(b, g, kEs)) {
    copy_sub_vectors<kPack, kEs, kSub>(k, g, j);
    return;
  }
  // windows [j * per, (j + 1) * per), and in a one-row tile the same windows of the next lap
  constexpr uint32_t per = kSub / (16 / kEs), lap = lap_windows(kEs);
  const uint32_t wpr = windows_per_row(g.nc, kEs, group), n = g.nr * wpr;
  if (threadIdx.x < per)
    for (uint32_t i = j * per + threadIdx.x; i < n; i += lap) {
      const uint32_t r = g.nr == 1 ? 0 : i / wpr;
      copy_window<kEs>(k.src + r * k.sld, k.dst + r * k.dld, i - r * wpr, g.nc, group);
    }
}

// All four kinds of a tile of at most one element per lane: the loads of all
// kinds before any store, and no windows to work out.  In windows such tiles took
// longer than element by element: 400 layers of hidden 6 and 10, unpack 196 and
// 200 us (180 and 189 by elements), 128 and 142 this way.
template <bool kPack>
__device__ __forceinline__ void copy_few(const CopyArgs& a, const CopyBox& b, char* mbase, const TileGeom& g) {
  const KindTile<kPack, 2> k0(a, b, mbase, g, 0);
  const KindTile<kPack, 4> k1(a, b, mbase, g, 1), k2(a, b, mbase, g, 2), k3(a, b, mbase, g, 3);
  if (kPack && g.last && b.pad) {
    k0.zero_pad(b);
    k1.zero_pad(b);
    k2.zero_pad(b);
    k3.zero_pad(b);
  }
  if (threadIdx.x >= g.nr * g.nc) return;
  const uint32_t r = g.nr == 1 ? 0 : threadIdx.x / g.nc, c = threadIdx.x - r * g.nc;
  const uint16_t v0 = *k0.from(r, c);
  const uint32_t v1 = *k1.from(r, c), v2 = *k2.from(r, c), v3 = *k3.from(r, c);
  *k0.to(r, c) = v0;
  *k1.to(r, c) = v1;
  *k2.to(r, c) = v2;
  *k3.to(r, c) = v3;
}

template <bool kPack>
__global__ __launch_bounds__(kSubThreads) void copy_sub_kernel(CopyArgs a) {
  const uint32_t t = blockIdx.x / kSubPerTile;
  uint32_t j = blockIdx.x % kSubPerTile;
  const uint32_t bi = box_of_tile(a.boxes, a.nbox, t);
  const CopyBox b = a.boxes[bi];
  const TileGeom g = tile_geom(b, t, a.boxes[bi + 1].tile0);
  char* mbase = a.peer[b.peer];
  if (sub_vectors(b, g, 2) && sub_vectors(b, g, 4)) {
    if (!(b.vec & kLineBox)) j = xcd_run(j, (g.nr * g.nc + kSubElems - 1) / kSubElems);
    copy_sub<kPack, 2, kSubElems>(a, b, mbase, g, j, 0);
    copy_sub<kPack, 4, kSubElems>(a, b, mbase, g, j, 1);
    copy_sub<kPack, 4, kSubElems>(a, b, mbase, g, j, 2);
    copy_sub<kPack, 4, kSubElems>(a, b, mbase, g, j, 3);
    return;
  }
  if (tile_few(g)) {
    if (j == 0) copy_few<kPack>(a, b, mbase, g);
    return;
  }
  const uint32_t used = sub_used(g);
  if (j >= used) return;
  const uint32_t run = xcd_run(j, used);
  copy_sub_any<kPack, 2, kSubElems>(KindTile<kPack, 2>(a, b, mbase, g, 0), b, g, j, run, window_group(g.nc, 2));
#pragma unroll 1  // one body for the three kinds: code that a small launch has to fetch
  for (int kind = 1; kind < 4; ++kind)
    copy_sub_any<kPack, 4, kSubElems>(KindTile<kPack, 4>(a, b, mbase, g, kind), b, g, j, run, window_group(g.nc, 4));
}

// ---------------------------------------------------------------------------
// One kind: kind_group(es) consecutive sub-chunks of kind_sub_elems(es)
// elements of one tile per workgroup.

template <bool kPack, int kEs>
__global__ __launch_bounds__(kSubThreads) void copy_kind_kernel(CopyArgs a) {
  constexpr uint32_t sub = kind_sub_elems(kEs), grp = kind_group(kEs);
  uint32_t t, q;
  if (!kind_wg_tile(blockIdx.x, a.ntiles, kEs, &t, &q)) return;  // past the last tile
  const uint32_t bi = box_of_tile(a.boxes, a.nbox, t);
  const CopyBox b = a.boxes[bi];
  const TileGeom g = tile_geom(b, t, a.boxes[bi + 1].tile0);
  // once per workgroup: with the kind known at launch only, the compiler would
  // work it out anew for every sub-chunk (tiny boxes 7 to 11 % slower)
  const KindTile<kPack, kEs> k(a, b, a.peer[b.peer], g, a.kind);
  if (sub_vectors(b, g, kEs)) {
    // a 4-byte kind moves in vectors of 4 elements, and boxes end at multiples of 8
    if (kPack && q == 0 && g.last && b.pad) k.zero_pad(b);
#pragma unroll
    for (uint32_t i = 0; i < grp; ++i) copy_sub_vectors<kPack, kEs, sub>(k, g, q * grp + i);
    return;
  }
  const uint32_t group = kind_window_group(g, kEs);
#pragma unroll 1
  for (uint32_t i = 0; i < grp; ++i) copy_sub_any<kPack, kEs, sub>(k, b, g, q * grp + i, q * grp + i, group);
}

// LDS reserved per workgroup and never touched, in all-kinds launches: with
// 160 KB of LDS per CU it lets at most 25 of these one-wave workgroups share
// a CU, where they would otherwise fill its 32 wave slots.  The copy keeps
// HBM's queues full either way.  With fewer requests queued, MI355X ran the
// 70B and 7B shares 2-3 % faster in their slower buffer placements, and
// every other all-kinds launch measured within -1 to +1.6 %.  A cap of 21
// workgroups ran 1-3.5 % below the cap of 25.  A one-kind launch, whose
// workgroups spend less of their time on finding their tile, runs 0.3 to 3 %
// faster with the cap from four rounds of all wave slots on (13B, 70B and 7B
// steps one kind at a time: 11637 -> 11312, 15227 -> 14777 and 11807 -> 11506
// us).  Smaller ones, where the rounds are few, ran from 3 % faster to 6 %
// slower (6400 to 8192 workgroups: two rounds instead of one) and keep all 32
// slots of a CU.
constexpr unsigned kSubLdsBytes = 6400;
constexpr uint64_t kCappedKindGrid = 4 * 256 * 32;

}  // namespace

hipError_t launch_copy(bool pack, const CopyBox* boxes, uint32_t nbox, uint32_t ntiles, uint32_t kind_mask,
                       MsgMode mode, void* const arena[4], void* const* peers, int npeers, hipStream_t stream) {
  if (ntiles == 0 || kind_mask == 0) return hipSuccess;
  const bool all = kind_mask == 0xFu;
  const bool single = kind_mask < 16 && (kind_mask & (kind_mask - 1)) == 0;
  if (!all && !single) return hipErrorInvalidValue;  // a launch copies all four kinds or one
  const uint64_t nwg = all ? uint64_t(ntiles) * kSubPerTile : kind_grid(ntiles, kind_mask == 1 ? 2 : 4);
  if (nwg > uint64_t(INT32_MAX)) return hipErrorInvalidValue;
  CopyArgs a{};
  a.boxes = boxes;
  a.nbox = nbox;
  a.ntiles = ntiles;
  a.kind = single ? __builtin_ctz(kind_mask) : 0;
  a.mode = mode;
  for (int k = 0; k < 4; ++k) a.arena[k] = static_cast<char*>(arena[k]);
  for (int p = 0; p < npeers; ++p) a.peer[p] = static_cast<char*>(peers[p]);
  const dim3 grid = dim3(uint32_t(nwg)), block = dim3(kSubThreads);
  const unsigned lds = all || nwg >= kCappedKindGrid ? kSubLdsBytes : 0;
#define ETC_COPY(...) hipLaunchKernelGGL((__VA_ARGS__), grid, block, lds, stream, a)
  if (all) {
    if (pack) ETC_COPY(copy_sub_kernel<true>);
    else ETC_COPY(copy_sub_kernel<false>);
  } else if (kind_mask == 1) {
    if (pack) ETC_COPY(copy_kind_kernel<true, 2>);
    else ETC_COPY(copy_kind_kernel<false, 2>);
  } else {
    if (pack) ETC_COPY(copy_kind_kernel<true, 4>);
    else ETC_COPY(copy_kind_kernel<false, 4>);
  }
#undef ETC_COPY
  return hipGetLastError();
}

}  // namespace etc
