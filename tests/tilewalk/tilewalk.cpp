// tilewalk.cpp -- host replay of the copy kernels' walks over the copy
// tables the planner builds (pack, unpack and Refer; all kinds at once, one
// sub-chunk of each kind per workgroup; one kind at a time, kind_group(es)
// sub-chunks of kind_sub_elems(es) elements per workgroup).  Tiles of whole
// aligned vectors are walked in vectors, others in windows and their pieces, and
// all-kinds launches in the order of their XCD runs, as the kernels do.  For
// every tile it checks that each access stays inside its arena, message
// section or source arena, that vectors are 16-byte aligned (of windows, the
// target side, and of pieces each to its own size), that a sub-chunk needs no
// more lanes than a workgroup has, and that the writes of a launch cover the
// target bytes exactly once: each message (padding included) for a pack, each
// target piece for the unpack plus Refer of one target.
// Every device pointer is 256-byte aligned, so addresses here count from 0.
//
// Test code: it links the library's host planner and its tile geometry
// header; it computes no expected values.
//
// usage: tilewalk arch L h nh nkv ffn V max_pos tied flags  tp pp dp  tp pp dp
//                 refer pairing [failed ...]
//   refer: 1 builds the plan with ETC_PLAN_DIRECT_REFER
//   pairing: "identity", "sketch", or comma-separated pair[d] (-1 = none)
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>
#include "copy_geom.hpp"
#include "plan.hpp"
using namespace etc;
struct Iv { uint64_t lo, hi; };
static int errors = 0;
#define FAIL(...) do { if (errors++ < 20) { fprintf(stderr, __VA_ARGS__); fputc('\n', stderr);} } while (0)

static void merge_equal(std::vector<Iv> w, std::vector<Iv> want, const std::string& what) {
  std::sort(w.begin(), w.end(), [](Iv a, Iv b) { return a.lo < b.lo; });
  for (size_t i = 1; i < w.size(); ++i)
    if (w[i].lo < w[i - 1].hi) { FAIL("%s: overlapping writes", what.c_str()); return; }
  std::vector<Iv> m;
  for (auto x : w) { if (!m.empty() && m.back().hi == x.lo) m.back().hi = x.hi; else m.push_back(x); }
  std::sort(want.begin(), want.end(), [](Iv a, Iv b) { return a.lo < b.lo; });
  std::vector<Iv> mw;
  for (auto x : want) { if (x.hi == x.lo) continue; if (!mw.empty() && mw.back().hi == x.lo) mw.back().hi = x.hi; else mw.push_back(x); }
  if (m.size() != mw.size()) { FAIL("%s: coverage pieces %zu vs %zu", what.c_str(), m.size(), mw.size()); return; }
  for (size_t i = 0; i < m.size(); ++i)
    if (m[i].lo != mw[i].lo || m[i].hi != mw[i].hi) { FAIL("%s: coverage differs", what.c_str()); return; }
}

// padded elements per kind section of message s -> d (0 when empty)
static uint64_t npad_of(const etc_plan_t& P, int s, int d) {
  const auto* m = P.find_msg(s, d);
  return m ? m->npad : 0;
}

// Sort and merge one tile's write intervals in place, failing on any overlap.
static void merge_tile(std::vector<Iv>& w, const char* what) {
  const auto before = [](Iv a, Iv b) { return a.lo < b.lo; };
  if (!std::is_sorted(w.begin(), w.end(), before)) std::sort(w.begin(), w.end(), before);
  size_t n = 0;  // merged so far
  for (const Iv x : w) {
    if (x.hi == x.lo) continue;
    if (n && x.lo < w[n - 1].hi) { FAIL("%s: sub-chunks of one tile overlap", what); continue; }
    if (n && w[n - 1].hi == x.lo) w[n - 1].hi = x.hi; else w[n++] = x;
  }
  w.resize(n);
}

// One kind of one tile: byte offsets of its first row on both sides, and what
// bounds them.
struct KindWalk {
  uint64_t a0, m0, a_end, m_lo, m_end;  // arena side, message side (or source arena)
  uint64_t a_ld, m_ld;                  // row pitches
  bool pack;
  int es, kind;
  std::vector<Iv>& writes;

  uint64_t to(uint32_t r) const { return pack ? m0 + r * m_ld : a0 + r * a_ld; }  // target side of row r
  // elements [c0, c1) of row r, moved by one lane
  void move(uint32_t r, int64_t c0, int64_t c1) {
    const uint64_t alo = a0 + r * a_ld + c0 * es, mlo = m0 + r * m_ld + c0 * es, n = uint64_t(c1 - c0) * es;
    if (alo + n > a_end) FAIL("arena OOB kind %d", kind);
    if (mlo < m_lo || mlo + n > m_end) FAIL("message OOB kind %d", kind);
    writes.push_back(pack ? Iv{mlo, mlo + n} : Iv{alo, alo + n});
  }
};

// The vectors of sub-chunk j of a tile.
static void walk_vectors(KindWalk& k, const TileGeom& g, uint32_t per, uint32_t j) {
  const uint32_t vw = 16u / uint32_t(k.es), vpr = g.nc / vw;
  if (per > kSubThreads) FAIL("a vector sub-chunk needs more lanes than threads");
  if (g.nc % vw) FAIL("vector rows not whole vectors");
  uint32_t lo, hi;
  sub_range(j, per, g.nr * vpr, &lo, &hi);
  if (lo >= hi) return;
  for (uint32_t r = lo / vpr; lo < hi && r <= (hi - 1) / vpr; ++r) {
    if ((k.a0 + r * k.a_ld) % 16 || (k.m0 + r * k.m_ld) % 16) FAIL("vector misaligned kind %d", k.kind);
    k.move(r, int64_t(std::max(lo, r * vpr) - r * vpr) * vw, int64_t(std::min(hi, (r + 1) * vpr) - r * vpr) * vw);
  }
}

// The windows of sub-chunk j of a tile, those of a second pass included.
static void walk_windows(KindWalk& k, const TileGeom& g, uint32_t per, uint32_t j, uint32_t group) {
  const uint32_t vw = 16u / uint32_t(k.es), wpr = windows_per_row(g.nc, k.es, group), n = g.nr * wpr;
  if (per > kSubThreads) FAIL("a sub-chunk of windows needs more lanes than threads");
  for (uint32_t lane = 0; lane < per; ++lane)
    for (uint32_t i = j * per + lane; i < n; i += lap_windows(k.es)) {
      const uint32_t r = i / wpr;
      const Window x = row_window(i - r * wpr, g.nc, k.to(r), k.es, group);
      if (x.hi <= x.lo) continue;
      const uint64_t at = k.to(r) + uint64_t(x.lo) * k.es;
      const uint32_t m = uint32_t(x.hi - x.lo);
      if (m == vw) {
        if (at % 16) FAIL("window off its 16-byte unit");
        k.move(r, x.lo, x.hi);
        continue;
      }
      const bool inside = at % 16 && (at + uint64_t(m) * k.es) % 16;
      const Pieces p = window_pieces(int32_t(m), uint32_t(at % 16) / uint32_t(k.es), k.es);
      const struct { bool is; int32_t e, n; } pieces[3] = {{p.p4, p.e4, 4}, {p.p2, p.e2, 2}, {p.p1, p.e1, 1}};
      for (const auto& q : pieces) {
        if (!q.is) continue;
        if (q.e < 0 || q.e + q.n > int32_t(m)) FAIL("a piece outside its window");
        if (!inside && (at + uint64_t(q.e) * k.es) % (uint64_t(q.n) * k.es)) FAIL("piece misaligned");
        k.move(r, x.lo + q.e, x.lo + q.e + q.n);
      }
    }
}

// A tile of at most one element per lane.
static void walk_few(KindWalk& k, const TileGeom& g) {
  for (uint32_t lane = 0; lane < kSubThreads && lane < g.nr * g.nc; ++lane) {
    const uint32_t r = g.nr == 1 ? 0 : lane / g.nc;
    k.move(r, lane - r * g.nc, lane - r * g.nc + 1);
  }
}

// Replay a launch as the kernels run it: for all four kinds, workgroup
// t * kSubPerTile + j copies sub-chunk j (kSubElems elements) of every kind
// of tile t, or the one that xcd_run gives in its place; for one kind of es
// bytes, workgroup w of kind_grid(ntiles, es) copies, when kind_wg_tile(w)
// gives it tile t and group q, its sub-chunks [q * G, (q + 1) * G) of
// kind_sub_elems(es) elements, G = kind_group(es).
static void replay_sub(const std::vector<CopyBox>& v, bool pack, bool sectioned, uint32_t kind_mask,
                       uint64_t arena_elems, const std::vector<uint64_t>& peer_bytes,
                       std::vector<std::vector<Iv>> W[4], std::vector<Iv> A[4], bool arenas) {
  const uint32_t nbox = uint32_t(v.size() - 1), ntiles = v.back().tile0;
  const bool all = kind_mask == 0xFu;
  const int kes = kind_mask == 1u ? 2 : 4;  // element size of a one-kind launch
  const uint32_t sub_elems = all ? kSubElems : kind_sub_elems(kes);
  const uint32_t subs_per_tile = kTileElems / sub_elems;
  // one-kind launches: the groups each tile receives, from the whole grid
  std::vector<std::vector<uint32_t>> groups_of;
  if (!all) {
    const uint64_t grid = kind_grid(ntiles, kes);
    if (grid > uint64_t(INT32_MAX)) { FAIL("grid over 2^31 - 1 workgroups"); return; }
    if (grid < uint64_t(ntiles) * kind_wg_per_tile(kes)) FAIL("one-kind grid smaller than the work");
    groups_of.resize(ntiles);
    for (uint64_t w = 0; w < grid; ++w) {
      uint32_t t, q;
      if (!kind_wg_tile(uint32_t(w), ntiles, kes, &t, &q)) continue;  // coverage below catches a wrong refusal
      if (t >= ntiles || q >= kind_wg_per_tile(kes)) { FAIL("workgroup %llu maps outside", (unsigned long long)w); continue; }
      groups_of[t].push_back(q);
    }
  }
  if (uint64_t(ntiles) * kSubPerTile > uint64_t(INT32_MAX)) { FAIL("grid over 2^31 - 1 workgroups"); return; }
  std::vector<uint32_t> subs;
  std::vector<char> seen;
  std::vector<Iv> writes;
  for (uint32_t t = 0; t < ntiles; ++t) {
    const uint32_t bi = box_of_tile(v.data(), nbox, t);  // the same for every j of the tile
    if (bi >= nbox) { FAIL("tile past last box"); return; }
    const CopyBox& b = v[bi];
    const TileGeom g = tile_geom(b, t, v[bi + 1].tile0);
    if (g.nr == 0 || g.nc == 0 || g.r0 >= b.rows || g.c0 >= b.cols) FAIL("empty/outside tile");
    if (!arenas && b.peer >= peer_bytes.size()) { FAIL("peer slot %u out of range", b.peer); return; }
    if (!arenas && b.m_ld != b.cols) FAIL("message box with a row stride");
    if (arenas && (b.pad || b.msg_npad)) FAIL("refer box with padding");
    // the sub-chunks of tile t that its workgroups copy
    subs.clear();
    if (all) {
      for (uint32_t w = t * kSubPerTile; w < (t + 1) * kSubPerTile; ++w) subs.push_back(w % kSubPerTile);
    } else {
      for (uint32_t q : groups_of[t])
        for (uint32_t i = 0; i < kind_group(kes); ++i) subs.push_back(q * kind_group(kes) + i);
    }
    seen.assign(subs_per_tile, 0);
    for (uint32_t j : subs)
      if (j >= subs_per_tile || seen[j]++) FAIL("sub-chunk %u of tile %u copied twice or out of range", j, t);
    if (subs.size() != subs_per_tile) FAIL("tile %u: %zu sub-chunks copied, %u in the tile", t, subs.size(),
                                           subs_per_tile);
    const bool vectors = sub_vectors(b, g, 2) && sub_vectors(b, g, 4);  // all-kinds: the tile's every kind
    const uint32_t used = sub_used(g);
    for (int k = 0; k < 4; ++k) {
      if (!(kind_mask & (1u << k))) continue;
      const int es = k == 0 ? 2 : 4;
      if (!all && es != kes) FAIL("one-kind launch of another element size");
      const uint64_t sec = (sectioned && !arenas) ? section_byte(b.msg_npad, k) : 0;
      const uint64_t sec_end = arenas ? peer_bytes[k] : std::min(sec + b.msg_npad * es, peer_bytes[b.peer]);
      KindWalk w{tile_arena_elem(b, g) * es, sec + tile_msg_elem(b, g) * es, arena_elems * es, sec, sec_end,
                 uint64_t(b.a_ld) * es, b.m_ld * es, pack, es, k, writes};
      writes.clear();
      if (std::max(w.a_ld, w.m_ld) * (g.nr - 1) + uint64_t(g.nc) * es >= (1ull << 31)) FAIL("tile extent over 2^31");
      const bool vk = sub_vectors(b, g, es);
      const uint32_t group = all ? window_group(g.nc, es) : kind_window_group(g, es);
      if (!vk && g.nr > 1 && g.nr * windows_per_row(g.nc, es, group) > kTileElems / (16u / uint32_t(es)))
        FAIL("a tile of %u rows of %u elements has windows for a second pass", g.nr, g.nc);
      const uint32_t per = sub_elems / (16u / uint32_t(es));  // vectors or windows per sub-chunk
      // whether every row starts on a line on both sides
      const bool lines = ((w.a0 | w.m0 | (g.nr == 1 ? 0 : w.a_ld | w.m_ld)) % kLineBytes) == 0;
      bool padded = false;
      for (uint32_t j : subs) {
        if (j >= subs_per_tile) continue;
        uint32_t run = j;
        if (all && vectors) {
          if (!(b.vec & kLineBox)) run = xcd_run(j, (g.nr * g.nc + kSubElems - 1) / kSubElems);
          if ((b.vec & kLineBox) && es == 4 && !lines) FAIL("a box marked as on lines is not");
        } else if (all && !tile_few(g)) {
          if (j >= used) continue;
          if (!lines) run = xcd_run(j, used);
        } else if (all && j) {
          continue;
        }
        if (j == 0 && pack && g.last && b.pad && !(all && vectors)) padded = true;
        if (all && !vectors && tile_few(g)) walk_few(w, g);
        else if (vk) walk_vectors(w, g, per, run);
        else walk_windows(w, g, per, run, group);
      }
      if (pack && g.last && b.pad && !padded) FAIL("the padding after a box is not written");
      if (padded) {
        const uint64_t plo = sec + (b.m_off + uint64_t(b.rows) * b.cols) * es, phi = plo + uint64_t(b.pad) * es;
        if (phi > sec_end) FAIL("pad overrun");
        w.writes.push_back({plo, phi});
      }
      merge_tile(w.writes, "sub-chunk walk");
      for (auto x : w.writes) {
        if (pack) W[k][b.peer].push_back(x); else A[k].push_back(x);
      }
    }
  }
}

// Replay one launch.  peer_bytes[p] = length of peer p's message; W[k][p]
// collects message writes (pack), A[k] arena writes.
static void replay(const std::vector<CopyBox>& v, bool pack, bool sectioned, uint32_t kind_mask,
                   uint64_t arena_elems, const std::vector<uint64_t>& peer_bytes,
                   std::vector<std::vector<Iv>> W[4], std::vector<Iv> A[4], bool arenas = false) {
  if (v.back().tile0 == 0) return;
  if (kind_mask != 0xFu && (kind_mask == 0 || (kind_mask & (kind_mask - 1)))) {
    FAIL("a launch of more than one kind but not all four");
    return;
  }
  replay_sub(v, pack, sectioned, kind_mask, arena_elems, peer_bytes, W, A, arenas);
}

static void check_plan(etc_plan_t& P, const char* name) {
  const int S = P.src.world(), D = P.dst.world();
  for (int sectioned = 1; sectioned >= 0; --sectioned) {
    for (int s = 0; s < S; ++s) {
      std::vector<int32_t> peers; uint64_t bytes;
      auto v = build_pack_boxes(P, s, &peers, &bytes);
      for (int k = 0; k < 4; ++k) {
        const uint32_t mask = sectioned ? 0xFu : (1u << k);
        if (sectioned && k) break;
        std::vector<uint64_t> pb;
        for (int d : peers) pb.push_back(npad_of(P, s, d) * (sectioned ? 14 : (k ? 4 : 2)));
        std::vector<std::vector<Iv>> W[4]; std::vector<Iv> A[4];
        for (int kk = 0; kk < 4; ++kk) W[kk].assign(peers.size(), {});
        replay(v, true, sectioned, mask, P.src_lay(s).elems, pb, W, A);
        for (int kk = 0; kk < 4; ++kk) {
          if (!(mask & (1u << kk))) continue;
          const int es = kk ? 4 : 2;
          for (size_t i = 0; i < peers.size(); ++i) {
            const uint64_t npad = npad_of(P, s, peers[i]);
            const uint64_t b0 = sectioned ? section_byte(npad, kk) : 0;
            merge_equal(W[kk][i], {{b0, b0 + npad * es}}, std::string(name) + " pack s" + std::to_string(s) + " peer " + std::to_string(i));
          }
        }
      }
    }
    for (int d = 0; d < D; ++d) {
      std::vector<int32_t> peers; uint64_t bytes;
      auto v = build_unpack_boxes(P, d, &peers, &bytes);
      for (int k = 0; k < 4; ++k) {
        const uint32_t mask = sectioned ? 0xFu : (1u << k);
        if (sectioned && k) break;
        std::vector<uint64_t> pb;
        for (int s : peers) pb.push_back(npad_of(P, s, d) * (sectioned ? 14 : (k ? 4 : 2)));
        std::vector<std::vector<Iv>> W[4]; std::vector<Iv> A[4];
        replay(v, false, sectioned, mask, P.dst_lay(d).elems, pb, W, A);
        if (P.flags & ETC_PLAN_DIRECT_REFER) {  // Refer writes complete the target
          uint64_t rb = 0;
          auto rv = build_refer_boxes(P, d, &rb);
          const int h = P.home[d];
          if (h < 0 && rv.size() > 1) FAIL("refer boxes without a paired source");
          if (h >= 0) {
            const uint64_t se = P.src_lay(h).elems;
            std::vector<uint64_t> sb = {se * 2, se * 4, se * 4, se * 4};
            std::vector<std::vector<Iv>> RW[4];
            replay(rv, false, false, mask, P.dst_lay(d).elems, sb, RW, A, true);
          }
        }
        for (int kk = 0; kk < 4; ++kk) {
          if (!(mask & (1u << kk))) continue;
          const int es = kk ? 4 : 2;
          std::vector<Iv> want;
          for (auto& q : P.dst_lay(d).pieces) want.push_back({q.off * es, (q.off + q.elems()) * es});
          merge_equal(A[kk], want, std::string(name) + " unpack d" + std::to_string(d));
        }
      }
    }
  }
}


int main(int argc, char** argv) {
  if (argc < 19) {
    fprintf(stderr, "usage: tilewalk arch L h nh nkv ffn V max_pos tied flags tp pp dp tp pp dp refer pairing [failed...]\n");
    return 2;
  }
  etc_model_desc m{};
  int i = 1;
  m.arch = atoi(argv[i++]); m.num_layers = atoi(argv[i++]); m.hidden = atoi(argv[i++]);
  m.num_heads = atoi(argv[i++]); m.num_kv_heads = atoi(argv[i++]); m.ffn_hidden = atoi(argv[i++]);
  m.vocab = atoi(argv[i++]); m.max_pos = atoi(argv[i++]); m.tied_embeddings = atoi(argv[i++]);
  m.flags = atoi(argv[i++]);
  etc_parallel_cfg a{atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2])};
  etc_parallel_cfg b{atoi(argv[i + 3]), atoi(argv[i + 4]), atoi(argv[i + 5])};
  i += 6;
  const bool refer = atoi(argv[i++]) != 0;
  const std::string pairing = argv[i++];
  etc_plan_t P;
  P.model = m;
  P.src = Grid{a.tp, a.pp, a.dp};
  P.dst = Grid{b.tp, b.pp, b.dp};
  if (refer) P.flags |= ETC_PLAN_DIRECT_REFER;
  try {
    validate(m, a, b);
    const int S = P.src.world(), D = P.dst.world();
    std::vector<char> dead(S, 0);
    if (i < argc) {
      P.failed_bits.assign((S + 31) / 32, 0u);
      for (; i < argc; ++i) {
        const int f = atoi(argv[i]);
        dead[f] = 1;
        P.failed_bits[f >> 5] |= 1u << (f & 31);
      }
    }
    P.tensors = build_tensor_table(m);
    build_route_tensors(P);
    P.home.assign(D, -1);
    if (pairing == "sketch") {
      sketch_pairing(P, dead);
    } else if (pairing == "identity") {
      for (int d = 0; d < D && d < S; ++d)
        if (!dead[d] && P.src.replica(d) == P.dst.replica(d)) P.home[d] = d;
    } else {
      size_t pos = 0;
      for (int d = 0; d < D; ++d) {
        const size_t c = pairing.find(',', pos);
        P.home[d] = atoi(pairing.substr(pos, c == std::string::npos ? std::string::npos : c - pos).c_str());
        pos = c == std::string::npos ? pairing.size() : c + 1;
      }
    }
    build_host_plan(P);
    check_plan(P, "plan");
  } catch (PlanError& e) {
    fprintf(stderr, "plan error %d %s\n", e.code, e.what());
    return 1;
  }
  printf("%s\n", errors ? "ERRORS" : "ok");
  return errors ? 1 : 0;
}
