// route.hpp -- which source rank sends which part of a tensor to which target
// rank.  Used by the host planner (boxes, message layouts) and by the cost
// matrix kernel (byte counts), so both sides see one definition.
//
// A tensor's TP shards are ranges of its split dim: shard tp of TP covers
// [tp*E/TP, (tp+1)*E/TP) where E is the split dim's extent; a replicated
// tensor is the single range [0, 1) of "whole tensor" units.  Because every
// split is even, two shards of the same TP are equal or disjoint, and the
// intersection of a source shard with a target shard is one range (a whole
// number of LCM(TP_src, TP_dst) slices, Sec. III-C).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "etc_internal.hpp"

namespace etc {

struct Span {
  int64_t lo, hi;
  __host__ __device__ int64_t len() const { return hi > lo ? hi - lo : 0; }
};

__host__ __device__ inline int64_t split_extent(const RouteTensor& t) {
  return t.split == kRows ? t.rows : t.split == kCols ? t.cols : 1;
}

// elements per unit of the split-dim range
__host__ __device__ inline int64_t unit_elems(const RouteTensor& t) {
  return t.split == kRows ? t.cols : t.split == kCols ? t.rows : t.rows * t.cols;
}

// copy role of the tensor held on stage pp (a stage holds at most one role)
__host__ __device__ inline int role_on(const int32_t stage[2], int pp) {
  return stage[0] == pp ? 0 : (stage[1] == pp ? 1 : -1);
}

// Lexicographic key of a candidate sender: prefer the target's own copy role,
// then the TP rank congruent to the target's, then lower stage, lower TP rank.
__host__ __device__ inline bool key_less(int role, int tp, int pp, int best_role, int best_tp,
                                         int best_pp, int role_d, int tpd_mod) {
  const int a0 = role != role_d, b0 = best_role != role_d;
  if (a0 != b0) return a0 < b0;
  const int a1 = tp != tpd_mod, b1 = best_tp != tpd_mod;
  if (a1 != b1) return a1 < b1;
  if (pp != best_pp) return pp < best_pp;
  return tp < best_tp;
}

__host__ __device__ inline bool rank_dead(const RouteCtx& c, int s) {
  return c.failed != nullptr && ((c.failed[s >> 5] >> (s & 31)) & 1u);
}

// Grid coordinates of a source rank.
struct SourceAt {
  int s, pp, tp, rep;
  bool dead;  // failed: it holds and sends nothing
};
__host__ __device__ inline SourceAt source_at(int s, const RouteCtx& c) {
  const int pt = c.tps * c.pps, rep = s / pt, r = s - rep * pt, pp = r / c.tps;
  return SourceAt{s, pp, r - pp * c.tps, rep, rank_dead(c, s)};
}

// Grid coordinates of a target rank, and of home, the source rank paired with
// it in the migration sketch (the same GPU), or -1.
struct TargetAt {
  int pp, tp, rep;
  int rep0;              // source replica that serves d's replica
  int tp_mod;            // tp mod TP_src
  int home, pp_h, tp_h;  // pp_h = -2, no stage, without a home
};
__host__ __device__ inline TargetAt target_at(int d, int home, const RouteCtx& c) {
  const int pt = c.tpd * c.ppd, rep = d / pt, r = d - rep * pt, pp = r / c.tpd, tp = r - pp * c.tpd;
  TargetAt t{pp, tp, rep, rep % c.dps, tp % c.tps, home, -2, 0};
  if (home >= 0) {
    t.pp_h = home / c.tps % c.pps;
    t.tp_h = home % c.tps;
  }
  return t;
}

// Whether live source a, which holds a tensor's shard (the whole tensor if
// `repl`), is the one that sends what target b needs of it.  src_stage: the stages
// of the tensor's copy roles in the source grid; role_d: the copy role that b
// holds.  Rules (Sec. III-D, Sec. III-C):
//  - data the paired source already holds stays with it (Refer);
//  - otherwise target replica j is served by source replica j mod DP_src (kept
//    replicas stay, scale-out replicas are fed round-robin), and within it by
//    the live holder with the smallest key_less key;
//  - if no live rank of that replica holds the data, the next replicas in
//    order stand in (fault tolerance through DP replicas).
// Data with no live holder is routed nowhere; the planner reports it as
// unrecoverable.
__host__ __device__ inline bool sends_shard(const SourceAt& a, const TargetAt& b, const int32_t src_stage[2],
                                            bool repl, int role_d, const RouteCtx& c) {
  if (a.s == b.home) return true;
  // does the paired source hold this shard?  Then it keeps it.
  if (role_on(src_stage, b.pp_h) >= 0 && (repl || b.tp_h == a.tp)) return false;
  // Holders of the shard in a replica: per copy role, the rank on that role's
  // stage (any TP rank for a replicated tensor); the first replica in serving
  // order with a live holder decides.
  const int pt = c.tps * c.pps;
  for (int step = 0, rep = b.rep0; step < c.dps; ++step, rep = rep + 1 == c.dps ? 0 : rep + 1) {
    // the holder with the smallest possible key, when it is alive
    const int pref = rep * pt + (src_stage[role_d] >= 0 ? src_stage[role_d] : src_stage[1 - role_d]) * c.tps +
                     (repl ? b.tp_mod : a.tp);
    if (!rank_dead(c, pref)) return pref == a.s;
    int best_role = -1, best_tp = 0, best_pp = 0;
    for (int r = 0; r < 2; ++r) {
      const int st = src_stage[r];
      if (st < 0) continue;
      const int tp_lo = repl ? 0 : a.tp;
      const int tp_hi = repl ? c.tps : a.tp + 1;
      for (int tp = tp_lo; tp < tp_hi; ++tp) {
        if (rank_dead(c, rep * pt + st * c.tps + tp)) continue;
        if (best_role < 0 || key_less(r, tp, st, best_role, best_tp, best_pp, role_d, b.tp_mod)) {
          best_role = r;
          best_tp = tp;
          best_pp = st;
        }
      }
    }
    if (best_role >= 0) return rep * pt + best_pp * c.tps + best_tp == a.s;
  }
  return false;
}

}  // namespace etc
