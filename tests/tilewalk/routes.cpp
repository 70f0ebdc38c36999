// routes.cpp -- the planner's sender lists in LCM slices against the routing
// rule, written out here on its own and asked tensor by tensor, its closed-form
// COST against sums over the tensors, the cost kernel's tables against the
// tensors, and the sketch in 64-bit against 128-bit whole numbers, on seeded
// configurations: tied and untied, uneven TP and PP degrees, replicas,
// failed ranks, pairings of every sort.  Prints "ok".  Test code.
#include <algorithm>
#include <cstdio>
#include <random>
#include <tuple>
#include <vector>
#include "etc_internal.hpp"
#include "plan.hpp"
#include "route.hpp"
using namespace etc;

static int errors = 0;
static void expect(bool ok, const char* what, int it) {
  if (!ok && errors++ < 20) printf("configuration %d: %s\n", it, what);
}

// The range of its split dim that a rank with TP rank tp of TP holds of t.
static Span shard_span(const RouteTensor& t, int tp, int TP) {
  if (t.split == kRepl) return Span{0, 1};
  const int64_t w = split_extent(t) / TP;
  return Span{tp * w, (tp + 1) * w};
}

// The copy role in which a stage holds a tensor, or -1.
static int role_of(const int32_t stage[2], int pp) { return stage[0] == pp ? 0 : stage[1] == pp ? 1 : -1; }

// The source that the rule names for the part of t that target d shares with
// source s's shard, or -1: the paired source where it holds that part; else the
// live holder, in the first replica from the serving one on that has any, of d's
// own copy role, of the TP rank congruent to d's, of the lowest stage, of the
// lowest TP rank, in this order.
static int sender(const etc_plan_t& P, const std::vector<char>& dead, const RouteTensor& t, int s, int d) {
  const int Sr = P.src.replica_size(), home = P.home[d];
  const auto holds = [&](int x) {
    return !dead[x] && role_of(t.src_stage, P.src.pp_of(x)) >= 0 &&
           (t.split == kRepl || P.src.tp_of(x) == P.src.tp_of(s));
  };
  if (home >= 0 && holds(home)) return home;
  const int role_d = role_of(t.dst_stage, P.dst.pp_of(d));
  for (int i = 0; i < P.src.dp; ++i) {
    const int rep = (P.dst.replica(d) + i) % P.src.dp;
    std::vector<std::tuple<bool, bool, int, int, int>> live;
    for (int x = rep * Sr; x < (rep + 1) * Sr; ++x)
      if (holds(x))
        live.emplace_back(role_of(t.src_stage, P.src.pp_of(x)) != role_d,
                          P.src.tp_of(x) != P.dst.tp_of(d) % P.src.tp, P.src.pp_of(x), P.src.tp_of(x), x);
    if (!live.empty()) return std::get<4>(*std::min_element(live.begin(), live.end()));
  }
  return -1;
}

// The range of t's split dim that source s sends to target d.
static Span routed(const etc_plan_t& P, const std::vector<char>& dead, const RouteTensor& t, int s, int d) {
  if (role_of(t.dst_stage, P.dst.pp_of(d)) < 0 || role_of(t.src_stage, P.src.pp_of(s)) < 0 || dead[s])
    return Span{0, 0};
  const Span need = shard_span(t, P.dst.tp_of(d), P.dst.tp), have = shard_span(t, P.src.tp_of(s), P.src.tp);
  const Span x{std::max(have.lo, need.lo), std::min(have.hi, need.hi)};
  return x.len() && sender(P, dead, t, s, d) == s ? x : Span{0, 0};
}

int main() {
  std::mt19937 rng(11);
  auto pick = [&](std::initializer_list<int> v) { return *(v.begin() + rng() % v.size()); };
  int planned = 0;
  for (int it = 0; it < 300; ++it) {
    etc_plan_t P;
    P.model = {};
    P.model.arch = pick({ETC_ARCH_GPT, ETC_ARCH_LLAMA});
    P.model.num_layers = 12;
    P.model.hidden = 12 * pick({1, 2, 5});
    P.model.num_heads = P.model.num_kv_heads = 12;
    P.model.ffn_hidden = 12 * pick({3, 7});
    P.model.vocab = 12 * pick({1, 5});
    P.model.max_pos = pick({0, 9});
    P.model.tied_embeddings = pick({0, 1});
    P.src = Grid{pick({1, 2, 3, 4, 6}), pick({1, 2, 3, 4}), pick({1, 1, 2, 3})};
    P.dst = Grid{pick({1, 2, 3, 4, 6}), pick({1, 2, 3, 4}), pick({1, 1, 2, 4})};
    const int S = P.src.world(), D = P.dst.world();
    if (pick({0, 1})) P.flags |= ETC_PLAN_DIRECT_REFER;
    std::vector<char> dead(S, 0);
    for (int n = P.src.dp > 1 ? pick({0, 0, 1, 3}) : 0; n > 0; --n) dead[rng() % S] = 1;
    if (std::count(dead.begin(), dead.end(), 1)) {
      P.failed_bits.assign((S + 31) / 32, 0u);
      for (int s = 0; s < S; ++s)
        if (dead[s]) P.failed_bits[s >> 5] |= 1u << (s & 31);
    }
    P.tensors = build_tensor_table(P.model);
    build_route_tensors(P);
    P.home.assign(D, -1);
    if (pick({0, 1})) {
      sketch_pairing(P, dead);
    } else {  // live old ranks on any new ranks
      std::vector<int> live;
      for (int s = 0; s < S; ++s)
        if (!dead[s]) live.push_back(s);
      std::shuffle(live.begin(), live.end(), rng);
      for (int d = 0; d < D && !live.empty(); ++d)
        if (pick({0, 1, 1})) P.home[d] = live.back(), live.pop_back();
    }
    // COST, tensor by tensor
    const int Sr = P.src.replica_size(), Dr = P.dst.replica_size();
    const std::vector<uint64_t> cost = host_replica_cost(P);
    for (int d = 0; d < Dr; ++d)
      for (int s = 0; s < Sr; ++s) {
        uint64_t need = 0, ov = 0;
        for (const RouteTensor& t : P.route_tensors) {
          if (role_of(t.dst_stage, P.dst.pp_of(d)) < 0) continue;
          const Span want = shard_span(t, P.dst.tp_of(d), P.dst.tp), have = shard_span(t, P.src.tp_of(s), P.src.tp);
          need += uint64_t(want.len() * unit_elems(t));
          if (role_of(t.src_stage, P.src.pp_of(s)) < 0) continue;
          ov += uint64_t(Span{std::max(have.lo, want.lo), std::min(have.hi, want.hi)}.len() * unit_elems(t));
        }
        expect(cost[size_t(d) * Sr + s] == (need - ov) * 14, "COST differs from the sum over the tensors", it);
      }
    // the cost kernel's tables: a pair lists each of its groups once and no
    // other, and they fit the room that static plans count for them
    const CostTable table = build_cost_table(P);
    expect(table.bytes() <= P.route_tensors.size() * sizeof(RouteTensor), "the cost tables need more room", it);
    for (int pd = 0; pd < P.dst.pp; ++pd)
      for (int ps = 0; ps < P.src.pp; ++ps) {
        const CostStage& st = table.stages[pd];
        const uint32_t at = uint32_t(ps - st.lo);
        const CostPair p = at < st.n ? table.pairs[st.first + at] : CostPair{};
        uint64_t held = 0, held1 = 0, listed = 0;  // elements per LCM slice, or of a whole tensor
        for (const RouteTensor& t : P.route_tensors) {
          if (role_of(t.dst_stage, pd) < 0 || role_of(t.src_stage, ps) < 0) continue;
          const uint64_t n = uint64_t(unit_elems(t)) *
                             (t.split == kRepl ? 1 : split_extent(t) / (lcm_slices(P).src * P.src.tp));
          held += n;
          held1 += t.single_copy ? n : 0;
        }
        for (uint32_t i = p.first; i < p.end; ++i) {
          const CostGroup& g = table.groups[i];
          listed += g.slice + g.whole;
          expect(role_of(g.src_stage, ps) >= 0, "a group of another source stage", it);
          for (uint32_t k = p.first; k < i; ++k)
            expect(g.role_d != table.groups[k].role_d || g.src_stage[0] != table.groups[k].src_stage[0] ||
                       g.src_stage[1] != table.groups[k].src_stage[1], "a group listed twice", it);
        }
        expect(p.end - p.first <= 3 && listed == held, "a pair's groups are not its tensors", it);
        expect(p.slice + p.whole == held && p.slice1 + p.whole1 == held1, "a pair's sums are not its tensors", it);
      }
    {  // the same matrix 2^k times over: past 2^59 the sketch works in 128 bits
      std::vector<uint64_t> big = cost;
      const uint64_t top = *std::max_element(cost.begin(), cost.end());
      int k = 0;
      while (top && (top << k) < (uint64_t(1) << 60)) ++k;
      for (uint64_t& x : big) x <<= k;
      std::vector<int32_t> a(Dr), b(Dr);
      const uint64_t ta = solve_sketch(cost.data(), Dr, Sr, a.data());
      const uint64_t tb = solve_sketch(big.data(), Dr, Sr, b.data());
      expect(a == b && (ta << k) == tb, "64-bit and 128-bit sketches differ", it);
    }
    bool recoverable = true;
    try {
      build_host_plan(P);
    } catch (const PlanError& e) {
      recoverable = false;
      expect(e.code == ETC_ERR_UNRECOVERABLE, e.what(), it);
    }
    planned += recoverable;
    // every box, in the order of d's arena and of the sources
    bool whole = true;
    for (int d = 0; d < D; ++d) {
      std::vector<size_t> at(S, 0);
      size_t kept = 0;
      const RankLayout L = build_layout(P.tensors, P.route_tensors, true, P.dst, d % Dr);
      for (const Piece& q : L.pieces) {
        const RouteTensor& t = P.route_tensors[q.tensor];
        uint64_t got = 0;
        for (int s = 0; s < S; ++s) {
          const Span x = routed(P, dead, t, s, d);
          got += uint64_t(x.len() * unit_elems(t));
          if (x.len() == 0 || !recoverable) continue;
          const bool keep = (P.flags & ETC_PLAN_DIRECT_REFER) && s == P.home[d];
          const auto* m = P.find_msg(s, d);
          const auto* boxes = keep ? &P.refer[d] : m ? &m->boxes : nullptr;
          size_t& i = keep ? kept : at[s];
          if (!boxes || i >= boxes->size()) {
            expect(false, "a box is missing", it);
            continue;
          }
          const auto& b = (*boxes)[i++];
          const bool rows = t.split == kRows, cols = t.split == kCols;
          expect(b.tensor == q.tensor && b.role_d == q.role && b.r0 == (rows ? x.lo : 0) &&
                     b.r1 == (rows ? x.hi : t.rows) && b.c0 == (cols ? x.lo : 0) && b.c1 == (cols ? x.hi : t.cols),
                 "a box differs from the rule", it);
        }
        whole = whole && got == q.elems();
      }
      for (int s = 0; recoverable && s < S; ++s) {
        const auto* m = P.find_msg(s, d);
        expect(at[s] == (m ? m->boxes.size() : 0), "a box too many", it);
      }
      if (recoverable) expect(kept == P.refer[d].size(), "a kept box too many", it);
    }
    expect(whole == recoverable, "the planner and the rule differ on what can be recovered", it);
  }
  expect(planned > 200, "too few of the configurations can be planned", -1);
  if (!errors) printf("ok\n");
  return errors != 0;
}
