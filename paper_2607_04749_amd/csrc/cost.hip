// cost.hip -- byte-overlap / routing / cost matrices over every (source,
// target) rank pair, on the GPU (Sec. III-B cost matrix, Sec. III-C LCM
// workload items).  In LCM slices a pair of shards overlaps alike in every
// split tensor, so a cell needs only the tensors' summed sizes per pair of
// stages (CostPair) and one product; ROUTE asks who sends for each of the
// pair's CostGroups, one or two.  Cells that the rules make empty or infinite
// (most of a data-parallel job's) read none.
// COST is ETC_COST_INF between ranks of different data-parallel replicas and
// towards failed ranks (Sec. III-C); a failed rank holds and sends nothing.
//
// Integer work on a few hundred bytes of tables: launch latency for a single
// replica's ranks.  For 1024 x 768 cells the integer divisions that turn ranks
// into grid coordinates took longest, so a workgroup covers a tile of the
// matrix: a thread stays in one column and the rows' coordinates are worked
// out once per workgroup.  Llama-70B, MI355X, kernel time, against two
// wavefronts per cell that looped over the 563 tensors:
//   64 x 32 cells       COST 2.8 us, ROUTE 4.2 us    (6.6 to 8.5 us)
//   1024 x 768 cells    COST 4.5 us, ROUTE 7.6 us, 10.9 us where a node of
//                       8 ranks was lost             (1030 to 1360 us)
// A cell that loops over all groups of its target stage is no way out where
// many source stages become one: 80 stages to 1, COST + ROUTE took 54.8 us
// like that, 10.1 with the loop over the tensors, and take 5.3 as it is.
// With ranks lost, a ROUTE cell asks only where its source's replica can stand
// in (`reach`): COST + ROUTE took 13.7 us a pass, 14.1 while every replica's
// cells asked.  The rest of those 10.9 us is one chain per cell: the groups one
// after another, each with the holders' failed bits to read.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "etc_internal.hpp"
#include "route.hpp"

namespace etc {

namespace {

constexpr int kCmThreads = 256;
constexpr int kCmRows = 32;    // rows of a workgroup's tile, at most

// A workgroup's tile: 1 << wbits columns by `rows` rows, kCmThreads >> wbits
// of them at a time.
struct CostTile {
  uint32_t wbits, rows, across;  // across: tiles side by side
};

// Whether a rank of [lo, lo + n) failed.
__device__ inline bool any_dead(const RouteCtx& c, int lo, int n) {
  if (c.failed == nullptr) return false;
  const int hi = lo + n;
  uint32_t found = 0;
  for (int w = lo >> 5; w <= (hi - 1) >> 5; ++w) {
    uint32_t bits = c.failed[w];
    if (w == lo >> 5) bits &= ~0u << (lo & 31);
    if (w == (hi - 1) >> 5) bits &= ~0u >> (31 - ((hi - 1) & 31));
    found |= bits;
  }
  return found != 0;
}

template <int kWhich>
__global__ __launch_bounds__(kCmThreads) void cost_kernel(CostView v, const int32_t* __restrict__ home, RouteCtx c,
                                                          LcmSlices lcm, CostTile tile, uint64_t* __restrict__ out) {
  constexpr bool kCost = kWhich == ETC_CM_COST;  // rows are targets; sources otherwise
  __shared__ SourceAt row_src[kCmRows];
  __shared__ TargetAt row_dst[kCmRows];
  __shared__ CostStage row_stage[kCmRows];
  const int S = c.tps * c.pps * c.dps, D = c.tpd * c.ppd * c.dpd;
  const uint32_t nrow = uint32_t(kCost ? D : S), ncol = uint32_t(kCost ? S : D);
  const uint32_t band = blockIdx.x / tile.across, row0 = band * tile.rows;
  const uint32_t col = ((blockIdx.x - band * tile.across) << tile.wbits) + (threadIdx.x & ((1u << tile.wbits) - 1));
  const uint32_t sub = threadIdx.x >> tile.wbits, step = kCmThreads >> tile.wbits;
  const int mine = int(col < ncol ? col : 0);
  // the column's coordinates stay in registers, the rows' in LDS
  SourceAt a{};
  TargetAt b{};
  CostStage st{};
  int reach = 0;  // ROUTE: the last replica, counted from the serving one, that may send to the target
  if (kCost) {
    a = source_at(mine, c);
    if (threadIdx.x < tile.rows && row0 + threadIdx.x < nrow) {
      const TargetAt t = target_at(int(row0 + threadIdx.x), -1, c);
      row_dst[threadIdx.x] = t;
      row_stage[threadIdx.x] = v.stages[t.pp];
    }
  } else {
    b = target_at(mine, kWhich == ETC_CM_ROUTE ? home[mine] : -1, c);
    st = v.stages[b.pp];
    if (kWhich == ETC_CM_ROUTE)
      for (int rep = b.rep0, n = c.tps * c.pps; reach + 1 < c.dps && any_dead(c, rep * n, n); ++reach)
        rep = rep + 1 == c.dps ? 0 : rep + 1;
    if (threadIdx.x < tile.rows && row0 + threadIdx.x < nrow)
      row_src[threadIdx.x] = source_at(int(row0 + threadIdx.x), c);
  }
  __syncthreads();
  for (uint32_t r = sub; r < tile.rows; r += step) {
    const uint32_t row = row0 + r;
    if (row >= nrow || col >= ncol) break;
    if (kCost) b = row_dst[r], st = row_stage[r];
    else a = row_src[r];
    bool held = !a.dead;  // whether the source may hold or send anything for the target
    if (kCost) held = held && a.rep == b.rep;
    if (kWhich == ETC_CM_OVERLAP_SHARDED) held = held && a.rep == b.rep0;
    // a replica beyond the serving one stands in only where that one and all between them lost ranks
    if (kWhich == ETC_CM_ROUTE)
      held = held && (a.s == b.home || (a.rep < b.rep0 ? a.rep - b.rep0 + c.dps : a.rep - b.rep0) <= reach);
    // elements of a slice / of whole tensors, moved or shared
    uint64_t slice = 0, whole = 0;
    const uint32_t at = uint32_t(a.pp - st.lo);
    if (held && at < st.n) {
      const CostPair& p = v.pairs[st.first + at];
      if (kWhich == ETC_CM_ROUTE) {
        for (uint32_t i = p.first; i < p.end; ++i) {
          const CostGroup& g = v.groups[i];
          if (sends_shard(a, b, g.src_stage, false, g.role_d, c)) slice += g.slice;
          if (sends_shard(a, b, g.src_stage, true, g.role_d, c)) whole += g.whole;
        }
      } else {
        slice = kWhich == ETC_CM_OVERLAP_SHARDED ? p.slice1 : p.slice;
        whole = kWhich == ETC_CM_OVERLAP_SHARDED ? p.whole1 : p.whole;
      }
    }
    const int64_t s0 = a.tp * lcm.src, d0 = b.tp * lcm.dst;  // first LCM slice of each shard
    const Span x{s0 > d0 ? s0 : d0, s0 + lcm.src < d0 + lcm.dst ? s0 + lcm.src : d0 + lcm.dst};
    constexpr uint64_t kBytesPerElem = 14;  // 2 (bf16) + 4 + 4 + 4 (fp32)
    uint64_t bytes = (uint64_t(x.len()) * slice + whole) * kBytesPerElem;
    if (kCost)
      bytes = held ? (uint64_t(lcm.dst) * st.slice + st.whole) * kBytesPerElem - bytes : uint64_t(ETC_COST_INF);
    out[size_t(row) * ncol + col] = bytes;
  }
}

}  // namespace

hipError_t launch_cost(const CostView& tables, const int32_t* home, RouteCtx ctx, LcmSlices lcm, int which,
                       uint64_t* out, hipStream_t stream) {
  const uint32_t S = uint32_t(ctx.tps * ctx.pps * ctx.dps), D = uint32_t(ctx.tpd * ctx.ppd * ctx.dpd);
  const uint32_t nrow = which == ETC_CM_COST ? D : S, ncol = which == ETC_CM_COST ? S : D;
  CostTile tile{0, 0, 0};
  while (tile.wbits < 8 && (1u << tile.wbits) < ncol) ++tile.wbits;
  tile.across = (ncol + (1u << tile.wbits) - 1) >> tile.wbits;
  // One pass of rows per workgroup, more only while 1024 workgroups are left:
  // rows of a thread follow each other.  One row per thread / this rule / the
  // same with 512 workgroups, in us, COST and ROUTE (graph replays):
  //   1024 x 768 cells    5.2 / 4.0 / 4.1      7.5 / 6.9 / 8.8
  //   1536 x 1280         9.8 / 6.3 / 6.7     15.3 / 12.4 / 15.7
  //   2048 x 2048        17.2 / 10.8 / 15.7   29.2 / 27.6 / 45.9
  //   4096 x 4096        56.5 / 28.3 / 28.4  111.2 / 69.6 / 69.5
  // Only ROUTE with a node lost is faster with one row at some sizes (1024 x 768:
  // 8.4 / 8.8 / 12.3, 2048 x 2048: 32.8 / 39.4 / 58.5).
  const uint32_t pass = std::min<uint32_t>(kCmThreads >> tile.wbits, kCmRows);
  tile.rows = pass;
  while (tile.rows * 2 <= kCmRows && uint64_t((nrow + 2 * tile.rows - 1) / (2 * tile.rows)) * tile.across >= 1024)
    tile.rows *= 2;
  const dim3 grid((nrow + tile.rows - 1) / tile.rows * tile.across), block(kCmThreads);
#define ETC_COST(W) \
  hipLaunchKernelGGL(cost_kernel<W>, grid, block, 0, stream, tables, home, ctx, lcm, tile, out)
  switch (which) {
    case ETC_CM_ROUTE: ETC_COST(ETC_CM_ROUTE); break;
    case ETC_CM_OVERLAP: ETC_COST(ETC_CM_OVERLAP); break;
    case ETC_CM_OVERLAP_SHARDED: ETC_COST(ETC_CM_OVERLAP_SHARDED); break;
    default: ETC_COST(ETC_CM_COST); break;
  }
#undef ETC_COST
  return hipGetLastError();
}

}  // namespace etc
