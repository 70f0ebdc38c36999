// sketch.hip -- the migration sketch (Sec. III-B): pair the new ranks with the
// old ranks so the total cost is minimal (objective Eq. (2); constraints
// Eq. (3) when M > N, Eq. (4) when M <= N).  As in Algorithm 1 the M x N cost
// matrix is padded with zeros to k x k, the square assignment problem is
// solved, and pairs involving padding are dropped.  The square problem is
// solved with the Kuhn-Munkres (Hungarian) method in its shortest-augmenting-
// path form with row and column potentials: O(k^3), microseconds for the
// k <= 128 of a PP x TP grid.  While rows are added, 0 <= u[i] <= the largest
// entry (a free column has potential 0) and -(largest entry) <= v[j] <= 0, so
// sums stay below four times the largest entry: 64-bit where that fits, else
// 128-bit (a host-only plan with 2^59 bytes on a rank; etc_sketch takes entries
// up to 2^52).  Potentials change once per row added, not on every step of its tree.
// Two assignments of 64 x 32 entries, one core: about 700 us with 128-bit
// potentials updated on every step, 180 us this way.
#include <algorithm>
#include <cstdint>
#include <vector>

#include "plan.hpp"

namespace etc {

namespace {

template <typename Pot>
uint64_t solve(const uint64_t* cost, int M, int N, int32_t* pair) {
  const int k = std::max(M, N);
  auto c = [&](int i, int j) -> Pot {  // 1-based rows / columns, zero padding
    return (i <= M && j <= N) ? Pot(cost[size_t(i - 1) * N + (j - 1)]) : 0;
  };
  const Pot INF = Pot(1) << (sizeof(Pot) == 8 ? 62 : 100);
  std::vector<Pot> u(k + 1, 0), v(k + 1, 0), slack(k + 1), dist(k + 1);
  std::vector<int> row_of(k + 1, 0), prev(k + 1, 0);  // row_of[j]: row matched to column j
  std::vector<char> visited(k + 1);
  std::vector<int> tree;  // the columns visited for this row, in order
  for (int i = 1; i <= k; ++i) {
    // grow an alternating tree from free row i until it reaches a free column;
    // slack[j]: length of the shortest path to column j found so far, `len` and
    // dist[j]: of the path to the last column and to a visited column j
    row_of[0] = i;
    int j0 = 0;
    Pot len = 0;
    std::fill(slack.begin(), slack.end(), INF);
    std::fill(visited.begin(), visited.end(), 0);
    tree.clear();
    do {
      visited[j0] = 1;
      dist[j0] = len;
      tree.push_back(j0);
      const int i0 = row_of[j0];
      const Pot base = len - u[i0];
      Pot best = INF;
      int j1 = 0;
      for (int j = 1; j <= k; ++j) {
        if (visited[j]) continue;
        const Pot through = c(i0, j) + base - v[j];
        if (through < slack[j]) {
          slack[j] = through;
          prev[j] = j0;
        }
        if (slack[j] < best) {
          best = slack[j];
          j1 = j;
        }
      }
      len = best;
      j0 = j1;
    } while (row_of[j0] != 0);
    for (const int j : tree) {
      u[row_of[j]] += len - dist[j];
      v[j] -= len - dist[j];
    }
    // flip the augmenting path
    do {
      const int j1 = prev[j0];
      row_of[j0] = row_of[j1];
      j0 = j1;
    } while (j0 != 0);
    v[0] = 0;  // not a column
  }
  uint64_t total = 0;
  for (int i = 0; i < M; ++i) pair[i] = -1;
  for (int j = 1; j <= k; ++j) {
    const int i = row_of[j];
    if (i >= 1 && i <= M && j <= N) {
      pair[i - 1] = j - 1;
      total += cost[size_t(i - 1) * N + (j - 1)];
    }
  }
  return total;
}

}  // namespace

uint64_t solve_sketch(const uint64_t* cost, int M, int N, int32_t* pair) {
  uint64_t top = 0;
  for (size_t i = 0; i < size_t(M) * N; ++i) top = std::max(top, cost[i]);
  return top < uint64_t(1) << 59 ? solve<int64_t>(cost, M, N, pair) : solve<__int128>(cost, M, N, pair);
}

}  // namespace etc
