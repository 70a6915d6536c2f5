// Host check of plan_run's list teams (no GPU): every team has each rank once,
// its members post to consecutive slots that no other team has, sit in one
// column of the grid (an XCD), and the teams' first entries and the list are
// every instance once, largest first. Prints "ok".
#include <stdio.h>

#include <random>
#include <vector>

#include "../paper_1507_02087_amd/csrc/host_plan.h"

int main() {
  std::mt19937 g(2);
  const int edges[3][5] = {{2, 3, 4, 0, 0}, {2, 3, 4, 5, 0}, {2, 4, 0, 0, 0}};
  int bad = 0, lists = 0;
  for (int it = 0; it < 300; ++it) {
    const int prec = it % 3, count = 100 + g() % 1500;
    std::vector<sp2::RunInst> in(count);
    for (auto& i : in) {
      i.n = 1 + g() % 1024;
      i.trivial = g() % 9 == 0;
    }
    const std::vector<int> grids(4, 512);
    const sp2::RunPlan p = sp2::plan_run(in, prec, edges[prec], grids, 256);
    if (p.mb == 0 || p.pull.empty()) continue;
    ++lists;
    std::vector<std::vector<int>> ranks(p.teams);
    std::vector<int> slot(p.seats.size(), 0), column(p.teams, -1), seen(count, 0), first(p.teams, -1);
    for (size_t k = 0; k < p.seats.size(); ++k) {
      const sp2::RunSeat& s = p.seats[k];
      if (s.size == 0) continue;
      auto& r = ranks[s.team];
      r.resize(s.size, 0);
      if (s.rank < 0 || s.rank >= s.size || static_cast<int>(r.size()) != s.size ||
          s.base + s.rank >= static_cast<int>(slot.size())) {
        ++bad;
        continue;
      }
      r[s.rank]++;
      slot[s.base + s.rank]++;
      const int x = static_cast<int>(k % 8);
      if (column[s.team] >= 0 && column[s.team] != x) ++bad;
      column[s.team] = x;
      if (first[s.team] >= 0 && first[s.team] != s.inst) ++bad;
      first[s.team] = s.inst;
    }
    for (const auto& r : ranks) {
      if (r.empty()) ++bad;
      for (int c : r) bad += c != 1;
    }
    for (int c : slot) bad += c > 1;
    std::vector<int> order(first);
    order.insert(order.end(), p.pull.begin(), p.pull.end());
    for (size_t k = 0; k < order.size(); ++k) {
      seen[order[k]]++;
      auto key = [&](int b) { return in[b].trivial ? int64_t{0} : in[b].n; };
      if (k > 0 && key(order[k - 1]) < key(order[k])) ++bad;
    }
    for (int c : seen) bad += c != 1;
  }
  if (lists < 50) ++bad;
  if (!bad) printf("ok\n");
  else fprintf(stderr, "%d faults in %d lists\n", bad, lists);
  return bad != 0;
}
