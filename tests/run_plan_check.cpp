// Host check of plan_run (no GPU): on random instances and batches, every
// team has each rank once, posts to slots of its own, fits the device, and
// the tiles its seats take (whole rounds and the last one) cover the upper
// triangle exactly once. Prints "ok" and returns 0 when every check holds.
#include <stdio.h>

#include <random>
#include <vector>

#include "../paper_1507_02087_amd/csrc/host_plan.h"

int main() {
  std::mt19937 g(1);
  const int edges[3][5] = {{2, 3, 4, 0, 0}, {2, 3, 4, 5, 0}, {2, 4, 0, 0, 0}};
  int bad = 0, planned = 0;
  for (int it = 0; it < 2000; ++it) {
    const int prec = g() % 3;
    const int count = it < 700 ? 1 : 1 + g() % (it % 2 ? 20 : 900);
    const int cus = (it % 7 == 0) ? 32 : 256;
    std::vector<sp2::RunInst> in(count);
    for (auto& i : in) {
      i.n = 1 + g() % (count == 1 ? 5000 : 1024);
      i.trivial = g() % 9 == 0;
    }
    std::vector<int> grids;
    for (int q = 0; edges[prec][q]; ++q) grids.push_back(cus * (1 + g() % 3));
    const sp2::RunPlan p = sp2::plan_run(in, prec, edges[prec], grids, cus);
    if (!p.mb) continue;
    ++planned;
    auto fail = [&](const char* what) {
      if (bad++ < 10) fprintf(stderr, "%s: case %d, %d instances\n", what, it, count);
    };
    int cap = 0;
    for (int q = 0; edges[prec][q]; ++q)
      if (edges[prec][q] == p.mb) cap = grids[q];
    if (static_cast<int>(p.seats.size()) > cap) fail("grid over the device");
    if (!p.pull.empty()) {
      // equal teams: every rank of every team once, first entries and list
      // together every instance once
      std::vector<int> seen(count, 0), slot(p.seats.size(), 0);
      std::vector<int> members(p.teams, 0), first(p.teams, -1);
      for (const sp2::RunSeat& s : p.seats) {
        if (s.size == 0) continue;
        if (s.team < 0 || s.team >= p.teams || s.rank < 0 || s.rank >= s.size ||
            s.base + s.rank >= static_cast<int>(p.seats.size()) || s.inst < 0 ||
            s.inst >= count || (first[s.team] >= 0 && first[s.team] != s.inst)) {
          fail("list seat");
          continue;
        }
        first[s.team] = s.inst;
        members[s.team] += 1 << s.rank % 30;
        slot[s.base + s.rank]++;
        if (s.rank == 0) seen[s.inst]++;
      }
      for (int c : slot)
        if (c > 1) fail("list slot");
      for (int t = 0; t < p.teams; ++t)
        if (first[t] < 0 || members[t] == 0) fail("empty team");
      for (int32_t b : p.pull) seen[b]++;
      for (int c : seen)
        if (c != 1) fail("list");
      continue;
    }
    std::vector<std::vector<int>> ranks(count), hit(count);
    std::vector<int> size(count, 0), ntile(count), slot(p.seats.size(), 0);
    for (int b = 0; b < count; ++b) {
      const int nt = static_cast<int>((in[b].n + 16 * p.mb - 1) / (16 * p.mb));
      ntile[b] = in[b].trivial ? 0 : nt * (nt + 1) / 2;
      hit[b].assign(ntile[b], 0);
    }
    for (const sp2::RunSeat& s : p.seats) {
      if (s.size == 0) continue;
      if (s.inst < 0 || s.inst >= count || s.rank < 0 || s.rank >= s.size ||
          s.base + s.rank >= static_cast<int>(p.seats.size()) ||
          (size[s.inst] && size[s.inst] != s.size)) {
        fail("seat");
        continue;
      }
      size[s.inst] = s.size;
      ranks[s.inst].resize(s.size, 0);
      ranks[s.inst][s.rank]++;
      slot[s.base + s.rank]++;
      // the kernel's walk over its tiles
      const int n = ntile[s.inst], whole = n / s.size * s.size;
      auto next = [&](int t) {
        return t + s.size < whole ? t + s.size : (t < whole ? s.last : n);
      };
      for (int t = whole > 0 ? s.rank : s.last; t < n; t = next(t)) hit[s.inst][t]++;
    }
    for (int c : slot)
      if (c > 1) fail("slot shared");
    for (int b = 0; b < count; ++b) {
      if (size[b] == 0) fail("no team");
      for (int r : ranks[b])
        if (r != 1) fail("rank");
      for (int h : hit[b])
        if (h != 1) fail("tile");
    }
  }
  if (planned < 500) ++bad;
  if (!bad) printf("ok\n");
  return bad != 0;
}
