// Host check of resident_batch_pays on batches that were timed with both
// drivers (a step, resident over other): a batch more than 5 % slower goes to
// the other one, one more than 15 % faster does not. Prints "ok" and returns 0
// when every check holds.
#include <stdio.h>

#include <random>
#include <vector>

#include "../paper_1507_02087_amd/csrc/host_plan.h"

namespace {

struct Timed {
  int precision;
  bool mcweeny;
  int count;
  int64_t lo, hi;
  double ratio;
};
const Timed kTimed[] = {
    // BF16x3
    {2, false, 8, 3500, 3500, 1.75}, {2, false, 4, 3500, 3500, 1.39}, {2, false, 3, 3000, 3000, 1.09},
    {2, false, 4, 2500, 2500, 1.12}, {2, false, 8, 2000, 2000, 1.47}, {2, false, 128, 1000, 1000, 1.31},
    {2, false, 1024, 1000, 1000, 1.79}, {2, false, 16, 500, 3000, 1.59}, {2, false, 12, 1000, 2000, 1.09},
    {2, false, 2, 2500, 2500, 0.77}, {2, false, 3, 2000, 2000, 0.80}, {2, false, 6, 1500, 1500, 0.81},
    {2, false, 64, 500, 500, 0.69}, {2, false, 2048, 300, 300, 0.51}, {2, false, 200, 60, 800, 0.73},
    {2, false, 256, 64, 1024, 0.80}, {2, false, 1500, 100, 400, 0.56}, {2, true, 4, 2500, 2500, 1.16},
    {2, true, 8, 1250, 1250, 1.20}, {2, true, 64, 750, 750, 1.18}, {2, true, 1024, 200, 200, 1.06},
    {2, true, 3, 2000, 2000, 1.19}, {2, true, 2, 1500, 1500, 0.69}, {2, true, 32, 750, 750, 0.80},
    {2, true, 256, 200, 200, 0.61}, {2, true, 2048, 100, 100, 0.75},
    // FP32
    {1, false, 3, 6000, 6000, 1.20}, {1, false, 8, 4000, 4000, 1.11}, {1, false, 6, 2500, 2500, 1.08},
    {1, false, 512, 1000, 1000, 1.08}, {1, false, 2, 3500, 3500, 0.84}, {1, false, 3, 2000, 2000, 0.78},
    {1, false, 512, 64, 1024, 0.84}, {1, false, 2048, 300, 300, 0.54}, {1, false, 96, 20, 200, 0.31},
    {1, true, 4, 2000, 2000, 1.16}, {1, true, 8, 4000, 4000, 1.19}, {1, true, 512, 1000, 1000, 1.11},
    {1, true, 3, 700, 700, 0.52}, {1, true, 512, 64, 1024, 0.80}, {1, true, 32, 400, 400, 0.56},
    // FP64
    {0, false, 8, 3500, 3500, 1.17}, {0, false, 3, 5000, 5000, 1.09}, 
    {0, false, 4, 2000, 2000, 1.08}, {0, false, 64, 1000, 1000, 1.09}, {0, false, 32, 700, 700, 1.14},
    {0, false, 64, 1500, 1500, 1.14},
    {0, false, 256, 64, 1024, 0.74}, {2, false, 1, 3400, 3400, 0.70}, {0, false, 2, 3000, 3000, 0.84}, {0, false, 4, 1500, 1500, 0.55},
    {0, false, 512, 64, 1024, 0.78}, {0, false, 96, 20, 200, 0.31}, {0, false, 2048, 400, 400, 0.69},
    {0, true, 4, 2000, 2000, 1.11}, {0, true, 32, 500, 500, 1.09}, {0, true, 128, 100, 100, 1.07},
    {0, true, 1000, 20, 200, 1.30}, {0, true, 600, 100, 400, 1.14}, {0, true, 16, 500, 500, 0.72},
    {0, true, 64, 100, 100, 0.46}, {0, true, 4, 1500, 1500, 0.75}, {0, true, 256, 32, 32, 0.15},
};

}  // namespace

int main() {
  int bad = 0;
  std::mt19937 g(3);
  for (const Timed& t : kTimed) {
    std::vector<sp2::RunInst> in(t.count);
    for (auto& i : in) i.n = t.lo + static_cast<int64_t>(g() % (t.hi - t.lo + 1));
    in.push_back(sp2::RunInst{6000, true});   // computes no square
    const bool pays = sp2::resident_batch_pays(in, t.precision, t.mcweeny);
    if ((t.ratio > 1.05 && pays) || (t.ratio < 0.85 && !pays)) {
      fprintf(stderr, "precision %d mcweeny %d: %d of %lld to %lld rows, ratio %.2f, resident %d\n",
              t.precision, t.mcweeny, t.count, static_cast<long long>(t.lo),
              static_cast<long long>(t.hi), t.ratio, pays);
      ++bad;
    }
  }
  if (!bad) printf("ok\n");
  return bad != 0;
}
