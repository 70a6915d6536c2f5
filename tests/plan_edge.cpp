// Prints the tile edge / 16 that plan_run takes for a single run or a batch
// on 256 CUs: plan_edge PRECISION N[xCOUNT]... (host code only).
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include "../paper_1507_02087_amd/csrc/host_plan.h"

int main(int argc, char** argv) {
  const int precision = atoi(argv[1]);
  std::vector<sp2::RunInst> in;
  for (int a = 2; a < argc; ++a) {
    long n = 0, count = 1;
    sscanf(argv[a], "%ldx%ld", &n, &count);
    in.insert(in.end(), count, sp2::RunInst{n, false});
  }
  const int edges[3][5] = {{2, 3, 4, 0, 0}, {2, 3, 4, 5, 0}, {2, 4, 0, 0, 0}};
  // co-resident workgroups: two per CU, FP32's single runs at 64- and
  // 80-tiles one; no 80-tiles for batches
  std::vector<int> grids;
  for (int q = 0; edges[precision][q]; ++q) {
    const int mb = edges[precision][q];
    const bool solo = in.size() == 1;
    grids.push_back(precision == 1 && mb == 5 && !solo ? 0 : (precision == 1 && mb >= 4 && solo ? 256 : 512));
  }
  printf("%d\n", sp2::plan_run(in, precision, edges[precision], grids, 256).mb);
  return 0;
}
