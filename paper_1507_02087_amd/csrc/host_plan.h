// Host-side planning of the square launches (internal): the padded row
// stride of an iterate, the order of the upper tiles of a tile grid, and the
// division of a launch group's tiles into workgroups (with K-split tail
// tiles). Pure host code with no GPU calls, built on its own with the
// sanitizers in the host checks of the test suite.
#pragma once

#include <stdint.h>

#include <vector>

#include "sp2_device.h"

namespace sp2 {

int64_t row_stride(int64_t np);

void append_tile_list(int nt, std::vector<int2>& out);

// Work plan of one launch group.
struct Plan {
  std::vector<WorkItem> items;   // one per workgroup
  std::vector<TailItem> tails;
  int split = 1;
};

Plan make_plan(const std::vector<int>& slots, const std::vector<int>& owner,
               const std::vector<int>& nk, int concurrency, int tail_split);

// Work plan of a resident run.
struct RunInst {
  int64_t n = 0;
  bool trivial = false;   // no squares: one workgroup forms the result
};
struct RunPlan {
  int mb = 0;                    // tile edge / 16 (0: no plan fits)
  std::vector<RunSeat> seats;    // one per workgroup
  int teams = 0;
  // instances that the teams take one after another, largest first, when
  // there are more than teams (empty: a team per instance)
  std::vector<int32_t> pull;
  double step_us = 0.0;          // estimated time of one product
};

// Seats for every instance of the batch on a device that holds `grid`
// workgroups of `num_cus` CUs at once (grid(mb): their number for a tile
// edge), with the tile edge (of `edges`, ended by 0) that the cost model
// finds fastest.
RunPlan plan_run(const std::vector<RunInst>& inst, int precision, const int* edges,
                 const std::vector<int>& grids, int num_cus);

}  // namespace sp2
