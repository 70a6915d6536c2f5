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

// FP64 resident runs past this N add up a wave's K part (a quarter of the K
// range) as one chain, without a second set of sums: the launch sequence
// adds the whole range as one chain there, so the result is still the more
// accurate one (N = 4096: 5.0e-15 against 8.5e-15), and rounding further
// below the resolution of the traces only delays the stop (ten runs at
// N = 3001: 303 steps with the second set, 292 without, 291 in sequence).
constexpr int kRunChainN = 1800;
// Single runs up to this N have chains of three blocks (48 columns in FP32, 24
// in FP64) at 32-tiles, and in FP32 at 48-tiles: the launch sequence splits
// the K range of such an instance into up to 16 pieces, and with the chains
// of the larger runs (9 or 12 blocks) errors were larger than its own (FP32
// N = 700: 7.6e-7 against 4.9e-7, FP64 N = 280: 1.52e-15 against 1.31e-15; with
// the short ones 4.2e-7 and 1.25e-15, and a step takes up to 1.5 % longer).
// Past it the sequence has the longer chains, and so has a batch's queue.
constexpr int kRunShortN = 1050;

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

// Whether the resident run is the faster driver of a batch: against the queue,
// or with `mcweeny` (two products a step) against the launch sequence.
bool resident_batch_pays(const std::vector<RunInst>& inst, int precision, bool mcweeny);

// Seats for every instance of the batch on a device that holds `grid`
// workgroups of `num_cus` CUs at once (grid(mb): their number for a tile
// edge), with the tile edge (of `edges`, ended by 0) that the cost model
// finds fastest.
RunPlan plan_run(const std::vector<RunInst>& inst, int precision, const int* edges,
                 const std::vector<int>& grids, int num_cus);

}  // namespace sp2
