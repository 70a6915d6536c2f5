// Host-side planning of the square launches; see host_plan.h.
#include "host_plan.h"

#include <algorithm>

namespace sp2 {

// Row stride of an instance's iterate buffers for padded dimension np: np,
// plus 128 elements when np is a multiple of 512 of at least 2048, so that
// the rows of a tile do not all start at one offset modulo the memory
// channel interleave (at N = 8192 this made the BF16x3 square 2 % faster;
// a 16-element pad, which breaks the 128-byte alignment of bf16 rows, was
// 7 % slower).
int64_t row_stride(int64_t np) {
  return (np >= 2048 && np % 512 == 0) ? np + 128 : np;
}

// Upper-triangle tiles (I <= J) of an nt x nt tile grid, ordered by groups of
// G x G neighbouring tiles so that consecutive list entries share row panels.
void append_tile_list(int nt, std::vector<int2>& out) {
  const int G = 4;
  for (int gi = 0; gi < nt; gi += G)
    for (int gj = gi; gj < nt; gj += G)
      for (int i = gi; i < gi + G && i < nt; ++i)
        for (int j = gj; j < gj + G && j < nt; ++j)
          if (i <= j) out.push_back(make_int2(i, j));
}

// Given the group's tiles (global slots, owning instance, K slices of each),
// splits the tiles of an incomplete last round of workgroups into K pieces
// and deals the work to the 8 XCDs: workgroup b runs on XCD b mod 8, so XCD x
// receives a contiguous chunk of the (neighbour-grouped) tile list followed
// by a chunk of the pieces, which keeps the panels its tiles share in its
// own L2. Pieces are numbered from 0 within the group.
Plan make_plan(const std::vector<int>& slots, const std::vector<int>& owner,
               const std::vector<int>& nk, int concurrency, int tail_split) {
  Plan pl;
  const int ntiles = static_cast<int>(slots.size());
  const int rounds = ntiles / concurrency;
  const int rem = ntiles % concurrency;
  int min_nk = 1 << 30;
  for (int k : nk) min_nk = std::min(min_nk, k);
  int split = 1;
  if (tail_split >= 2) {
    split = tail_split;
  } else if (tail_split == 0 && rem > 0 && 2 * rem <= concurrency) {
    split = std::min({concurrency / rem, min_nk / 2, 16});
  }
  split = std::max(1, std::min(split, min_nk));
  const int ntail = (split > 1) ? (rounds > 0 ? rem : ntiles) : 0;
  const int nfull = ntiles - ntail;
  const int npieces = ntail * split;
  pl.split = split;
  for (int t = 0; t < ntail; ++t)
    pl.tails.push_back(TailItem{owner[nfull + t], slots[nfull + t],
                                     t * split, 0});
  const int X = 8;
  std::vector<int> f0(X + 1, 0), q0(X + 1, 0);
  for (int x = 0; x < X; ++x) {
    f0[x + 1] = f0[x] + nfull / X + (x < nfull % X ? 1 : 0);
    q0[x + 1] = q0[x] + npieces / X + (x < npieces % X ? 1 : 0);
  }
  int per = 0;
  for (int x = 0; x < X; ++x)
    per = std::max(per, (f0[x + 1] - f0[x]) + (q0[x + 1] - q0[x]));
  pl.items.assign(static_cast<size_t>(per) * X,
                  WorkItem{0, -1, -1, 0, 0, 0});
  for (int x = 0; x < X; ++x) {
    const int nf = f0[x + 1] - f0[x], nq = q0[x + 1] - q0[x];
    for (int r = 0; r < nf + nq; ++r) {
      WorkItem& w = pl.items[static_cast<size_t>(r) * X + x];
      if (r < nf) {
        const int t = f0[x] + r;
        w = WorkItem{owner[t], slots[t], -1, 0, nk[t], 0};
      } else {
        const int q = q0[x] + (r - nf);
        const int t = nfull + q / split, j = q % split;
        w = WorkItem{
            owner[t], slots[t], q,
            static_cast<int32_t>(static_cast<int64_t>(j) * nk[t] / split),
            static_cast<int32_t>(static_cast<int64_t>(j + 1) * nk[t] / split),
            0};
      }
    }
  }
  return pl;
}

namespace {

// Time (us) of one tile of edge 16 mb over k columns on a CU that works on
// `share` tiles at once, and of a product's meeting: a fit to runs of N = 48
// to 5000 at every edge. Measured single runs take 0.66 to 0.87 of it up to
// N = 350, where only the small tile is in question, and 0.89 to 1.14 past
// that; batches of up to 1000 rows 0.6 to 1.7 of it, of larger ones up to 2.5
// (it knows nothing of the caches), so it ranks layouts and is not what
// resident_batch_pays goes by.
double run_tile_us(int precision, int mb, double k, double share) {
  // flops / us of a CU's matrix cores, by precision and edge
  static const double rate[3][6] = {{0, 0, 0.272e6, 0.272e6, 0.272e6, 0},
                                    {0, 0, 0.55e6, 0.55e6, 0.55e6, 0.55e6},
                                    {0, 0, 0.95e6, 0, 1.56e6, 0}};
  // reduction, epilogue and store of a tile
  static const double epi[3][6] = {{0, 0, 4.4, 6.3, 5.5, 0},
                                   {0, 0, 3.3, 5.4, 7.0, 10.0},
                                   {0, 0, 3.2, 0, 7.0, 0}};
  const double bm = 16.0 * mb;
  return share * (2.0 * bm * bm * k / rate[precision][mb] + epi[precision][mb]);
}
constexpr double kRunMeetUs = 8.0;

}  // namespace

// Measured on 32 to 6144 rows and 2 to 2048 instances, equal and mixed (time of
// a step, resident over other driver). The other drivers' 128-tiles need
// many large instances to fill the device, and waste what they pad; then
// they are the faster ones, because an element of theirs is fetched half as
// often as one of a 32- to 64-tile, and the teams of several large
// instances evict each other's iterates from the L2s. `work` is the sum of
// N^2 (tiles), `padded` the same over whole 128-tiles.
//   One large instance with small ones as a single run; two: 0.3 to 0.99
//             (BF16x3 2 x 3500: 1.01, McWeeny 2500: 1.04)
//   FP64      (whole runs: the more accurate sums stop some steps later)
//             256 x 600: 0.97, 32 x 700: 1.14, 16 x 1000: 0.98, 64: 1.09, 64 x 1500: 1.14, 8 x 1750: 1.07,
//             4 x 2000: 1.08, 8 x 3000: 1.15; 256 of 64 to 1024 rows (padded 1.2): 0.74,
//             64 of 200 to 1500 (1.14): 0.93
//     McWeeny 16 x 500: 0.72, 32: 1.09, 16 x 1750: 0.93, 32: 1.01, 128 x 100: 1.07
//   FP32      128 x 1000: 0.99, 512: 1.08, 64 x 2000: 0.97, 128: 1.05, 3 x 3000: 1.05,
//             512 of 64 to 1024 rows (padded 1.19): 0.84
//     McWeeny 128 x 1000: 1.00, 512: 1.11, 64 x 1500: 1.00, 4 x 2000: 1.16
//   BF16x3    2048 x 500: 0.97, 32 x 1000: 0.92, 64: 1.04, 1024: 1.79, 6 x 1500: 0.81,
//             8: 1.03, 4 x 2000: 1.02, 8 x 3500: 1.75; 512 of 64 to 1024 rows: 0.90
//     McWeeny 256 x 200: 0.61, 1024: 1.06, 32 x 750: 0.80, 64: 1.18, 6 x 1250: 0.94,
//             8: 1.20, 3 x 2000: 1.19
bool resident_batch_pays(const std::vector<RunInst>& inst, int precision, bool mcweeny) {
  int64_t most = 0, active = 0;
  double work = 0.0, padded = 0.0;
  for (const RunInst& i : inst) {
    if (i.trivial) continue;
    const double n = static_cast<double>(i.n), p = static_cast<double>((i.n + 127) / 128 * 128);
    ++active;
    most = std::max(most, i.n);
    work += n * n;
    padded += p * p;
  }
  const double m2 = static_cast<double>(most) * static_cast<double>(most);
  if (work <= 1.2 * m2) return true;   // as a single run
  if (work <= 2.05 * m2) return precision != 2 || most <= (mcweeny ? 2200 : 3000);
  if (precision == 0) {
    const bool mixed = padded >= 1.115 * work && work <= 0.7 * m2 * static_cast<double>(active);
    if (!mcweeny)
      return most <= 600 || (most <= 1750 && (active <= 16 || (mixed && work <= 200e6)));
    return most <= 32 || (most <= 1750 && active <= (most <= 100 ? 64 : 16));
  }
  if (precision == 1) {
    const bool fits = work <= (mcweeny ? 125e6 : 150e6) || padded >= 1.1 * work;
    return most <= (mcweeny ? 1500 : 2000) && fits;
  }
  if (mcweeny)
    return most <= 160 || work <= (most <= 450 ? 40e6 : (most <= 1100 ? 20e6 : 9.4e6));
  return most <= 600 || work <= (most <= 1100 ? 36e6 : 15e6) ||
         (most <= 1100 && padded >= 1.15 * work && work <= 200e6);
}

RunPlan plan_run(const std::vector<RunInst>& inst, int precision, const int* edges,
                 const std::vector<int>& grids, int num_cus) {
  const int count = static_cast<int>(inst.size());
  RunPlan best;
  std::vector<int> best_size;
  int best_cap = 0, best_team = 0;
  for (int q = 0; edges[q]; ++q) {
    // a single run in FP32 or BF16x3 takes one workgroup per CU: its four
    // waves alone keep the matrix cores busy, and a second workgroup only
    // gets in their way (FP32, N = 4000, 48-tiles: 553 us a step against
    // 585). In FP64 a second one hides the first's epilogue (N = 4000,
    // 64-tiles: 966 us against 1023), and the instances of a batch hide each
    // other's waits.
    const int mb = edges[q], bm = 16 * mb;
    const int cap =
        (count == 1 && precision != 0) ? std::min(grids[q], num_cus) : grids[q];
    if (cap < 1) continue;
    // FP64 64-tiles leave no registers for the second set of sums, so a
    // wave's K part is one chain; up to kRunChainN rows the launch sequence
    // of a single run has shorter ones (N = 1225 to 1400: its errors were
    // 1.15 to 1.19 times smaller). A batch's other driver never has.
    if (count == 1 && precision == 0 && mb == 4 && inst[0].n <= kRunChainN) continue;
    std::vector<int64_t> tiles(count);
    std::vector<double> tile_us(count);
    int64_t total = 0;
    for (int b = 0; b < count; ++b) {
      const int64_t nt = (inst[b].n + bm - 1) / bm;
      tiles[b] = inst[b].trivial ? 1 : nt * (nt + 1) / 2;
      total += tiles[b];
    }
    if (count == 1) {
      const double us = run_tile_us(precision, mb, static_cast<double>(inst[0].n), 1.0) *
                        static_cast<double>((total + num_cus - 1) / num_cus);
      if (best.mb == 0 || us + kRunMeetUs < best.step_us) {
        best.mb = mb;
        best_cap = cap;
        best.step_us = us + kRunMeetUs;
        best_size.assign(1, static_cast<int>(std::min<int64_t>(total, cap)));
      }
      continue;
    }
    // how many tiles a CU works on at once
    const double share = std::min<double>(
        std::max(1.0, static_cast<double>(total) / num_cus), static_cast<double>(cap) / num_cus);
    double lo = 0.0, hi = 0.0;
    for (int b = 0; b < count; ++b) {
      tile_us[b] = inst[b].trivial
                       ? 1.0
                       : run_tile_us(precision, mb, static_cast<double>(inst[b].n), share);
      hi = std::max(hi, tile_us[b] * static_cast<double>(tiles[b]));
    }
    // smallest step time whose teams fit: a team of ceil(tiles / rounds)
    auto seats_for = [&](double us, std::vector<int>* size) {
      int64_t s = 0;
      for (int b = 0; b < count; ++b) {
        const int64_t rounds = static_cast<int64_t>(us / tile_us[b]);
        if (rounds < 1) return static_cast<int64_t>(cap) + 1;
        const int64_t g = (tiles[b] + rounds - 1) / rounds;
        if (size) (*size)[b] = static_cast<int>(g);
        s += g;
      }
      return s;
    };
    hi *= 1.0001;
    // Teams of equal size that take instances from a list: each step of an
    // instance costs its team the rounds and the meeting, and the list is
    // done when the teams' shares are, but not before its longest entry.
    // (512 FP32 instances of 64 to 1024 rows: teams of 4 or 8 at 48- or
    // 64-tiles 41 to 42 ms, of 16 43 to 44, the queue 48.8; 200 BF16x3 ones
    // of 60 to 800 rows: teams of 8 at 64-tiles 7.2 ms, of 4 9.7, queue 10.3.)
    for (int size = 1; size <= std::min(cap, 32); size *= 2) {
      const int teams = cap / size / 8 * 8;   // the same number on every XCD
      if (teams == 0 || teams >= count) continue;
      double sum = 0.0, longest = 0.0;
      for (int b = 0; b < count; ++b) {
        if (inst[b].trivial) continue;
        const double us = tile_us[b] * static_cast<double>((tiles[b] + size - 1) / size) +
                          kRunMeetUs;
        sum += us;
        longest = std::max(longest, us);
      }
      // (per step of the batch, as the other estimates)
      const double us = std::max(sum / teams, longest);
      if (best.mb == 0 || us < best.step_us) {
        best.mb = mb;
        best.step_us = us;
        best_cap = cap;
        best_team = size;
      }
    }
    if (cap < count || seats_for(hi, nullptr) > cap) continue;
    for (int it = 0; it < 40; ++it) {
      const double mid = 0.5 * (lo + hi);
      (seats_for(mid, nullptr) <= cap ? hi : lo) = mid;
    }
    if (best.mb == 0 || hi + kRunMeetUs < best.step_us) {
      best.mb = mb;
      best_cap = cap;
      best.step_us = hi + kRunMeetUs;
      best_team = 0;
      best_size.assign(count, 0);
      seats_for(hi, &best_size);
    }
  }
  if (best.mb == 0) return best;
  if (best_team > 0) {
    // the list, largest first; team t starts with its t-th entry. A team's
    // seats are consecutive in an XCD's column of the grid.
    std::vector<int32_t> list(count);
    for (int b = 0; b < count; ++b) list[b] = b;
    std::stable_sort(list.begin(), list.end(), [&](int32_t a, int32_t b) {
      return (inst[a].trivial ? 0 : inst[a].n) > (inst[b].trivial ? 0 : inst[b].n);
    });
    const int X = 8, teams = best_cap / best_team / 8 * 8;
    best.teams = teams;
    const int rows = teams / X * best_team;
    best.seats.assign(static_cast<size_t>(rows) * X, RunSeat{0, 0, 0, 0, 0, 0});
    for (int t = 0; t < teams; ++t)
      for (int r = 0; r < best_team; ++r)
        best.seats[static_cast<size_t>(t / X * best_team + r) * X + t % X] =
            RunSeat{list[t], r, best_team, t * best_team, 0, t};
    best.pull.assign(list.begin() + teams, list.end());
    return best;
  }
  best.teams = count;
  // Workgroup b runs on XCD b mod 8: a team of up to 32 workgroups (the CUs
  // of an XCD) goes to the least loaded XCD, whose L2 then serves all its
  // exchanges; a larger one is dealt in eight contiguous parts, so that
  // neighbouring tiles share their panels' XCD.
  const int X = 8;
  std::vector<int> order(count);
  for (int b = 0; b < count; ++b) order[b] = b;
  std::stable_sort(order.begin(), order.end(),
                   [&](int a, int b) { return best_size[a] > best_size[b]; });
  std::vector<std::vector<RunSeat>> col(X);
  std::vector<int> base(count, 0);
  int next = 0;
  for (int b = 0; b < count; ++b) {
    base[b] = next;
    next += best_size[b];
  }
  auto least = [&]() {
    int x = 0;
    for (int y = 1; y < X; ++y)
      if (col[y].size() < col[x].size()) x = y;
    return x;
  };
  int total = 0;
  for (int s : best_size) total += s;
  const size_t rows = static_cast<size_t>((total + X - 1) / X);
  for (int b : order) {
    const int size = best_size[b];
    const int x = least();
    const bool fits = (count == 1) ? size * X <= best_cap : col[x].size() + size <= rows;
    if (size <= 32 && fits) {
      for (int r = 0; r < size; ++r) col[x].push_back(RunSeat{b, r, size, base[b], 0, b});
    } else {
      int r = 0;
      for (int y = 0; y < X; ++y) {
        const int part = (size - r + X - y - 1) / (X - y);
        for (int k = 0; k < part && col[y].size() < rows; ++k)
          col[y].push_back(RunSeat{b, r++, size, base[b], 0, b});
      }
      while (r < size) col[least()].push_back(RunSeat{b, r++, size, base[b], 0, b});
    }
  }
  size_t depth = 0;
  for (const auto& c : col) depth = std::max(depth, c.size());
  best.seats.assign(depth * X, RunSeat{0, 0, 0, 0, 0, 0});
  for (int x = 0; x < X; ++x)
    for (size_t k = 0; k < col[x].size(); ++k) best.seats[k * X + x] = col[x][k];
  // The last round's tiles go to the seats of the lowest rows of the grid
  // (row k of an XCD's column is its k-th workgroup, so the first rows are
  // the first workgroups of its CUs), numbered XCD by XCD. Dealt by rank,
  // they would all fall on the CUs of the first XCDs.
  std::vector<int64_t> rem(count), given(count, 0), number(count);
  for (int b = 0; b < count; ++b) {
    const int64_t nt = (inst[b].n + 16 * best.mb - 1) / (16 * best.mb);
    const int64_t tiles = inst[b].trivial ? 0 : nt * (nt + 1) / 2;
    rem[b] = tiles % best_size[b];
    number[b] = tiles - rem[b];
  }
  const int none = INT32_MAX;
  for (RunSeat& s : best.seats) {
    if (s.size == 0) continue;
    s.last = (given[s.inst]++ < rem[s.inst]) ? 0 : none;
  }
  for (int x = 0; x < X; ++x)
    for (size_t k = 0; k < depth; ++k) {
      RunSeat& s = best.seats[k * X + x];
      if (s.size > 0 && s.last != none) s.last = static_cast<int32_t>(number[s.inst]++);
    }
  return best;
}

}  // namespace sp2
