// The symbolic count kernel of the block-sparse path on the CPU: its text
// (count_kernel.inc, taken from bsr.hip) with a thread per GPU thread. The
// workgroup of the scalar step sets `done` while the row workgroups look at
// it, so a read may give either value, and the waves' reads are independent:
// under every combination of values that the four waves may see, the threads
// of a workgroup pass the same barriers and read nothing out of range. With
// `done` unset for all, the counts and bitmaps are those of a direct
// computation. Prints "ok" and returns 0 when every check holds.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <barrier>
#include <memory>
#include <random>
#include <thread>
#include <vector>

#define __global__ static
#define __shared__ static
#define __launch_bounds__(n)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) read_flag(*(p))

namespace {

using std::min;
constexpr int kMaxBlockCols = 2048;
constexpr int kThreads = 256;

struct Index {
  int x;
};
thread_local Index threadIdx, blockIdx;
thread_local int barriers;            // passed by this thread
unsigned seen_done = 0;               // bit w: wave w reads done = 1
std::unique_ptr<std::barrier<>> group, waves[kThreads / 64];
int64_t lanes[kThreads];
double dlanes[kThreads];
int counted[kThreads];
int bad = 0, scalar_steps = 0;

void report(const char* what) {
  if (__atomic_fetch_add(&bad, 1, __ATOMIC_RELAXED) < 10) fprintf(stderr, "%s\n", what);
}

struct Flag {
  operator int() const { return (seen_done >> (threadIdx.x >> 6)) & 1; }
};
int read_flag(const Flag& f) { return f; }
struct DevState {
  Flag done;
};

template <typename T>
struct Checked {
  std::vector<T>* v;
  T& operator[](size_t i) const {
    static T none{};
    if (i < v->size()) return (*v)[i];
    report("access out of range");
    return none;
  }
};
struct BsrMat {
  Checked<int32_t> row_ptr, col, flag;
};
struct BsrSymbolic {
  Checked<uint32_t> bitmap;
  Checked<int32_t> wpre, qcnt, ucnt, nzrow;
};
struct BsrCounters {};
struct HostMirror {};
struct Instance {};
struct BsrScalar {
  const Instance* inst;
  const double* part;
  int32_t count;
  int32_t* ndone;
  HostMirror* mirror;
};

void __syncthreads() {
  ++barriers;
  group->arrive_and_wait();
}
int __syncthreads_count(bool x) {
  counted[threadIdx.x] = x;
  __syncthreads();
  int n = 0;
  for (int c : counted) n += c;
  __syncthreads();
  --barriers;
  return n;
}
// value of lane `src` of this thread's wave
template <typename T, typename A>
T exchange(A* arr, T x, int src) {
  const int t = threadIdx.x, w = t >> 6;
  arr[t] = x;
  waves[w]->arrive_and_wait();
  const T r = static_cast<T>(arr[64 * w + src]);
  waves[w]->arrive_and_wait();
  return r;
}
int __shfl_up(int x, int off, int) {
  const int l = threadIdx.x & 63;
  return exchange(lanes, x, l >= off ? l - off : l);
}
int __shfl_xor(int x, int off, int) { return exchange(lanes, x, (threadIdx.x & 63) ^ off); }
double wave_sum(double x) {
  for (int off = 32; off > 0; off >>= 1) x += exchange(dlanes, x, (threadIdx.x & 63) ^ off);
  return x;
}
int __popc(uint32_t x) { return __builtin_popcount(x); }
void atomicOr(uint32_t* p, uint32_t x) { __atomic_fetch_or(p, x, __ATOMIC_RELAXED); }
bool finalize_scalar(const Instance&, int iter, double a, double b, double c, double, int,
                     int32_t*, int, HostMirror*) {
  if (iter != 6 || a != 3.0 || b != 6.0 || c != 9.0) report("scalar step");
  ++scalar_steps;
  return true;
}

#include "count_kernel.inc"

}  // namespace

int main() {
  static_assert(kCountThreads == kThreads, "a thread per GPU thread");
  std::mt19937 g(7);
  // row lengths on both sides of a wave and of a workgroup
  const int nb = 300, nbw = (nb + 31) / 32;
  std::vector<int32_t> rp(1, 0), col, flag;
  for (int r = 0; r < nb; ++r) {
    const int want = (r % 7 == 0) ? nb : (r % 7 == 1 ? 1 : 1 + static_cast<int>(g() % 90));
    for (int c = 0; c < nb; ++c)
      if (c == r || static_cast<int>(g() % nb) < want) {
        col.push_back(c);
        flag.push_back(g() % 4 != 0);
      }
    rp.push_back(static_cast<int32_t>(col.size()));
  }
  std::vector<uint32_t> bits(nb * nbw);
  std::vector<int32_t> wpre(nb * nbw), qcnt(nb), ucnt(nb), nz(nb);
  const BsrMat A{{&rp}, {&col}, {&flag}};
  const BsrSymbolic sym{{&bits}, {&wpre}, {&qcnt}, {&ucnt}, {&nz}};
  std::vector<double> part;
  for (int i = 0; i < 3; ++i)
    for (double x : {1.0, 2.0, 3.0}) part.push_back(x);
  const Instance inst;
  const BsrScalar fin{&inst, part.data(), 3, nullptr, nullptr};
  DevState st;
  auto launch = [&](int block) {
    group = std::make_unique<std::barrier<>>(kThreads);
    for (auto& w : waves) w = std::make_unique<std::barrier<>>(64);
    std::vector<int> passed(kThreads);
    std::vector<std::thread> th;
    for (int t = 0; t < kThreads; ++t)
      th.emplace_back([&, t] {
        threadIdx.x = t;
        blockIdx.x = block;
        barriers = 0;
        bsr_symbolic_count_kernel(A, nb, nbw, sym, nullptr, &st, 7, fin);
        passed[t] = barriers;
        group->arrive_and_drop();   // a wave that has ended is not waited for
      });
    for (auto& t : th) t.join();
    for (int p : passed)
      if (p != passed[0]) {
        report("the waves of a workgroup take different branches");
        break;
      }
  };
  // every row counted, against a direct computation
  for (int I = 0; I < nb; I += 3) {
    launch(I);
    std::vector<bool> on(nb, false);
    on[I] = true;
    int flagged = 0, all = 0, upper = 0;
    for (int q = rp[I]; q < rp[I + 1]; ++q) {
      if (!flag[q]) continue;
      ++flagged;
      on[col[q]] = true;
      for (int k = rp[col[q]]; k < rp[col[q] + 1]; ++k)
        if (flag[k]) on[col[k]] = true;
    }
    for (int J = 0; J < nb; ++J) {
      all += on[J];
      upper += on[J] && J >= I;
      if (((bits[I * nbw + J / 32] >> (J % 32)) & 1) != on[J]) report("bitmap");
    }
    if (nz[I] != flagged || qcnt[I] != all || ucnt[I] != upper) report("counts");
  }
  launch(nb);
  if (scalar_steps != 1) report("scalar step not taken once");
  // done being set while a row workgroup looks at it
  for (int I : {0, 1, 2, 6})
    for (seen_done = 1; seen_done < 16; ++seen_done) launch(I);
  if (!bad) printf("ok\n");
  return bad != 0;
}
