// Spectral norm of E = X~ - X~^2 for one dense instance whose iterate fits
// the register files of the device (the Lanczos process of spectral.hip, for
// dimensions up to spectral_resident_rows).
//
// A Lanczos step applies the iterate twice, and the process takes up to 64
// steps. Read from memory each time, 64 MB at N = 4000 in FP32, the iterate
// bounds the norm (35 us a product where every chunk of rows waits for its
// share, 3.0 ms a norm). Here one cooperative launch loads it once: every
// wave keeps RPW rows in its registers, 16 rows of 4000 floats a CU, and the
// products read only the vector, from LDS.
//
// All workgroups hold the Lanczos vectors q_{j-1}, q_j whole, in LDS, and
// compute alpha, beta and the normalisation redundantly (4000 elements over
// 512 threads), so that a step exchanges nothing but the two products'
// outputs: each workgroup writes its rows through to where every XCD sees
// them, then its phase, and waits for the phases of all others. Two buffers
// suffice: a workgroup that writes phase p + 2 has seen everyone's phase
// p + 1, which follows their reading of p. The last workgroup holds no rows;
// it follows the recurrence coefficients, updates the estimate from T_j and
// decides whether it is final (the same tests as spectral.hip), beside the
// products and not between them. The others run on meanwhile and stop when
// they see the decision.
//
// Measured, us a Lanczos step (two products; chunked kernel -> here): N = 100
// 30 -> 12, FP32 1000 39 -> 15, 4000 67 -> 21; FP64 1000 41 -> 15, 2500 59 ->
// 18. What is left: two exchanges (3 to 4 us each at N = 100), the vector's
// way through the memory side (8 bytes of every row to every CU) and, at
// N <= 1000, the deciding workgroup. Reading the vector through the L2 after
// an acquire fence instead of past it was slower (N = 4000: 25.8 us a step).
#include <math.h>

#include "sp2_device.h"

namespace sp2 {
namespace {

constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr double kSpecTol = 1e-12;
typedef double f64x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double wave_sum(double x) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// Sum over the workgroup, returned to every thread (fixed order).
__device__ __forceinline__ double block_sum(double x, double* red) {
  x = wave_sum(x);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = x;
  __syncthreads();
  double t = red[0];
  for (int w = 1; w < kWaves; ++w) t += red[w];
  return t;
}

__device__ __forceinline__ int peek(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double peek(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void post(int32_t* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void post(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Eigenvalues below x of a tridiagonal with diagonal a and squared
// off-diagonal b2 (b2[i] couples rows i and i - 1; b2[0] = 0), scaled to a
// Gershgorin bound of 1: the sign changes of the leading principal minors, one
// dependent fused multiply-add a row where the pivots of sturm_below take a
// division. A zero minor has the sign opposite to the one before it. Rows are
// taken in blocks of eight, read from LDS ahead of their chain; rows past the
// order (a = 2, b2 = 0, but kPadLink in the first) keep the sign. The link
// gives a zero last minor (x is an eigenvalue) a successor of the sign it
// counts as, where a chain of zeros would count one change a row; to a minor
// that is not zero to within rounding it adds nothing. (The test for it in
// the loop, on two zeros, took 0.7 us a Lanczos step.) The minors shrink by at
// most some 2^-50 a row, so a rescale every block keeps them in range.
constexpr double kPadLink = 0x1p-100;
__device__ __forceinline__ int minors_below(const double* a, const double* b2, int blocks,
                                            double x) {
  double p0 = 0.0, p1 = 1.0;
  bool neg = false;
  int cnt = 0;
  f64x2 av[4], bv[4];
  auto fetch = [&](int q) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      av[e] = *reinterpret_cast<const f64x2*>(a + 8 * q + 2 * e);
      bv[e] = *reinterpret_cast<const f64x2*>(b2 + 8 * q + 2 * e);
    }
  };
  fetch(0);
  for (int q = 0; q < blocks; ++q) {
    double d[8], b[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      d[e] = av[e >> 1][e & 1] - x;
      b[e] = bv[e >> 1][e & 1];
    }
    if (q + 1 < blocks) fetch(q + 1);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const double p2 = fma(d[e], p1, -b[e] * p0);
      const bool ng = (p2 == 0.0) ? !neg : p2 < 0.0;
      cnt += (ng != neg) ? 1 : 0;
      neg = ng;
      p0 = p1;
      p1 = p2;
    }
    if (fmax(fabs(p0), fabs(p1)) < 0x1p-400) {
      p0 *= 0x1p+400;
      p1 *= 0x1p+400;
    }
  }
  return cnt;
}

// Both end eigenvalues of (ta, tb) of order m <= 64 at once by 256 threads,
// as tridiag_ends finds them (128 points a round and end, six rounds): sa, sb
// take the scaled matrix, hits is an LDS array of 4 ints.
__device__ __forceinline__ void ends(const double* ta, const double* tb, int m, double* sa,
                                     double* sb, int* hits, double* out, double* bottom,
                                     double* top) {
  static_assert(kLanczosMax == 64, "a row per lane");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double lo = INFINITY, hi = -INFINITY;
  if (lane < m) {
    const double r = (lane > 0 ? fabs(tb[lane - 1]) : 0.0) + (lane + 1 < m ? fabs(tb[lane]) : 0.0);
    lo = ta[lane] - r;
    hi = ta[lane] + r;
  }
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off, 64));
    hi = fmax(hi, __shfl_xor(hi, off, 64));
  }
  const double scale = fmax(fabs(lo), fabs(hi));
  if (!(scale > 0.0) || !isfinite(scale)) {   // T = 0, or not a number
    *bottom = *top = scale;
    return;
  }
  const double is = 1.0 / scale;
  __syncthreads();   // sa, sb may still be read for the previous order
  if (wave == 0) {
    sa[lane] = (lane < m) ? ta[lane] * is : 2.0;
    const double b = (lane > 0 && lane < m) ? tb[lane - 1] * is : 0.0;
    sb[lane] = (lane == m) ? kPadLink : b * b;
  }
  __syncthreads();
  lo *= is;
  hi *= is;
  const int half = wave >> 1, t = threadIdx.x & 127;
  const int rank = half ? m : 1;
  for (int round = 0; round < 6; ++round) {
    const double h = (hi - lo) / 128;
    const bool hit = minors_below(sa, sb, (m + 7) / 8, lo + h * (t + 1)) >= rank;
    const unsigned long long mask = __ballot(hit);
    __syncthreads();   // hits may still be read from the previous round
    if (lane == 0)
      hits[wave] = mask ? (wave & 1) * 64 + __ffsll(static_cast<long long>(mask)) - 1 : 127;
    __syncthreads();
    const int first = min(hits[2 * half], hits[2 * half + 1]);
    hi = lo + h * (first + 1);
    lo = lo + h * first;
  }
  if (t == 0) out[half] = 0.5 * (lo + hi) * scale;
  __syncthreads();
  *bottom = out[0];
  *top = out[1];
}

// The deciding workgroup: T_j for j = 1, 2, ... from the coefficients as the
// first workgroup posts them. Its first 256 threads find the end
// eigenvalues.
__device__ __forceinline__ void decide(const SpecRunArgs& a, const Instance& in, double* ta,
                                       double* tb, double* sa, double* sb, int* hits,
                                       double* out, int* flag) {
  if (threadIdx.x >= 256) return;
  double prev = 0.0;
  for (int j = 1;; ++j) {
    if (threadIdx.x == 0) {
      const long long t0 = wall_clock64();
      int ok = 1;
      while (peek(a.ctl + kSpecRunCount) < a.iter * 256 + j) {
        if (wall_clock64() - t0 > a.wait_limit || peek(a.err) != 0) {
          post(a.err, 1);
          ok = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
      asm volatile("" ::: "memory");
      if (ok) {
        ta[j - 1] = peek(a.hist + 2 * (j - 1));
        tb[j - 1] = peek(a.hist + 2 * (j - 1) + 1);
      }
      *flag = ok;
    }
    __syncthreads();
    if (!*flag) return;
    const double beta = tb[j - 1];
    double bot, top;
    ends(ta, tb, j, sa, sb, hits, out, &bot, &top);
    const double theta = fmax(fabs(top), fabs(bot));
    const bool fin = !(beta > 1e-14 * theta) || !isfinite(beta) ||
                     (j >= 2 && fabs(theta - prev) <= kSpecTol * theta) ||
                     j == kLanczosMax || j == in.n;
    if (fin) {
      if (threadIdx.x == 0) {
        in.st->m[a.iter - 1] = theta;
        in.st->krylov[a.iter - 1] = j;
        post(a.ctl + kSpecRunStop, a.iter);
      }
      return;
    }
    prev = theta;
  }
}

// T: storage of the iterate; RPW rows of at most 256 SEG columns per wave.
template <typename T, int RPW, int SEG>
__global__ __launch_bounds__(kThreads, 2) void spectral_resident_kernel(SpecRunArgs a) {
  constexpr int NV = 256 * SEG;      // length of the vectors in LDS
  constexpr int RPB = kWaves * RPW;  // rows of a workgroup
  constexpr int NE = (NV + kThreads - 1) / kThreads;   // entries of a thread
  typedef T vec2 __attribute__((ext_vector_type(2)));
  __shared__ __attribute__((aligned(16))) double vec[3][NV];
  __shared__ double red[kWaves];
  __shared__ __attribute__((aligned(16))) double ta[kLanczosMax], tb[kLanczosMax],
      sa[kLanczosMax], sb[kLanczosMax];
  __shared__ int hits[kWaves], flag;
  const Instance& in = *a.inst;
  if (in.st->done) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int iter = a.iter;
  const int rows_wg = gridDim.x - 1;   // workgroups with rows
  if (static_cast<int>(blockIdx.x) == rows_wg) {
    decide(a, in, ta, tb, sa, sb, hits, red, &flag);
    return;
  }
  const int n = in.n, ld = in.ld;
  const int nr = min(rows_wg * RPB, NV);   // rows that some workgroup writes
  const int row0 = blockIdx.x * RPB + wave * RPW;
  // the rows of this wave: lane l holds columns 2 l, 2 l + 1 of every run of
  // 128 columns, so that the vector's reads from LDS are contiguous
  const T* X = static_cast<const T*>(in.X[(iter - 1) & 1]);
  vec2 x[RPW][2 * SEG];
#pragma unroll
  for (int r = 0; r < RPW; ++r)
#pragma unroll
    for (int s = 0; s < 2 * SEG; ++s) {
      const int row = row0 + r, col = 128 * s + 2 * lane;
      // the padding columns of the iterate are zero
      x[r][s] = (row < n && col < ld)
                    ? *gro(reinterpret_cast<const vec2*>(X + static_cast<size_t>(row) * ld + col))
                    : vec2{0, 0};
    }
  const OpMap m = op_map(in.prm.method, in.st->p[iter], in.st->alpha[iter]);
  auto matvec = [&](const double* v, double (&out)[RPW]) {
#pragma unroll
    for (int r = 0; r < RPW; ++r) out[r] = 0.0;
#pragma unroll
    for (int s = 0; s < 2 * SEG; ++s) {
      const f64x2 q = *reinterpret_cast<const f64x2*>(v + 128 * s + 2 * lane);
#pragma unroll
      for (int r = 0; r < RPW; ++r) {
        // opaque, or the conversions to FP64 would be hoisted out of the
        // Lanczos loop into twice the registers
        asm volatile("" : "+v"(x[r][s]));
        out[r] = fma(static_cast<double>(x[r][s].x), q.x, out[r]);
        out[r] = fma(static_cast<double>(x[r][s].y), q.y, out[r]);
      }
    }
#pragma unroll
    for (int r = 0; r < RPW; ++r) out[r] = wave_sum(out[r]);
  };
  int phase = iter * 256;
  // Every wave's outputs are complete before the phase is posted.
  auto publish = [&]() {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    ++phase;
    if (tid == 0) post(a.phase + blockIdx.x, phase);
  };
  // Waits for every workgroup's phase; false once the estimate is final (or
  // a wait exceeded its limit).
  auto collect = [&]() -> bool {
    bool stop = false;
    if (tid < rows_wg) {
      const long long t0 = wall_clock64();
      while (peek(a.phase + tid) < phase) {
        if (peek(a.ctl + kSpecRunStop) == iter || peek(a.err) != 0) {
          stop = true;
          break;
        }
        if (wall_clock64() - t0 > a.wait_limit) {
          post(a.err, 1);
          stop = true;
          break;
        }
      }
    }
    asm volatile("" ::: "memory");
    return !__syncthreads_or(stop);
  };
  double* qp = vec[0];
  double* qn = vec[1];
  double* const vin = vec[2];
  for (int i = tid; i < NV; i += kThreads) qp[i] = 0.0;
  for (int j = 0;; ++j) {
    // u_j = w_{j-1} - alpha_{j-1} q_{j-1}, beta_{j-1} = ||u_j||, q_j
    double w[NE];
    double alpha = 0.0;
    if (j > 0) {
      if (!collect()) return;
      const double* src = a.data + (phase & 1) * kSpecRunMax;
      const double* dot = a.dots + (phase & 1) * kSpecRunMax;
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const int i = tid + e * kThreads;
        w[e] = (i < nr) ? peek(src + i) : 0.0;
      }
      double d = 0.0;
      for (int i = tid; i < rows_wg * kWaves; i += kThreads) d += peek(dot + i);
      alpha = block_sum(d, red);
    } else {
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const int i = tid + e * kThreads;
        w[e] = (i < n) ? spec_start_entry(i) : 0.0;
      }
    }
    double nu = 0.0;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int i = tid + e * kThreads;
      if (i < NV) w[e] -= alpha * qp[i];
      nu += w[e] * w[e];
    }
    const double beta = sqrt(block_sum(nu, red));
    if (j > 0 && blockIdx.x == 0 && tid == 0) {
      post(a.hist + 2 * (j - 1), alpha);
      post(a.hist + 2 * (j - 1) + 1, beta);
      __builtin_amdgcn_s_waitcnt(0);
      post(a.ctl + kSpecRunCount, iter * 256 + j);
    }
    if (j == kLanczosMax) return;
    const double inv = (beta > 0.0) ? 1.0 / beta : 0.0;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int i = tid + e * kThreads;
      if (i < NV) qn[i] = w[e] * inv;
    }
    __syncthreads();
    // y = X~ q_j: the buffer holds Y = a X~ + c I (OpMap)
    double y[RPW], z[RPW];
    matvec(qn, y);
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
      const int row = row0 + r;
      y[r] = (row < n) ? (y[r] - m.c * qn[row]) / m.a : 0.0;
      if (lane == 0 && row < kSpecRunMax) post(a.data + ((phase + 1) & 1) * kSpecRunMax + row, y[r]);
    }
    publish();
    if (!collect()) return;
    {
      const double* src = a.data + (phase & 1) * kSpecRunMax;
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const int i = tid + e * kThreads;
        if (i < NV) vin[i] = (i < nr) ? peek(src + i) : 0.0;
      }
    }
    __syncthreads();
    // w_j = X~ q_j - X~ (X~ q_j) - beta_{j-1} q_{j-1}; q_j . w_j
    matvec(vin, z);
    double dot = 0.0;
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
      const int row = row0 + r;
      if (row >= n) z[r] = 0.0;
      else z[r] = y[r] - (z[r] - m.c * y[r]) / m.a - beta * qp[row];
      dot += (row < n) ? qn[row] * z[r] : 0.0;
      if (lane == 0 && row < kSpecRunMax) post(a.data + ((phase + 1) & 1) * kSpecRunMax + row, z[r]);
    }
    if (lane == 0) post(a.dots + ((phase + 1) & 1) * kSpecRunMax + blockIdx.x * kWaves + wave, dot);
    publish();
    double* const t = qp;
    qp = qn;
    qn = t;
  }
}

struct Pick {
  const void* fn = nullptr;
  int rpb = 0;   // rows of a workgroup
};

// The smallest kernel whose registers hold n rows on a device of num_cus
// CUs, one of which decides.
Pick pick(bool fp64, int n, int num_cus) {
  struct Entry {
    const void* fn;
    int rpw, cols;
  };
#define SP2_SPEC(T, R, S) \
  Entry { reinterpret_cast<const void*>(&spectral_resident_kernel<T, R, S>), R, 256 * S }
  static const Entry f32[] = {SP2_SPEC(float, 1, 2), SP2_SPEC(float, 1, 4), SP2_SPEC(float, 1, 8),
                              SP2_SPEC(float, 2, 12), SP2_SPEC(float, 2, 16)};
  static const Entry f64[] = {SP2_SPEC(double, 1, 2), SP2_SPEC(double, 1, 4),
                              SP2_SPEC(double, 1, 8), SP2_SPEC(double, 2, 11)};
#undef SP2_SPEC
  const Entry* e = fp64 ? f64 : f32;
  const int cnt = fp64 ? 4 : 5;
  for (int q = 0; q < cnt; ++q)
    if (n <= e[q].cols && n <= e[q].rpw * kWaves * (num_cus - 1))
      return Pick{e[q].fn, e[q].rpw * kWaves};
  return Pick{};
}

}  // namespace

int spectral_resident_grid(bool fp64_store, int n, int num_cus) {
  const Pick p = pick(fp64_store, n, num_cus);
  if (!p.fn) return 0;
  const int grid = (n + p.rpb - 1) / p.rpb + 1;
  int per = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, p.fn, kThreads, 0) != hipSuccess ||
      per * num_cus < grid)
    return 0;
  return grid;
}

hipError_t launch_spectral_resident(const SpecRunArgs& a, bool fp64_store, int n, int num_cus,
                                    int grid, hipStream_t s) {
  const Pick p = pick(fp64_store, n, num_cus);
  if (!p.fn || grid != (n + p.rpb - 1) / p.rpb + 1) return hipErrorInvalidValue;
  SpecRunArgs arg = a;
  void* params[] = {&arg};
  return hipLaunchCooperativeKernel(p.fn, dim3(grid), dim3(kThreads), params, 0, s);
}

}  // namespace sp2
