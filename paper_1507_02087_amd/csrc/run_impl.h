// Resident runs: one launch computes a whole purification, from the affine
// start to the stop, for every instance of the batch (included by
// run_f64.hip, run_f32.hip and run_b3.hip). Its workgroups wait for each other,
// so it is a cooperative launch, or an ordinary one behind a gate (run_gate).
//
// What bounds a run of small or middle size is not the matrix cores but the
// chain of launches of a step (square, tail reduction, scalar step: 20 us a
// step at N = 100, of which the arithmetic is under 1 us) and, in between,
// K-range pieces that travel through memory. Here every workgroup stays on
// its CU for the whole run. The workgroups of one instance (its team) meet
// once per product: the first of the team sums the partials, takes the scalar
// step (finalize_scalar) and releases the others.
//
// Iterates are stored in operand order: blocks of 16 rows by 64 bytes (8
// FP64, 16 FP32 or 32 bf16 columns), 1 KiB each, lane l of a wave holding 16
// bytes of row l % 16, so that a wave reads an MFMA operand block as one
// contiguous KiB straight into registers. The main loop needs neither LDS nor
// barriers: each wave of a workgroup takes a part of the K range for the
// whole tile, and the parts meet in LDS once per tile.
//
// Measured on one MI355X, us a step (launch sequence -> resident, floor = the
// product at the rate of a large library product, 70 / 150 / 354 TFLOP/s):
//   FP64  N = 100: 20.3 -> 9.2   1000: 61 -> 35 (14)   2500: 391 -> 279 (223)
//         4096: 1124 -> 1068 (982)
//   FP32  100: 22.5 -> 9.2   1000: 42 -> 24 (7)   1777: 98 -> 70 (37)
//         3001: 290 -> 248 (180)   4000: 618 -> 525 (427)
//   BF16x3  100: 23 -> 9.1   1000: 43 -> 22 (3)   2500: 99 -> 92 (44)
// What is left at small N is the meeting of a team (4.5 us: stores seen by
// the other XCDs, the collection, the scalar step, the release) and the
// latency of the first operands after it; at N >= 2000 the tiles of the last
// round and the reduction and store of each tile (3 to 10 us, see plan_run).
// Matrix cores busy over a whole run: FP64 N = 1000 40 %, FP32 1777 57 %, 3001
// 69 %, 512 instances of 64 to 1024 rows 66 %, BF16x3 2500 (McWeeny) 23 %.
#pragma once

#include "square_impl.h"

namespace sp2 {
namespace {

typedef double doublex2 __attribute__((ext_vector_type(2)));

template <int P>
struct RunType;
template <>
struct RunType<0> {
  using T = double;
  using Vec = doublex2;
  using Op = doublex2;
  using AccV = doublex4;
};
template <>
struct RunType<1> {
  using T = float;
  using Vec = floatx4;
  using Op = floatx4;
  using AccV = floatx4;
};
template <>
struct RunType<2> {
  using T = float;
  using Vec = floatx4;
  using Op = bf16x8;
  using AccV = floatx4;
};

// Precision P, tiles of 16 MB rows, NW waves. SOLO: for single runs, one
// workgroup per CU where that buys registers. BRIEF: with the short chains.
template <int P_, int MB_, int NW_, bool SOLO, bool BRIEF_ = false>
struct RunCfg {
  static constexpr bool BRIEF = BRIEF_;
  static constexpr int P = P_, MB = MB_, NW = NW_;
  using T = typename RunType<P>::T;
  using Vec = typename RunType<P>::Vec;
  using Op = typename RunType<P>::Op;
  using AccV = typename RunType<P>::AccV;
  static constexpr int BM = 16 * MB, THREADS = 64 * NW;
  static constexpr int V = 16 / sizeof(T);         // elements of a vector
  static constexpr int KC = 64 / sizeof(T);        // columns of a block of X
  static constexpr int KO = (P == 2) ? 32 : KC;    // ... of an operand block
  static constexpr int NBC = BM / KC;              // block columns of a tile
  static constexpr int NBLK = MB * NBC;            // blocks of a tile
  static constexpr int NBW = (NBLK + NW - 1) / NW; // ... of a wave
  // LDS row stride of the tile: 16-byte rows; FP32: 4 LD = 16 mod 64 banks,
  // so that the four row groups of an accumulator fall on distinct banks
  static constexpr int LD = (P == 0) ? BM + 2 : BM + 4;
  static constexpr int SLOT = BM * LD;             // elements per K part
  // one slot of LDS per K part (two for the largest FP64 tile: its upper
  // waves hand their parts over first); the small tiles leave room for a
  // second workgroup on the CU, in registers as well
  static constexpr int R = (P == 0 && MB == 4) ? NW / 2 : NW;
  static constexpr int SMEM = R * SLOT * static_cast<int>(sizeof(T));
  // waves per SIMD the registers are budgeted for: one where the two sets of
  // accumulators need more than half of them
  static constexpr int WAVES = (SOLO && P == 1 && MB >= 4) ? 1 : 2;
  static_assert(SMEM <= (MB <= 4 ? 78 : 156) * 1024, "LDS of a CU");
  // every operand block lies within the padded matrix
  static_assert(BM % KO == 0, "whole operand blocks per tile");
  // operand sets in flight
  static constexpr int DEPTH = (P == 2) ? (MB >= 3 ? 2 : 4) : (MB == 2 ? 6 : (MB == 4 && WAVES == 2 ? 2 : 3));
  // the old values are loaded before the main loop and the next tile's first
  // sets before the epilogue, where the registers hold them
  static constexpr bool AHEAD = (P == 1 && (MB <= 3 || WAVES == 1)) || MB <= 2;
  // FP64 (where the registers allow) and FP32: after CHAIN blocks of columns
  // the running sums go into a second set of accumulators, so that rounding
  // grows with the chain and not with the wave's whole K part
  static constexpr bool TWO = (P == 0) ? MB <= 3 : P == 1;
  static constexpr int CHAIN = (8 + DEPTH - 1) / DEPTH * DEPTH;   // blocks
  // or, in the kernels of small single runs (kRunShortN), after three
  static constexpr int SHORT = 3;
  static_assert(!BRIEF || (TWO && DEPTH % SHORT == 0), "whole chains per round");
  struct Acc {
    AccV c[MB][MB];
  };
};

__device__ __forceinline__ int run_uni(int x) {
  return __builtin_amdgcn_readfirstlane(x);
}

// ------------------------------------------------------------- main loop
// Operands of one K block of a tile: FP64 and FP32 straight from the iterate,
// BF16x3 from its split (H and L).
template <class C>
struct RunSet {
  static constexpr int NS = (C::P == 2) ? 2 : 1;
  typename C::Op a[NS][C::MB], b[NS][C::MB];
};

// One wave's part of the K blocks of tile (I, J): A_I B_J^T.
template <class C>
struct RunTile {
  static constexpr int MB = C::MB;
  static constexpr int NS = RunSet<C>::NS;
  static constexpr int EB = (C::P == 2) ? 512 : 16 * C::KC;   // elements of a block
  using E = typename std::conditional<C::P == 2, __bf16, typename C::T>::type;
  const E *ap[NS], *bp[NS];
  size_t kbs;
  int k0, k1, lo;

  __device__ __forceinline__ RunTile(const typename C::T* A, const typename C::T* B,
                                     const __bf16* AH, const __bf16* AL, const __bf16* BH,
                                     const __bf16* BL, int ld, int I, int J, int kb,
                                     int wave) {
    kbs = static_cast<size_t>(ld / C::KO);
    k0 = run_uni(wave * kb / C::NW);
    k1 = run_uni((wave + 1) * kb / C::NW);
    lo = (threadIdx.x & 63) * static_cast<int>(16 / sizeof(E));
    const size_t ao = static_cast<size_t>(I) * MB * kbs * EB;
    const size_t bo = static_cast<size_t>(J) * MB * kbs * EB;
    if constexpr (C::P == 2) {
      ap[0] = AH + ao;
      ap[1] = AL + ao;
      bp[0] = BH + bo;
      bp[1] = BL + bo;
    } else {
      ap[0] = A + ao;
      bp[0] = B + bo;
    }
  }

  __device__ __forceinline__ void load(RunSet<C>& o, int k) const {
    k = min(k, k1 - 1);   // past the end: a re-read that nothing uses
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
      for (int m = 0; m < MB; ++m)
        o.a[s][m] = *gro(reinterpret_cast<const typename C::Op*>(
            ap[s] + (m * kbs + k) * EB + lo));
#pragma unroll
      for (int m = 0; m < MB; ++m)
        o.b[s][m] = *gro(reinterpret_cast<const typename C::Op*>(
            bp[s] + (m * kbs + k) * EB + lo));
    }
  }

  // The first sets, issued ahead of the main loop (and of the epilogue of
  // the tile before). A wave without K blocks loads nothing.
  __device__ __forceinline__ void begin(RunSet<C> (&o)[C::DEPTH]) const {
    if (k0 >= k1) return;
#pragma unroll
    for (int d = 0; d < C::DEPTH; ++d) {
      load(o[d], k0 + d);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
};

template <class C>
__device__ __forceinline__ void run_main(const RunTile<C>& tile, RunSet<C> (&o)[C::DEPTH],
                                         int chain, typename C::Acc& acc) {
  constexpr int MB = C::MB;
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < MB; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc.c[m][n][j] = 0;
  const int k0 = tile.k0, k1 = tile.k1;
  if (k0 >= k1) return;
  auto mma = [&](const RunSet<C>& o) {
    if constexpr (C::P == 2) {
#pragma unroll
      for (int t = 0; t < 3; ++t)   // H H, H L, L H
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int n = 0; n < MB; ++n)
            acc.c[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                o.a[t == 2 ? 1 : 0][m], o.b[t == 1 ? 1 : 0][n], acc.c[m][n], 0, 0, 0);
    } else {
#pragma unroll
      for (int e = 0; e < C::V; ++e)
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int n = 0; n < MB; ++n) {
            if constexpr (C::P == 0)
              acc.c[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                  o.a[0][m][e], o.b[0][n][e], acc.c[m][n], 0, 0, 0);
            else
              acc.c[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                  o.a[0][m][e], o.b[0][n][e], acc.c[m][n], 0, 0, 0);
          }
    }
  };
  constexpr int D = C::DEPTH;
  int k = k0;
  // f(d) after the products of set d
  auto rounds = [&](int end, auto f) {
    for (; k + D <= end; k += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        mma(o[d]);
        tile.load(o[d], k + d + D);
        __builtin_amdgcn_sched_barrier(0);
        f(d);
      }
    }
  };
  auto rest = [&](auto f) {
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
      if (k + d < k1) {
        mma(o[d]);
        f(d);
      }
  };
  auto none = [](int) {};
  if constexpr (C::TWO) {
    typename C::Acc sum = acc;
    auto flush = [&]() {
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < MB; ++n) {
          sum.c[m][n] += acc.c[m][n];
#pragma unroll
          for (int j = 0; j < 4; ++j) acc.c[m][n][j] = 0;
        }
    };
    if constexpr (C::BRIEF) {
      auto each = [&](int d) {
        if ((d + 1) % C::SHORT == 0) flush();
      };
      rounds(k1, each);
      rest(each);
    } else {
      while (k1 - k > chain) {
        rounds(k + chain, none);
        flush();
      }
      rounds(k1, none);
      rest(none);
    }
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int n = 0; n < MB; ++n) acc.c[m][n] += sum.c[m][n];
  } else {
    rounds(k1, none);
    rest(none);
  }
}

// --------------------------------------------------------------- epilogue
// Stores that write through to where every XCD sees them (cache policy SC1,
// the agent scope of the memory model): once they are counted complete, the
// team can be told with a plain word. A release fence instead would write
// back the whole L2 of the XCD, once per workgroup.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t run_out(void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, 0xffffffffu, 0x00027000);
}
constexpr int kWriteThrough = 16;
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));
template <typename Vec>
__device__ __forceinline__ void run_store16(__amdgpu_buffer_rsrc_t r, size_t elem, Vec v) {
  __builtin_amdgcn_raw_buffer_store_b128(
      __builtin_bit_cast(uintx4, v), r,
      static_cast<int>(static_cast<unsigned>(elem * sizeof(v[0]))), 0, kWriteThrough);
}
__device__ __forceinline__ void run_store8(__amdgpu_buffer_rsrc_t r, size_t elem, bf16x4 v) {
  __builtin_amdgcn_raw_buffer_store_b64(
      __builtin_bit_cast(uintx2, v), r, static_cast<int>(static_cast<unsigned>(elem * 2)), 0,
      kWriteThrough);
}
// The split of a vector of the output at (row, col).
template <class C>
__device__ __forceinline__ void run_split(__amdgpu_buffer_rsrc_t Yh,
                                          __amdgpu_buffer_rsrc_t Yl, int row, int col,
                                          int ld, floatx4 v) {
  bf16x4 hi, lo;
  split_bf16(v, hi, lo);
  const size_t o = op_off<__bf16>(row, col, ld);
  run_store8(Yh, o, hi);
  run_store8(Yl, o, lo);
}

// Sums the K parts of the tile in LDS, applies the step's epilogue to the
// upper triangle and stores the tile and its transpose (for BF16x3 the
// transpose of the split only: nothing reads the FP32 lower triangle).
// old: the step's stored matrix X, or in mode 2 the square S, at this wave's
// blocks.
template <class C>
struct RunOld {
  typename C::Vec v[C::NBW];
  __device__ __forceinline__ void load(const typename C::T* M, int ld, int I, int J,
                                       int wave) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < C::NBW; ++q) {
      const int b = min(wave + q * C::NW, C::NBLK - 1);
      v[q] = *gro(reinterpret_cast<const typename C::Vec*>(
          M + op_off<typename C::T>(I * C::BM + 16 * (b / C::NBC) + (lane & 15),
                                    J * C::BM + C::KC * (b % C::NBC) + C::V * (lane >> 4),
                                    ld)));
    }
  }
};

template <class C, int MODE>
__device__ __forceinline__ void run_epi(const RunOld<C>& old, __amdgpu_buffer_rsrc_t Y,
                                        __amdgpu_buffer_rsrc_t Yh,
                                        __amdgpu_buffer_rsrc_t Yl,
                                        int ld, int n, int I, int J, int wave,
                                        typename C::Acc& acc, const Coef<typename C::T>& kf,
                                        double tau, char* smem, Sums& sums) {
  using T = typename C::T;
  using Vec = typename C::Vec;
  constexpr int BM = C::BM, LD = C::LD, V = C::V;
  T* S = reinterpret_cast<T*>(smem);
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const bool diag = (I == J);
  // calls f on every accumulator and its place in a slot
  auto each = [&](int slot, auto f) {
    T* p = S + slot * C::SLOT;
#pragma unroll
    for (int m = 0; m < C::MB; ++m)
#pragma unroll
      for (int nn = 0; nn < C::MB; ++nn)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int rr = 16 * m + (C::P == 0 ? g + 4 * j : 4 * g + j);
          f(p[rr * LD + 16 * nn + r], m, nn, j);
        }
  };
  auto put = [&](T& x, int m, int nn, int j) { x = acc.c[m][nn][j]; };
  __syncthreads();   // the previous tile's reads of S are done
  if constexpr (C::R < C::NW) {
    static_assert(C::NW == 2 * C::R, "one hand-over");
    if (wave >= C::R) each(wave - C::R, put);
    __syncthreads();
    if (wave < C::R)
      each(wave, [&](T& x, int m, int nn, int j) { x += acc.c[m][nn][j]; });
  } else {
    each(wave, put);
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < C::NBW; ++q) {
    const int b = wave + q * C::NW;
    if (b >= C::NBLK) continue;
    const int lr = 16 * (b / C::NBC) + r, lc = C::KC * (b % C::NBC) + V * g;
    const int gr = I * BM + lr, gc = J * BM + lc;
    T* s0 = S + lr * LD + lc;
    Vec s = *reinterpret_cast<const Vec*>(s0);
#pragma unroll
    for (int w = 1; w < C::R; ++w)
      s += *reinterpret_cast<const Vec*>(s0 + w * C::SLOT);
    Vec xn;
#pragma unroll
    for (int e = 0; e < V; ++e) {
      double d2;
      if (!diag) {
        xn[e] = epilogue_elem<T, MODE>(s[e], MODE != 2 ? old.v[q][e] : T(0),
                                       MODE == 2 ? old.v[q][e] : T(0), kf, tau, 2.0,
                                       false, sums, d2);
      } else if (gr <= gc + e) {
        const bool on = (gr == gc + e);
        const T x = epilogue_elem<T, MODE>(s[e], MODE != 2 ? old.v[q][e] : T(0),
                                           MODE == 2 ? old.v[q][e] : T(0), kf, tau,
                                           on ? 1.0 : 2.0, on && gr < n, sums, d2);
        s0[e] = x;
        S[(lc + e) * LD + lr] = x;
      }
    }
    if (!diag) {
      run_store16(Y, op_off<T>(gr, gc, ld), xn);
      if constexpr (C::P == 2) run_split<C>(Yh, Yl, gr, gc, ld, xn);
      *reinterpret_cast<Vec*>(s0) = xn;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < C::NBW; ++q) {
    const int b = wave + q * C::NW;
    if (b >= C::NBLK) continue;
    const int lr = 16 * (b / C::NBC) + r, lc = C::KC * (b % C::NBC) + V * g;
    // row lr of the transposed tile: column lr of the tile (a diagonal tile
    // is symmetric by now)
    const int gr = J * BM + lr, gc = I * BM + lc;
    Vec v;
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = S[(lc + e) * LD + lr];
    if (diag || C::P != 2)
      run_store16(Y, op_off<T>(gr, gc, ld), v);
    if constexpr (C::P == 2) run_split<C>(Yh, Yl, gr, gc, ld, v);
  }
}

// ----------------------------------------------------------- affine start
// X_0 (f0_kernel's arithmetic) in operand order: the blocks of the padded
// matrix are dealt to the waves of the team; returns this thread's traces.
template <class C>
__device__ __forceinline__ void run_start(const Instance& in, int np, int rank, int size,
                                          int wave, Sums& sums) {
  using T = typename C::T;
  using Vec = typename C::Vec;
  const int lane = threadIdx.x & 63;
  const int n = in.n, ld = in.ld;
  const double* F = in.F;
  const int64_t ldf = in.ldf;
  const double lmax = in.lmax, width = in.width, tau = in.tau;
  const int n_occ = static_cast<int>(in.prm.n_occ);
  const int trivial = (n_occ == 0) ? 1 : (n_occ == n ? 2 : 0);
  const OpMap m1 = step_map(in, 1);
  const bool stretch = !trivial && (m1.a != 1.0 || m1.c != 0.0);
  const auto X = run_out(in.X[0]), XH = run_out(in.XH[0]), XL = run_out(in.XL[0]);
  const int kbs = ld / C::KC;
  const int nblk = np / 16 * kbs;
  constexpr int U = 4;   // blocks whose loads are in flight together
  const int stride = size * C::NW;
  for (int b0 = rank * C::NW + wave; b0 < nblk; b0 += stride * U) {
    double f[U][C::V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int b = b0 + u * stride;
      const int row = 16 * (b / kbs) + (lane & 15);
      const int col = C::KC * (b % kbs) + C::V * (lane >> 4);
#pragma unroll
      for (int e = 0; e < C::V; ++e)
        f[u][e] = (b < nblk && row < n && col + e < n && !trivial)
                      ? *gro(F + static_cast<int64_t>(row) * ldf + col + e)
                      : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int b = b0 + u * stride;
      if (b >= nblk) continue;
      const int row = 16 * (b / kbs) + (lane & 15);
      const int col = C::KC * (b % kbs) + C::V * (lane >> 4);
      Vec v;
#pragma unroll
      for (int e = 0; e < C::V; ++e) {
        const int j = col + e;
        double x = 0.0;
        if (row < n && j < n) {
          if (trivial) {
            x = (trivial == 2 && row == j) ? 1.0 : 0.0;
          } else {
            x = ((row == j) ? lmax - f[u][e] : -f[u][e]) / width;
            if (fabs(x) < tau) x = 0.0;
          }
        }
        const T xt = static_cast<T>(x);
        const double xd = static_cast<double>(xt);
        v[e] = stretch ? static_cast<T>(__builtin_fma(
                             m1.a, xd, (row == j && row < n) ? m1.c : 0.0))
                       : xt;
        sums.t2 += xd * xd;
        if (row == j) sums.t1 += xd;
      }
      run_store16(X, op_off<T>(row, col, ld), v);
      if constexpr (C::P == 2) run_split<C>(XH, XL, row, col, ld, v);
    }
  }
}

// ------------------------------------------------------------------ kernel
// Waits until *w reaches `want`; returns the word, or -1 past the limit (the
// error flag then makes every workgroup give up).
__device__ __forceinline__ int run_wait(const int32_t* w, int want, int32_t* err,
                                        long long limit) {
  const long long t0 = wall_clock64();
  for (;;) {
    const int v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (v >= want) return v;
    if (wall_clock64() - t0 > limit ||
        __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
      __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return -1;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

// The gate of an ordinary launch, which the device does not promise to place
// as a whole: open once every workgroup has arrived, shut by the first that
// waits too long (the others may wait for room that a run like this one
// holds). Nothing has been done before it, so a shut run can be launched anew.
__device__ __forceinline__ int run_gate(int32_t* gate, int members, long long limit) {
  int free = 0;
  const int k = __hip_atomic_fetch_add(gate, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (k == members - 1)
    __hip_atomic_compare_exchange_strong(gate + 1, &free, kGateOpen, __ATOMIC_RELAXED,
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const long long t0 = wall_clock64();
  for (;;) {
    const int g = __hip_atomic_load(gate + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (g != 0) return g;
    if (wall_clock64() - t0 > limit) {
      free = 0;
      __hip_atomic_compare_exchange_strong(gate + 1, &free, kGateShut, __ATOMIC_RELAXED,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// What a workgroup tells its team's first: its partial sums and the number
// of the phase they belong to.
__device__ __forceinline__ double run_peek(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <class C, bool MW>
__global__ __launch_bounds__(C::THREADS, C::WAVES) void run_kernel(RunArgs a) {
  using T = typename C::T;
  __shared__ __attribute__((aligned(16))) char smem[C::SMEM];
  __shared__ double sh[C::NW][3];
  __shared__ int word;
  const auto* seat = cro(a.seats + blockIdx.x);
  const int rank = seat->rank, size = seat->size, base = seat->base, team = seat->team;
  if (size == 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = run_uni(tid >> 6);
  if (a.members > 0) {
    if (tid == 0) word = run_gate(a.gate, a.members, a.gate_limit);
    __syncthreads();
    const int g = word;
    __syncthreads();   // word may be rewritten only after every read
    if (g != kGateOpen) return;
  }
  const bool affine = a.stretch != 0;
  double* const ec = a.coef + 8 * team;   // StepCoef of the next product
  int32_t* const flag = a.flag + 32 * team;
  int phase = 0;
  int inst = seat->inst;
  for (;;) {
  const Instance& gin = a.inst[inst];
  const auto* in = cro(a.inst + inst);
  DevState* const st = in->st;
  const int n = in->n, ld = in->ld;
  const int tile0 = in->tile0, ntiles = in->ntiles;
  const double tau = in->tau;
  T* const Xb[2] = {static_cast<T*>(in->X[0]), static_cast<T*>(in->X[1])};
  __bf16* const Hb[2] = {static_cast<__bf16*>(in->XH[0]), static_cast<__bf16*>(in->XH[1])};
  __bf16* const Lb[2] = {static_cast<__bf16*>(in->XL[0]), static_cast<__bf16*>(in->XL[1])};
  T* const Sq = static_cast<T*>(in->S);
  __bf16* const SH = static_cast<__bf16*>(in->SH);
  __bf16* const SL = static_cast<__bf16*>(in->SL);
  const int kb = (n + C::KO - 1) / C::KO;
  const int chain = (C::P == 0 && n > a.chain_n) ? kb : C::CHAIN;
  const int np = (n + C::BM - 1) / C::BM * C::BM;
  // tiles of this workgroup: rank, rank + size, ... over the whole rounds,
  // then its tile of the incomplete last round, if it has one
  const int whole = ntiles / size * size;
  const int last_tile = a.npull ? whole + rank : seat->last;
  auto first_tile = [&]() { return whole > 0 ? rank : last_tile; };
  auto next_tile = [&](int t) {
    return t + size < whole ? t + size : (t < whole ? last_tile : ntiles);
  };

  // The team meets. Every workgroup posts its partial sums and the phase;
  // the first of the team collects them, takes the scalar step of `iter`
  // (unless scalar is false) and publishes the word 4 phase + 2 p + done.
  // Returns that word, or -1 after a wait past its limit. All of it is
  // written through, so the only fence is the acquire that drops what the
  // caches hold of the old iterate.
  auto meet = [&](bool scalar, int iter, Sums s) -> int {
    ++phase;
    RunPost* const post = a.post + base;
    if (scalar) {
      s.v = wave_sum(s.v);
      s.t1 = wave_sum(s.t1);
      s.t2 = wave_sum(s.t2);
      if (lane == 0) {
        sh[wave][0] = s.v;
        sh[wave][1] = s.t1;
        sh[wave][2] = s.t2;
      }
      __syncthreads();
      if (tid < 3) {
        double t = sh[0][tid];
        for (int w = 1; w < C::NW; ++w) t += sh[w][tid];
        __hip_atomic_store(&post[rank].sum[tid], t, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    // every wave's stores are complete before the phase is posted
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (rank != 0) {
      if (tid == 0) {
        __hip_atomic_store(&post[rank].phase, phase, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        word = run_wait(flag, 4 * phase, a.err, a.wait_limit);
      }
    } else {
      double pv = 0.0, p1 = 0.0, p2 = 0.0;
      bool ok = true;
      for (int i = tid; i < size; i += C::THREADS) {
        if (i > 0 && run_wait(&post[i].phase, phase, a.err, a.wait_limit) < 0) ok = false;
        asm volatile("" ::: "memory");   // the sums after the phase
        if (scalar) {
          pv += run_peek(&post[i].sum[0]);
          p1 += run_peek(&post[i].sum[1]);
          p2 += run_peek(&post[i].sum[2]);
        }
      }
      if (scalar) {
        pv = wave_sum(pv);
        p1 = wave_sum(p1);
        p2 = wave_sum(p2);
        if (lane == 0) {
          sh[wave][0] = pv;
          sh[wave][1] = p1;
          sh[wave][2] = p2;
        }
      }
      ok = __syncthreads_and(ok);
      if (tid == 0) {
        word = -1;
        if (ok) {
          word = 4 * phase;
          if (scalar) {
            for (int w = 1; w < C::NW; ++w) {
              pv += sh[w][0];
              p1 += sh[w][1];
              p2 += sh[w][2];
            }
            const bool done = persist_finalize(gin, iter, pv, p1, p2, a.ndone, a.count, nullptr);
            word += (st->p[iter + 1] != 0 ? 2 : 0) + (done ? 1 : 0);
            if (affine) {
              for (int q = 0; q < 5; ++q)
                __hip_atomic_store(ec + q, st->ecoef[q], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
              __builtin_amdgcn_s_waitcnt(0);
            }
          }
          if (size > 1)
            __hip_atomic_store(flag, word, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    if (tid == 0 && (size > 1 || affine)) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __syncthreads();
    const int w = word;
    __syncthreads();   // word may be rewritten only after every read
    return run_uni(w);
  };

  Sums sums;
  // One product over this workgroup's tiles: A B^T with the epilogue of MODE
  // on `old`, into Y. The first operands of the next tile are loaded before
  // the epilogue of the current one.
  auto product = [&](auto mode, const T* A, const __bf16* AH, const __bf16* AL, const T* B,
                     const __bf16* BH, const __bf16* BL, const T* old, T* Y, __bf16* Yh,
                     __bf16* Yl, const Coef<T>& kf, double tq) {
    constexpr int MODE = decltype(mode)::value;
    int t = first_tile();
    if (t >= ntiles) return;
    const auto y = run_out(Y), yh = run_out(Yh), yl = run_out(Yl);
    RunSet<C> sets[C::DEPTH];
    int2 tt = {cro(a.tiles + tile0 + t)->x, cro(a.tiles + tile0 + t)->y};
    RunTile<C> tile(A, B, AH, AL, BH, BL, ld, tt.x, tt.y, kb, wave);
    if (C::AHEAD) tile.begin(sets);
    for (;;) {
      if (!C::AHEAD) tile.begin(sets);
      RunOld<C> was;
      if (C::AHEAD) was.load(old, ld, tt.x, tt.y, wave);
      typename C::Acc acc;
      run_main<C>(tile, sets, chain, acc);
      if (!C::AHEAD) was.load(old, ld, tt.x, tt.y, wave);
      const int2 at = tt;
      t = next_tile(t);
      const bool more = t < ntiles;
      if (more) {
        tt = {cro(a.tiles + tile0 + t)->x, cro(a.tiles + tile0 + t)->y};
        tile = RunTile<C>(A, B, AH, AL, BH, BL, ld, tt.x, tt.y, kb, wave);
        if (C::AHEAD) tile.begin(sets);
      }
      run_epi<C, MODE>(was, y, yh, yl, ld, n, at.x, at.y, wave, acc, kf, tq, smem, sums);
      if (!more) break;
    }
  };

  run_start<C>(gin, np, rank, size, wave, sums);
  int w = meet(true, 0, sums);
  for (int iter = 1; w >= 0 && !(w & 1); ++iter) {
    const int cur = (iter - 1) & 1, nxt = iter & 1;
    const T* X = Xb[cur];
    sums = Sums{};
    if constexpr (!MW) {
      const bool p1 = (w & 2) != 0;
      const Coef<T> kf{p1 ? T(1) : T(-1), p1 ? T(0) : T(2), T(0), 0, affine, ec};
      product(std::integral_constant<int, 0>{}, X, Hb[cur], Lb[cur], X, Hb[cur], Lb[cur], X,
              Xb[nxt], Hb[nxt], Lb[nxt], kf, tau);
    } else {
      const Coef<T> k1{T(1), T(0), T(0), 1, affine, ec};
      product(std::integral_constant<int, 1>{}, X, Hb[cur], Lb[cur], X, Hb[cur], Lb[cur], X,
              Sq, SH, SL, k1, 0.0);
      if (meet(false, iter, sums) < 0) return;
      const Coef<T> k2{T(-2), T(0), T(3), 2, affine, ec};
      product(std::integral_constant<int, 2>{}, X, Hb[cur], Lb[cur], Sq, SH, SL, Sq, Xb[nxt],
              Hb[nxt], Lb[nxt], k2, tau);
    }
    w = meet(true, iter, sums);
  }
  if (w < 0 || a.npull == 0) return;
  // A team of a batch takes the next instance of the list. Its number has a
  // word of its own: nobody has posted since the release word, which a slower
  // member may still be about to read.
  ++phase;
  if (tid == 0) {
    int next = 0;
    if (rank == 0) {
      const int k = __hip_atomic_fetch_add(a.next, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      next = (k < a.npull) ? a.pull[k] : -1;
      if (size > 1) {
        __hip_atomic_store(flag + 1, next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0);
        __hip_atomic_store(flag + 2, phase, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    } else {
      next = (run_wait(flag + 2, phase, a.err, a.wait_limit) < 0) ? -1 : 0;
      asm volatile("" ::: "memory");
      if (next == 0)
        next = __hip_atomic_load(flag + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    word = next;
  }
  __syncthreads();
  inst = run_uni(word);
  __syncthreads();
  if (inst < 0) return;
  }
}

template <class C>
const void* run_fn(bool mw) {
  return mw ? reinterpret_cast<const void*>(&run_kernel<C, true>)
            : reinterpret_cast<const void*>(&run_kernel<C, false>);
}

}  // namespace
}  // namespace sp2
