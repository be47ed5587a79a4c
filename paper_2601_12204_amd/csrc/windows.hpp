// Windows of chunks of a long system: device code shared by the forward solvers (window.hip, and btcs.hip where a
// system beyond the windows' bound comes within it) and the adjoint.
#pragma once

#include <hip/hip_runtime.h>

#include "interface.hpp"
#include "internal.hpp"
#include "staging.hpp"
#include "stencil.hpp"

#pragma clang fp contract(off)

namespace burgers {

constexpr int kChunkRows = 16;     // rows (slots) of a window's chunk
constexpr int kMaxPcr = 4;         // PCR steps of a window's solve at most
constexpr int kStepHalo = 1 << kMaxPcr;   // chunks lost at either end of a window over one step
constexpr int kDeepLanes = 512;
// Chunks lost at either end of a window over a launch of several steps: 24, 12, 6 or 3 of them with S = 1 to 4, at ten
// times the CFL step 12 or 6.  (One grid of 2^24 rows, 128 steps / 10^4 ragged problems, ms: 32 chunks 3.16 / 19.9, 48:
// 3.18 / 19.4, 64: 3.32 / 19.5, repeated on a warm chip.)
constexpr int kDeepHalo = 48;

// Chunks of a system of R > 8192 rows: P = ceil(R / 16) of them, all of 16 rows but `lack` < 16 of 15 rows, the chunks
// 31, 63, 95, ... (P > 32 lack): no two of those are within 32 chunks of each other, around a periodic system too, so
// 2^S <= 16 consecutive chunks hold at least 16 2^S - 1 rows.
struct Chunks {
  int R, P, lack;
  __device__ __forceinline__ explicit Chunks(int rows)
      : R(rows), P((rows + kChunkRows - 1) / kChunkRows), lack(kChunkRows * P - rows) {}
  __device__ __forceinline__ bool lacks(int c) const { return (c & 31) == 31 && (c >> 5) < lack; }
  __device__ __forceinline__ int base(int c) const { return kChunkRows * c - (c >> 5 < lack ? c >> 5 : lack); }
  // rows of the run of n chunks from c on (c < P; the run may pass the end of a periodic system)
  __device__ __forceinline__ int rows(int c, int n) const {
    const int e = c + n;
    return e <= P ? base(e) - base(c) : R - base(c) + base(e - P);
  }
};

// ... and over a launch of reverse steps (10 of them with S = 3), whose windows take longer to load: three states a
// window of one workgroup per CU.  (256 x 16384 rows, us per reverse step: 48 chunks 21, 80: 18.)
constexpr int kAdjDeepHalo = 80;

// Steps of a call that launch `launch` takes on an instance with `pcr` PCR steps per solve, after `done`.
template <int HALO = kDeepHalo>
__device__ __forceinline__ int deep_steps(const ChunkWin& w, int pcr, int launch, int nsteps, int& done) {
  const int per = HALO >> pcr, total = w.limit > 0 && w.limit < nsteps ? w.limit : nsteps;
  done = launch * per;
  return done >= total ? 0 : (total - done < per ? total - done : per);
}

// Interface solve of a window of L chunks, lane t < L holding chunk t (see interface_solve; the first chunk has
// no coupling to its left, the last none to its right).  A partner beyond the ends is replaced by the end
// chunk: its coefficient is zero there.
template <int NT, bool LdsOnly = false>
__device__ __forceinline__ void window_solve(const InterfaceSpace<double, NT>& w, int L, int S, bool own, double al0,
                                             double ga0, double de0, double alL, double gaL, double deL, double ia,
                                             double ib, double ic, double id, double& y, double& yp) {
  const int t = threadIdx.x;
  constexpr int kV = InterfaceSpace<double, NT>::kVoteWords;
  if (own) {
    w.xchg[t] = al0;
    w.xchg[NT + t] = ga0;
    w.xchg[2 * NT + t] = de0;
  }
  wg_barrier<LdsOnly>();
  double a = 0.0, c = 0.0, d = 0.0;
  bool live = false;
  if (own) {
    const int n = t + 1 < L ? t + 1 : t;
    const double nal = w.xchg[n], nga = w.xchg[NT + n], nde = w.xchg[2 * NT + n];
    const double inv = recip(__builtin_fma(-ic, nal, __builtin_fma(-ia, gaL, ib)));
    a = -(ia * alL) * inv;
    c = -(ic * nga) * inv;
    d = __builtin_fma(-ic, nde, __builtin_fma(-ia, deL, id)) * inv;
    live = (__builtin_fabs(a) + __builtin_fabs(c)) > kNegligible;
    a = live ? a : 0.0;
    c = live ? c : 0.0;
    w.rows[t] = a;
    w.rows[NT + t] = c;
    w.rows[2 * NT + t] = d;
  }
  wg_barrier<LdsOnly>();
  int b = 0;
  bool done = false;
  for (int i = 0; i < S && !done; ++i) {
    const double* A = w.rows + b * 3 * NT;
    const double* C = A + NT;
    const double* D = C + NT;
    if (own) {
      if (live) {
        const int s = 1 << i;
        const int mi = t >= s ? t - s : 0, pi = t + s < L ? t + s : L - 1;
        pcr_combine(a, c, d, A[mi], C[mi], D[mi], A[pi], C[pi], D[pi], a, c, d);
        live = (__builtin_fabs(a) + __builtin_fabs(c)) > kNegligible;
        a = live ? a : 0.0;
        c = live ? c : 0.0;
      }
      double* nA = w.rows + (1 - b) * 3 * NT;
      nA[t] = a;
      nA[NT + t] = c;
      nA[2 * NT + t] = d;
    }
    const bool wave_live = __ballot(live) != 0;
    if ((t & 63) == 0) reinterpret_cast<unsigned char*>(w.votes + (1 - b) * kV)[t >> 6] = wave_live ? 1 : 0;
    wg_barrier<LdsOnly>();
    b = 1 - b;
    uint64_t any = 0;
#pragma unroll
    for (int k = 0; k < kV; ++k) any |= w.votes[b * kV + k];
    done = any == 0;
  }
  // (couplings left after S steps are dropped: at most theta^(n_S))
  y = d;
  yp = own ? w.rows[b * 3 * NT + 2 * NT + (t > 0 ? t - 1 : 0)] : 0.0;
}

// ---- Steps on windows (forward) ------------------------------------------------------------------------

__host__ __device__ __forceinline__ double theta_bound(const InstDesc& d, double M) {
  const double C = d.r * M;
  return 2.0 * (d.D + C) / ((1.0 + 2.0 * d.D + C) + __builtin_sqrt((1.0 + C) * (1.0 + C) + 4.0 * d.D));
}

// A running maximum of |v|, infinite once a value is not finite, so that its instance fails the bound (`zero` turns into
// a NaN then, which the maximum itself would pass over).
template <typename S>
struct Magnitude {
  S big = S(0), zero = S(0);
  __device__ __forceinline__ void take(S v) {
    if constexpr (sizeof(S) == 8) {
      big = __builtin_fmax(big, __builtin_fabs(v));
      zero = __builtin_fma(v, 0.0, zero);
    } else {
      big = __builtin_fmaxf(big, __builtin_fabsf(v));
      zero = __builtin_fmaf(v, 0.0f, zero);
    }
  }
  __device__ __forceinline__ double value() const { return zero == S(0) ? static_cast<double>(big) : __builtin_inf(); }
};

// LDS of a window: its rows staged between HBM and the lanes, overlaid by the interface solve.
template <typename S, int NT>
struct WindowSpace {
  static constexpr int kStageBytes = padded_size(NT * kChunkRows) * static_cast<int>(sizeof(S));
  static constexpr int kIface = InterfaceSpace<double, NT>::kBytes;
  static constexpr int kBytes = kStageBytes > kIface ? kStageBytes : kIface;
};

// A window's place in its system.
struct Frame {
  Chunks ch;
  int r0, total;           // its first row and its rows
  __device__ __forceinline__ Frame(int R, const ChunkWin& w) : ch(R), r0(ch.base(w.first)), total(ch.rows(w.first, w.chunks)) {}
};

// The lane's chunk: its slots' first row counted from the window's, and its part in the solve.
__device__ __forceinline__ int window_lane(const Frame& f, const ChunkWin& w, int t, SlotLane& l) {
  int c = w.first + t, wrap = 0;
  if (c >= f.ch.P) {
    c -= f.ch.P;
    wrap = f.ch.R;
  }
  const bool dummy = f.ch.lacks(c);
  l.base = 0;
  l.own = t < w.chunks;
  l.dummy = dummy;
  l.first = t == 0;
  l.last = t == w.chunks - 1;
  l.tie = t == 0 ? 0.0 : -1.0;
  return f.ch.base(c) - (dummy ? 1 : 0) - f.r0 + wrap;   // (-1 for a first chunk of 15 rows)
}

// `steps` steps of a window's rows, from and to the staged rows; watch(de) sees the lane's rows before each of them.
template <typename S, int NT, typename Watch>
__device__ __forceinline__ void window_advance(const InterfaceSpace<double, NT>& ws, S* stage, const Frame& f,
                                               const ChunkWin& w, const InstDesc& d, int steps, int pcr, Watch&& watch) {
  const int t = threadIdx.x;
  SlotLane l;
  const int at = window_lane(f, w, t, l);
  const bool dir = d.bc == kDirichlet;
  const SlotRows rows{d.r, d.D, dir && w.first == 0 ? d.a : 0.0,
                      dir && w.first + w.chunks == f.ch.P ? d.b : 0.0};
  double al[kChunkRows], ga[kChunkRows], de[kChunkRows];
  // (a window without short chunks, as most are: its lanes' rows begin at multiples of 16, one address each)
  const bool plain = f.total == kChunkRows * w.chunks;
  if (plain) {
    const S* rows_at = stage + padded(kChunkRows * t);
#pragma unroll
    for (int j = 0; j < kChunkRows; ++j) de[j] = l.own ? static_cast<double>(rows_at[j]) : 0.0;
  } else {
#pragma unroll
    for (int j = 0; j < kChunkRows; ++j)
      de[j] = l.own ? static_cast<double>(stage[padded(j == 0 && at < 0 ? 0 : at + j)]) : 0.0;
  }
  __syncthreads();                           // every lane's rows read: the interface LDS overlays them
  for (int step = 0; step < steps; ++step) {
    watch(de);
    double ia = 0.0, ib = 1.0, ic = 0.0, id = 0.0, y, yp;
    if (l.own) slot_eliminate<kChunkRows, false>(rows, l, al, ga, de, ia, ib, ic, id);
    constexpr int k = kChunkRows - 2;
    window_solve<NT>(ws, w.chunks, pcr, l.own, l.dummy ? al[1] : al[0], l.dummy ? ga[1] : ga[0],
                     l.dummy ? de[1] : de[0], al[k], ga[k], de[k], ia, ib, ic, id, y, yp);
#pragma unroll
    for (int j = 0; j < kChunkRows; ++j)
      de[j] = static_cast<double>(static_cast<S>(slot_value<kChunkRows>(j, al, ga, de, yp, y)));
  }
  __syncthreads();                           // the interface unknowns read before the rows are rewritten
  SlotLane o;                                // (formed anew: not held across the solve)
  const int again = opaque_lane(t), to = window_lane(f, w, again, o);
  if (plain) {
    S* rows_at = stage + padded(kChunkRows * again);
#pragma unroll
    for (int j = 0; j < kChunkRows; ++j)
      if (o.own) rows_at[j] = static_cast<S>(de[j]);
  } else if (o.own) {
#pragma unroll
    for (int j = 0; j < kChunkRows; ++j)
      if (j > 0 || !o.dummy) stage[padded(to + j)] = static_cast<S>(de[j]);
  }
  __syncthreads();
}

// The window's rows into LDS, every load in flight at once; MAX: also their largest magnitude (the lane's).
template <typename S, int NT, bool MAX>
__device__ __forceinline__ double window_load(const S* __restrict__ x, S* stage, const Frame& f) {
  const int t = threadIdx.x;
  S v[kChunkRows];
  if (f.r0 + NT * kChunkRows <= f.ch.R) {      // (uniform) the rows from r0 on are there: one address
    const S* __restrict__ p = x + f.r0;
#pragma unroll
    for (int j = 0; j < kChunkRows; ++j) v[j] = p[t + j * NT];
  } else {
#pragma unroll
    for (int j = 0; j < kChunkRows; ++j) {
      const int i = t + j * NT;
      int k = f.r0 + (i < f.total ? i : f.total - 1);
      if (k >= f.ch.R) k -= f.ch.R;
      v[j] = x[k];
    }
  }
  Magnitude<S> m;                              // (rows beyond the window's at most raise it)
#pragma unroll
  for (int j = 0; j < kChunkRows; ++j) {
    if constexpr (MAX) m.take(v[j]);
    stage[padded(t + j * NT)] = v[j];
  }
  return m.value();
}

// The window's kept rows, put(row of the system, row of the window), of NT - 2 HALO chunks at most; the lane index is
// formed anew.
template <int NT, int HALO, typename Put>
__device__ __forceinline__ void window_kept(const Frame& f, const ChunkWin& w, Put&& put) {
  int c = w.first + w.lo;
  if (c >= f.ch.P) c -= f.ch.P;
  const int first = f.ch.base(c), count = f.ch.rows(c, w.count);
  const int from = first - f.r0 + (first < f.r0 ? f.ch.R : 0);
  const int t = opaque_lane(static_cast<int>(threadIdx.x));
#pragma unroll
  for (int j = 0; j < (kChunkRows * (NT - 2 * HALO) + NT - 1) / NT; ++j) {
    const int o = t + j * NT;
    if (o < count) put(first + o, from + o);   // (kept chunks of a window do not wrap)
  }
}

// The Dirichlet nodes next to the kept rows.
template <typename S>
__device__ __forceinline__ void window_ends(const Frame& f, const ChunkWin& w, const InstDesc& d, S* __restrict__ out) {
  if (d.bc != kDirichlet || threadIdx.x != 0) return;
  if (w.first + w.lo == 0) out[d.off] = static_cast<S>(d.a);
  if (w.first + w.lo + w.count == f.ch.P) out[d.off + d.n - 1] = static_cast<S>(d.b);
}

__device__ __forceinline__ int system_rows(const InstDesc& d) { return d.bc == kDirichlet ? d.n - 2 : d.n; }

template <int NT>
__device__ __forceinline__ double workgroup_max(double big, double* wave_max) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) big = __builtin_fmax(big, __shfl_xor(big, m, 64));
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = big;
  __syncthreads();
  double M = 0.0;
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) M = __builtin_fmax(M, wave_max[k]);
  return M;
}

}  // namespace burgers
