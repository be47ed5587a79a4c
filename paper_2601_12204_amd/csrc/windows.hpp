// Windows of chunks of a long system: device code shared by the forward solver (window.hip) and the adjoint.
#pragma once

#include <hip/hip_runtime.h>

#include "interface.hpp"
#include "internal.hpp"

#pragma clang fp contract(off)

namespace burgers {

constexpr int kChunkRows = 16;     // rows (slots) of a window's chunk
constexpr int kMaxPcr = 4;         // PCR steps of a window's solve at most
constexpr int kDeepLanes = 512;
// Chunks lost at either end of a window over a launch of several steps: with S = 3, the usual case at ten times
// the CFL step, 6 steps a launch (one grid of 2^24 rows, 128 steps: 32 chunks 3.48 ms, 48: 3.16, 64: 3.21).
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

}  // namespace burgers
