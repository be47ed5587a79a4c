// The interface partition of a tridiagonal system held by one workgroup: device code shared by the solvers
// that keep systems on chip and those that step them through HBM.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "stencil.hpp"
#include "wave.hpp"

#pragma clang fp contract(off)

namespace burgers {

// Reciprocal of a binary64 value to about one ulp: the hardware estimate r (relative error e = 1 - x r
// below 2^-24 on gfx950, measured) refined to third order, r (1 + e + e^2), whose remaining error e^3
// is below 2^-72: within one ulp of the correctly rounded reciprocal (99.98% equal to it over 4 M
// arguments), as two Newton steps are, in four instructions instead of five.  The solve only multiplies
// by reciprocals of pivots; in binary64 the resulting per-step bias stays near 1e-17 and does not show
// at the 1e-12 parity bar.
__device__ __forceinline__ double recip(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, __builtin_fma(e, e, e), r);
}

// Couplings below this fraction of a row's (unit) diagonal are negligible: dropping them changes a
// solution value by less than half an ulp of the largest value it couples to.
constexpr double kNegligible = 0x1p-54;

// Dirichlet values of a level-0 system: row 0 reads x_{-1} = a, row R-1 reads x_R = b.  In the reduced
// rows, x_{-1} enters only the chunk's F row (coefficient AF) and x_R only its E row (coefficient CE),
// so moving the known values to the right-hand side is DF -= AF a, AF = 0 and DE -= CE b, CE = 0.
struct DirichletEnds {
  double a, b;
  bool dirichlet;
  __device__ __forceinline__ void apply(int s, int m, int R, double& AF, double& DF, double& CE,
                                        double& DE) const {
    if (!dirichlet) return;
    if (s == 0) {
      DF = __builtin_fma(-AF, a, DF);
      AF = 0.0;
    }
    if (s + m == R) {
      DE = __builtin_fma(-CE, b, DE);
      CE = 0.0;
    }
  }
};

// Chunk layout of a system of R rows split into P chunks: sizes q or q+1, the longer ones first.
__device__ __forceinline__ void chunk_span(int k, int R, int P, int& s, int& m) {
  const int q = R / P, rho = R - q * P;
  s = k * q + (k < rho ? k : rho);
  m = q + (k < rho ? 1 : 0);
}

// One PCR step on a row normalised to a unit diagonal,  a x_{i-s} + x_i + c x_{i+s} = d,  with its two
// partners  x_{i-s} + cm x_i + ... = dm  (coefficients am, cm, dm) and  ap x_i + x_{i+s} + ... = dp:
// subtracting a times the first and c times the second leaves a row coupling x_{i-2s} and x_{i+2s},
// renormalised.
template <typename T>
__device__ __forceinline__ void pcr_combine(T a0, T c0, T d0, T am, T cm, T dm, T ap, T cp, T dp, T& na, T& nc,
                                            T& nd) {
  const T inv = recip(__builtin_fma(-c0, ap, __builtin_fma(-a0, cm, T(1))));
  const T a = a0 * inv, c = c0 * inv;
  na = -(a * am);
  nc = -(c * cp);
  nd = __builtin_fma(-c, dp, __builtin_fma(-a, dm, d0 * inv));
}

// ---- Interface partition of a whole system (the resident and the per-step workgroup solvers) ----------
//
// Lane t < P owns rows s..s+m-1 (m >= 2) of a system of R rows, and its last row is the chunk's interface
// unknown y_t = x_{s+m-1}.  The interior rows j = 0..m-2 lie between y_{t-1} (row s-1, the previous
// chunk's interface; cyclically for a periodic system) and y_t, so eliminating them expresses each as
//     x_j = de[j] - al[j] y_{t-1} - ga[j] y_t.
// Substituting into y_t's own row its two neighbours, x_{m-2} of this chunk and the first interior row
// of the next chunk (received from lane t+1), leaves one row per chunk,
//     A_t y_{t-1} + y_t + C_t y_{t+1} = D_t,
// a cyclic system of P rows solved by PCR with one row per lane.  A Dirichlet system moves its two
// boundary values into the right-hand sides of its first and last rows, which removes the couplings
// across its ends, so its interface system is not cyclic.  Compared with reducing every chunk to two
// rows (F, E), this halves the reduced system and replaces its first PCR step by one exchange between
// neighbouring lanes.

// Eliminates the interior rows and returns the interface row's coefficients (ia on the neighbour
// x_{m-2}, ib, ic on the row after the chunk, id).
template <typename T, int M, typename Src>
__device__ __forceinline__ void interface_eliminate(const Src& src, int s, int m, int R, T (&al)[M], T (&ga)[M],
                                                    T (&de)[M], T& ia, T& ib, T& ic, T& id) {
  const DirichletEnds& ends = src.ends;
#pragma unroll
  for (int j = 0; j < M; ++j) {
    if (j < m) {
      T aj, bj, cj, dj;
      src.row(j, s + j, R, aj, bj, cj, dj);
      if (j == 0 && ends.dirichlet && s == 0) {   // x_{-1} = a
        dj = __builtin_fma(-aj, static_cast<T>(ends.a), dj);
        aj = T(0);
      }
      if (j == m - 1) {
        if (ends.dirichlet && s + m == R) {        // x_R = b
          dj = __builtin_fma(-cj, static_cast<T>(ends.b), dj);
          cj = T(0);
        }
        ia = aj;
        ib = bj;
        ic = cj;
        id = dj;
      } else if (j == 0) {
        const T inv = recip(bj);
        al[0] = aj * inv;
        ga[0] = cj * inv;
        de[0] = dj * inv;
      } else {
        const T inv = recip(__builtin_fma(-aj, ga[j - 1], bj));
        const T ai = aj * inv;
        al[j] = -(ai * al[j - 1]);
        ga[j] = cj * inv;
        de[j] = __builtin_fma(-ai, de[j - 1], dj * inv);
      }
    }
  }
  // backward: the coupling to x_{j+1} becomes a coupling to y_t (row m-2 already has this form)
#pragma unroll
  for (int j = M - 3; j >= 0; --j) {
    if (j <= m - 3) {
      const T g = ga[j];
      de[j] = __builtin_fma(-g, de[j + 1], de[j]);
      al[j] = __builtin_fma(-g, al[j + 1], al[j]);
      ga[j] = -(g * ga[j + 1]);
    }
  }
}

// Workgroup barrier.  LdsOnly: for exchanges through LDS alone, it waits for this wave's LDS accesses but
// not for its vector memory accesses, so that rows streaming into another LDS buffer (global_load_lds,
// whose LDS writes a full barrier would wait for) stay in flight across it.
template <bool LdsOnly>
__device__ __forceinline__ void wg_barrier() {
  if constexpr (LdsOnly) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else __syncthreads();
}

// LDS of the interface solve: the first interior rows exchanged between neighbouring lanes, and two
// buffers of the interface rows for PCR (three arrays of NT each), plus one stop flag per wave and buffer.
template <typename T, int NT>
struct InterfaceSpace {
  static constexpr int kWaves = (NT + 63) / 64;
  static constexpr int kVoteWords = (kWaves + 7) / 8;   // one byte per wave, read back as 64-bit words
  static constexpr int kBytes = 3 * 3 * NT * static_cast<int>(sizeof(T));
  T* xchg;          // 3 x NT
  T* rows;          // 2 buffers x 3 arrays x NT
  uint64_t* votes;  // 2 x kVoteWords; zeroed once (clear_votes) before the kernel's first barrier
  __device__ __forceinline__ void clear_votes() const {
    if (threadIdx.x < 2 * kVoteWords) votes[threadIdx.x] = 0;
  }
};

// What a lane learns of the next chunk: its first interior row (as exchanged) and its interface unknown.
template <typename T>
struct NextChunk {
  T al, ga, de;   // x_first = de - al y_t - ga y_{t+1}
  T y;            // y_{t+1}
};

// interface_solve on one wave: the rows cross lanes by permutes (between neighbours of a full wave by DPP moves)
// instead of LDS, and the stop vote is a ballot.  full: P = 64.  (us a step of one / 4096 systems, with the rows written
// to LDS, waited for and read back and with the votes there: 101 rows 1.56 / 3.19, 200 rows 1.50 / 3.52, 500 rows
// 1.44 / 3.77; this way 1.18 / 3.33, 0.95 / 3.08, 0.93 / 3.19.  As one body that tests `full` at each exchange: 1.37,
// 1.32 and 1.22 for one system.)
template <bool full>
__device__ __forceinline__ void wave_interface_solve(int P, double al0, double ga0, double de0, double alL, double gaL,
                                                     double deL, double ia, double ib, double ic, double id, double& y,
                                                     double& yp, NextChunk<double>* next) {
  const int t = static_cast<int>(threadIdx.x) & 63;
  const bool own = full || t < P;
  const int mask = 4 * (P - 1);
  const int before = (4 * t - 4) & mask, after = (4 * t + 4) & mask;
  double a = 0.0, c = 0.0, d = 0.0, nal, nga, nde;
  if (full) {
    nal = wave_move<0x134>(al0);
    nga = wave_move<0x134>(ga0);
    nde = wave_move<0x134>(de0);
  } else {
    nal = lane_value(al0, after);
    nga = lane_value(ga0, after);
    nde = lane_value(de0, after);
  }
  if (next) {
    next->al = nal;
    next->ga = nga;
    next->de = nde;
  }
  if (own) {
    const double inv = recip(__builtin_fma(-ic, nal, __builtin_fma(-ia, gaL, ib)));
    a = -(ia * alL) * inv;
    c = -(ic * nga) * inv;
    d = __builtin_fma(-ic, nde, __builtin_fma(-ia, deL, id)) * inv;
  }
  bool done = false;
  auto combine = [&](double am, double cm, double dm, double ap, double cp, double dp) {
    bool live = false;
    if (own) {
      pcr_combine(a, c, d, am, cm, dm, ap, cp, dp, a, c, d);
      live = (__builtin_fabs(a) + __builtin_fabs(c)) > kNegligible;
    }
    done = __ballot(live) == 0;
  };
  if constexpr (full)
    combine(wave_move<0x13C>(a), wave_move<0x13C>(c), wave_move<0x13C>(d), wave_move<0x134>(a), wave_move<0x134>(c), wave_move<0x134>(d));
  for (int s = full ? 2 : 1; s < P && !done; s <<= 1) {
    const int mi = (4 * (t - s)) & mask, pi = (4 * (t + s)) & mask;
    combine(lane_value(a, mi), lane_value(c, mi), lane_value(d, mi), lane_value(a, pi), lane_value(c, pi), lane_value(d, pi));
  }
  y = d;
  if (!done) y = d / ((1.0 + a) + c);   // (uniform) every row still coupled couples only to itself
  yp = full ? wave_move<0x13C>(y) : lane_value(y, before);
  if (next) next->y = full ? wave_move<0x134>(y) : lane_value(y, after);
}

// Solves the interface system.  Lane t < P passes its chunk's first interior row (al0, ga0, de0), its
// last interior row (alL, gaL, deL) and its interface row (ia, ib, ic, id); on return y = y_t and
// yp = y_{t-1}, and `next` (optional) holds the next chunk's first row and unknown.  Ends with a barrier after its last write to LDS; its last reads (yp) follow that
// barrier, so a caller that reuses the LDS for anything else must synchronise first.
template <typename T, int NT, bool LdsOnly = false>
__device__ __forceinline__ void interface_solve(const InterfaceSpace<T, NT>& w, int P, T al0, T ga0, T de0,
                                                T alL, T gaL, T deL, T ia, T ib, T ic, T id, T& y, T& yp,
                                                NextChunk<T>* next = nullptr) {
  if constexpr (NT == 64) {
    if (P == 64) wave_interface_solve<true>(P, al0, ga0, de0, alL, gaL, deL, ia, ib, ic, id, y, yp, next);
    else wave_interface_solve<false>(P, al0, ga0, de0, alL, gaL, deL, ia, ib, ic, id, y, yp, next);
    return;
  }
  constexpr int kR = NT;
  const int t = threadIdx.x;
  const bool own = t < P;
  const int mask = P - 1;
  if (own) {
    w.xchg[t] = al0;
    w.xchg[NT + t] = ga0;
    w.xchg[2 * NT + t] = de0;
  }
  wg_barrier<LdsOnly>();
  T a = T(0), c = T(0), d = T(0);
  if (own) {
    const int n = (t + 1) & mask;
    const T nal = w.xchg[n], nga = w.xchg[NT + n], nde = w.xchg[2 * NT + n];
    if (next) {
      next->al = nal;
      next->ga = nga;
      next->de = nde;
    }
    const T inv = recip(__builtin_fma(-ic, nal, __builtin_fma(-ia, gaL, ib)));
    a = -(ia * alL) * inv;
    c = -(ic * nga) * inv;
    d = __builtin_fma(-ic, nde, __builtin_fma(-ia, deL, id)) * inv;
    T* A = w.rows;
    A[t] = a; A[kR + t] = c; A[2 * kR + t] = d;
  }
  wg_barrier<LdsOnly>();
  int b = 0;
  bool done = false;
  for (int s = 1; s < P && !done; s <<= 1) {
    const T* A = w.rows + b * 3 * kR;
    const T* C = A + kR;
    const T* D = C + kR;
    bool live = false;
    if (own) {
      const int mi = (t - s) & mask, pi = (t + s) & mask;
      pcr_combine(a, c, d, A[mi], C[mi], D[mi], A[pi], C[pi], D[pi], a, c, d);
      live = (__builtin_fabs(a) + __builtin_fabs(c)) > kNegligible;
      T* nA = w.rows + (1 - b) * 3 * kR;
      nA[t] = a; nA[kR + t] = c; nA[2 * kR + t] = d;
    }
    const bool wave_live = __ballot(live) != 0;
    constexpr int kV = InterfaceSpace<T, NT>::kVoteWords;
    if ((t & 63) == 0) reinterpret_cast<unsigned char*>(w.votes + (1 - b) * kV)[t >> 6] = wave_live ? 1 : 0;
    wg_barrier<LdsOnly>();
    b = 1 - b;
    uint64_t any = 0;
#pragma unroll
    for (int k = 0; k < kV; ++k) any |= w.votes[b * kV + k];
    done = any == 0;
  }
  y = T(0);
  yp = T(0);
  if (own) {
    // every row's final coefficients are in buffer b; a row still coupled after all log2(P) steps
    // couples only to itself
    const int mi = (t - 1) & mask;
    const T* A = w.rows + b * 3 * kR;
    y = d;
    yp = A[2 * kR + mi];
    const int pi = (t + 1) & mask;
    if (next) next->y = A[2 * kR + pi];
    if (!done) {   // (uniform across the workgroup)
      y = d / ((T(1) + a) + c);
      yp = yp / ((T(1) + A[mi]) + A[kR + mi]);
      if (next) next->y = next->y / ((T(1) + A[pi]) + A[kR + pi]);
    }
  }
}

// ---- Whole systems in slots --------------------------------------------------------------------------
// A system of R rows on P lanes (a power of two, 2P <= R) gives a lane M = ceil(R / P) rows or one fewer,
// the longer chunks first.  Every lane works on M slots, so that no row is selected at a run-time index:
// a chunk one row short takes the later slots and leaves slot 0 a copy of y_{t-1} (x_0 = y_{t-1}, i.e.
// al = -1, ga = de = 0), through which its next row couples to y_{t-1} without any rounding.  The
// interface row is slot M - 1 and the last interior row slot M - 2 in every lane.  (Before, chunks of a
// run-time length compiled to about 100 register moves per lane and step beside 135 arithmetic
// instructions, and sizes other than 8192 or 16384 were held to 8 rows a lane to keep them from spilling.)
struct SlotLane {
  int base;          // row of slot 0 (the row before the chunk where slot 0 is no row)
  bool own;          // lanes P and beyond hold nothing
  bool dummy;        // slot 0 is no row
  bool first, last;  // the Dirichlet system's first row is in slot 0, its last row in slot M - 1
  double tie = -1.0; // al of a slot 0 that is no row: x_0 = -al y_{t-1}
};

// FULL: every lane holds M rows (R = P M with P the workgroup's lanes).
template <int M, bool FULL>
__device__ __forceinline__ SlotLane slot_lane(int t, int R, int P, bool dirichlet) {
  if constexpr (FULL) return SlotLane{t * M, true, false, dirichlet && t == 0, dirichlet && t == P - 1};
  const int rho = R - (M - 1) * P;   // chunks of M rows (R = (M - 1) P + rho, 1 <= rho <= P)
  const bool dummy = t >= rho;
  return SlotLane{t * (M - 1) + (dummy ? rho - 1 : t), t < P, dummy, dirichlet && t == 0, dirichlet && t == P - 1};
}

// BTCS rows for slot_eliminate: slot j from its old value.
struct SlotRows {
  double r, D, a, b;   // a, b: Dirichlet values
  static constexpr bool kInOrder = false;
  __device__ __forceinline__ void row(int, double ui, double& al, double& be, double& ga, double& de) const {
    btcs_row(ui, r, D, al, be, ga);
    de = ui;
  }
};

// Eliminates a lane's interior slots: on return slot j < M - 1 reads x_j = de[j] - al[j] y_{t-1} - ga[j] y_t
// and the interface row is (ia, ib, ic, id).  de[j] holds slot j's old value on entry.
template <int M, bool FULL, typename Rows>
__device__ __forceinline__ void slot_eliminate(const Rows& rows, const SlotLane& l, double (&al)[M], double (&ga)[M],
                                               double (&de)[M], double& ia, double& ib, double& ic, double& id) {
#pragma unroll
  for (int j = 0; j < M; ++j) {
    double aj, bj, cj, dj;
    rows.row(j, de[j], aj, bj, cj, dj);
    if (j == 0) {                        // x_{-1} = a at a Dirichlet system's first row
      dj = l.first ? __builtin_fma(-aj, rows.a, dj) : dj;
      aj = l.first ? 0.0 : aj;
    }
    if (j == M - 1) {                    // x_R = b at its last
      id = l.last ? __builtin_fma(-cj, rows.b, dj) : dj;
      ic = l.last ? 0.0 : cj;
      ia = aj;
      ib = bj;
    } else if (j == 0) {
      const double inv = recip(bj);
      al[0] = !FULL && l.dummy ? l.tie : aj * inv;
      ga[0] = !FULL && l.dummy ? 0.0 : cj * inv;
      de[0] = !FULL && l.dummy ? 0.0 : dj * inv;
    } else {
      const double inv = recip(__builtin_fma(-aj, ga[j - 1], bj));
      const double ai = aj * inv;
      al[j] = -(ai * al[j - 1]);
      ga[j] = cj * inv;
      de[j] = __builtin_fma(-ai, de[j - 1], dj * inv);
    }
    // (rows of many terms: assembled one after another, or the scheduler forms them all up front and holds
    // them in registers through the pivot chain)
    if constexpr (Rows::kInOrder) __builtin_amdgcn_sched_barrier(0);
  }
  // backward: the coupling to x_{j+1} becomes a coupling to y_t (slot M-2 already has this form)
#pragma unroll
  for (int j = M - 3; j >= 0; --j) {
    const double g = ga[j];
    de[j] = __builtin_fma(-g, de[j + 1], de[j]);
    al[j] = __builtin_fma(-g, al[j + 1], al[j]);
    ga[j] = -(g * ga[j + 1]);
  }
}

// One interface-partition solve of a whole system: eliminate (lanes with rows), exchange, PCR.  On
// return y = y_t and yp = y_{t-1} (see interface_solve for the LDS contract).
template <int NT, int M, bool FULL, bool LdsOnly = false, typename Rows>
__device__ __forceinline__ void slot_step(const InterfaceSpace<double, NT>& w, const Rows& rows, const SlotLane& l,
                                          int P, double (&al)[M], double (&ga)[M], double (&de)[M], double& y,
                                          double& yp, NextChunk<double>* next = nullptr) {
  double ia = 0.0, ib = 1.0, ic = 0.0, id = 0.0;
  slot_eliminate<M, FULL>(rows, l, al, ga, de, ia, ib, ic, id);
  const bool f = !FULL && l.dummy;       // the chunk's first interior row (M >= 3 where slot 0 is no row)
  constexpr int k = M > 2 ? 1 : 0;
  interface_solve<double, NT, LdsOnly>(w, P, f ? al[k] : al[0], f ? ga[k] : ga[0], f ? de[k] : de[0], al[M - 2],
                                       ga[M - 2], de[M - 2], ia, ib, ic, id, y, yp, next);
}

// Slot j from the interface unknowns, not rounded to the state type.
template <int M>
__device__ __forceinline__ double slot_value(int j, const double (&al)[M], const double (&ga)[M],
                                             const double (&de)[M], double yp, double y) {
  return j < M - 1 ? __builtin_fma(-ga[j], y, __builtin_fma(-al[j], yp, de[j])) : y;
}

// The slot counts of a class: M = ceil(R / P) is 2 to 8 on 64 lanes (P may be less there), 5 to 8 on wider
// workgroups, 9 to 16 in the classes of longer chunks (see btcs_width_class).
template <int NT, int MC, typename F>
__device__ __forceinline__ void with_slots(int R, int P, F&& f) {
#define BURGERS_SLOTS(K)                                                             \
  case K:                                                                            \
    if constexpr (K <= MC && (MC == 16 ? K > 8 : K > 4 || NT == 64)) f.template run<K, false>(); \
    break;
  if constexpr (NT > 64) {
    if (R == NT * MC) {   // every lane full: no slot is tested
      f.template run<MC, true>();
      return;
    }
  }
  switch ((R + P - 1) / P) {
    BURGERS_SLOTS(2) BURGERS_SLOTS(3) BURGERS_SLOTS(4) BURGERS_SLOTS(5) BURGERS_SLOTS(6) BURGERS_SLOTS(7)
    BURGERS_SLOTS(8) BURGERS_SLOTS(9) BURGERS_SLOTS(10) BURGERS_SLOTS(11) BURGERS_SLOTS(12) BURGERS_SLOTS(13)
    BURGERS_SLOTS(14) BURGERS_SLOTS(15) BURGERS_SLOTS(16)
    default: break;
  }
#undef BURGERS_SLOTS
}

}  // namespace burgers
