// Reverse steps of the BTCS adjoint with lam on chip: the discrete adjoint of a step y = u^k -> x = u^(k+1) solves
// A(y)^T mu = lam' and sets lam = (1 - G) mu with G_i = r (x_i - x_{i-1}) for y_i >= 0, r (x_{i+1} - x_i) otherwise;
// dJ/dD += -mu . (2 x_i - x_{i-1} - x_{i+1}).  Row i of A^T couples mu_{i-1} with p_{i-1} (the super-diagonal entry
// of row i-1 of A), mu_i with d_i and mu_{i+1} with l_{i+1}.
//
// A lane holds its chunk of lam, of the two states and of the elimination in registers for a run of reverse steps,
// in the slots of the forward solvers (interface.hpp); a step reads u^k alone (u^(k+1) is the last step's) and has
// the next step's state in flight behind its solve.  Systems of up to 8192 rows are solved whole, exactly, for a
// whole segment (adj_btcs_whole_kernel).  Longer ones take windows of several steps (adj_btcs_deep_kernel) over the
// chunks of the forward windows (window.hip), with the same locality: a window loses 2^S chunks at either end with
// each step, and how the steps are spread over launches does not show.  dJ/dD is carried per lane over its rows and all steps, in a slot per
// chunk of the system, so the sums do not depend on how the steps are grouped into launches.
//
// What bounds the windows: the latency of the transposed solve, two waves per SIMD that issue half of the time; 58 vector
// instructions per row of a window and step (counted), 85 per row kept.
//
// Error of a window's kept row, per step: as of the forward windows, that of the couplings dropped.  A row that couples
// mu_f outside a run of rows to mu_i inside it through A_w^{-T} does so with at most D + C (C = r max|u|) times
// (A_w^{-1})_{f',i}, f' the run's row beside f.  A_w is a strictly row-diagonally dominant M-matrix with row sums >= 1, so
// A_w^{-1} >= 0 with row sums <= 1, and its columns decay from the diagonal like theta of the forward windows: after S
// PCR steps the couplings are within (D + C) theta^(n_S - 1).  With (D + C) theta^257 <= 2^-55 (S = 4) or (D + C)
// theta^(15 2^S) <= 2^-56 (S < 4), theta from the largest |u| at the start of the call (the states' maximum principle), what
// is dropped costs about 2^-53 max|mu| at most.  Systems beyond the bound are solved whole by one workgroup of 1024
// lanes (up to 16384 rows) or by the partition levels' array path.
#include "interface.hpp"
#include "internal.hpp"
#include "staging.hpp"
#include "stencil.hpp"
#include "windows.hpp"

#pragma clang fp contract(off)

namespace burgers {
namespace {

// Where a lane's rows lie: lane t of L holds rows [row(t), row(t + 1)) (past a periodic system's end in a window),
// node(k) is the instance node of such a row.
template <int M>
struct WholeLayout {
  int R, L, rho, first;
  __device__ __forceinline__ WholeLayout(const InstDesc& d, int rows, int P)
      : R(rows), L(P), rho(rows - (M - 1) * P), first(d.bc == kDirichlet ? 1 : 0) {}
  __device__ __forceinline__ int row(int t) const { return (M - 1) * t + (t < rho ? t : rho); }
  __device__ __forceinline__ int node(int k) const { return k + first; }
  __device__ __forceinline__ bool dummy(int t) const { return t >= rho; }
};
struct WindowLayout {
  Chunks ch;
  int R, c0, L, first;
  __device__ __forceinline__ WindowLayout(const InstDesc& d, const ChunkWin& w)
      : ch(d.bc == kDirichlet ? d.n - 2 : d.n), R(ch.R), c0(w.first), L(w.chunks), first(d.bc == kDirichlet ? 1 : 0) {}
  __device__ __forceinline__ int row(int t) const {
    const int c = c0 + t;
    return c >= ch.P ? ch.base(c - ch.P) + ch.R : ch.base(c);
  }
  __device__ __forceinline__ int node(int k) const { return (k >= ch.R ? k - ch.R : k) + first; }
  __device__ __forceinline__ bool dummy(int t) const {
    const int c = c0 + t;
    return ch.lacks(c >= ch.P ? c - ch.P : c);
  }
};

// The lanes' rows between HBM and their slots in two steps, half a wave's lanes at a time, 64 consecutive rows per
// instruction: fetch issues the loads, spread passes the values through the wave's region of LDS (slot 0 of a lane
// without a row there is left to the caller).
template <int M, typename Lay>
__device__ __forceinline__ void fetch(const double* __restrict__ src, const Lay& lay, double (&v)[2 * ((M + 1) / 2)]) {
  constexpr int H = (M + 1) / 2;
  const int lt = opaque_lane(static_cast<int>(threadIdx.x)), lane = lt & 63;
  const int t0 = __builtin_amdgcn_readfirstlane(lt) & ~63;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int ta = t0 + 32 * h < lay.L ? t0 + 32 * h : lay.L, tb = ta + 32 < lay.L ? ta + 32 : lay.L;
    const int ra = lay.row(ta), at = ra >= lay.R ? ra - lay.R : ra;
    if (at + 64 * H <= lay.R) {                // (uniform) the rows from here on are there, whosever: one address
      const double* __restrict__ p = src + lay.first + at;
#pragma unroll
      for (int i = 0; i < H; ++i) v[H * h + i] = p[lane + 64 * i];
      continue;
    }
    const int last = lay.row(tb) - 1;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int k = ra + lane + 64 * i;
      v[H * h + i] = src[lay.node(k < last ? k : last)];
    }
  }
}

template <int M, typename Lay>
__device__ __forceinline__ void spread(const double (&v)[2 * ((M + 1) / 2)], double* region, const Lay& lay,
                                       double (&out)[M]) {
  constexpr int H = (M + 1) / 2;
  const int lt = opaque_lane(static_cast<int>(threadIdx.x)), lane = lt & 63;
  const int t0 = __builtin_amdgcn_readfirstlane(lt) & ~63;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int i = 0; i < H; ++i) region[apad(lane) + 68 * i] = v[H * h + i];   // (apad(lane + 64 i))
    wave_sync();
    if ((lane >> 5) == h && lt < lay.L) {
      const int at = lay.row(lt) - lay.row(t0 + 32 * h) - (lay.dummy(lt) ? 1 : 0);
      const int low = at & 15, from = apad(at);
#pragma unroll
      for (int j = 0; j < M; ++j)              // (apad(at + j); slot 0's place may be the one before the region)
        out[j] = region[j > 0 ? from + j + (low + j > 15 ? 1 : 0) : (at < 0 ? 0 : from)];
    }
    wave_sync();
  }
}

// The lanes' rows in [lo, hi) back to dst.
template <int M, typename Lay>
__device__ __forceinline__ void put_rows(const double (&x)[M], double* region, const Lay& lay, int lo, int hi,
                                         double* __restrict__ dst) {
  constexpr int H = (M + 1) / 2;
  const int lt = opaque_lane(static_cast<int>(threadIdx.x)), lane = lt & 63;
  const int t0 = __builtin_amdgcn_readfirstlane(lt) & ~63;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int ta = t0 + 32 * h < lay.L ? t0 + 32 * h : lay.L, tb = ta + 32 < lay.L ? ta + 32 : lay.L;
    const int ra = lay.row(ta), rb = lay.row(tb);
    if ((lane >> 5) == h && lt < lay.L) {
      const int at = lay.row(lt) - ra, shift = lay.dummy(lt) ? 1 : 0;
#pragma unroll
      for (int j = 0; j < M; ++j)
        if (j > 0 || !shift) region[apad(at - shift + j)] = x[j];
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int k = ra + lane + 64 * i;
      const double v = region[apad(lane) + 68 * i];   // (apad(lane + 64 i))
      if (k < rb && k >= lo && k < hi) dst[lay.node(k)] = v;
    }
    wave_sync();
  }
}

// LDS of a workgroup.
template <int NT, int MC>
struct AdjSpace {
  static constexpr int kRegion = 64 * ((MC + 1) / 2) + 4 * ((MC + 1) / 2);   // (apad of the last)
  InterfaceSpace<double, NT> iface;
  double* region;   // the wave's
  double* ends;     // 2 x NT: every lane's first and last value of a state
};

// Rows of A(y)^T for slot_eliminate, y in the lane's slots, yl and yr beyond.
template <int M>
struct TransposedRows {
  const double (&y)[M];
  double yl, yr, r, D;
  double a = 0.0, b = 0.0;   // (the couplings beyond a Dirichlet system's or a window's ends just vanish)
  static constexpr bool kInOrder = M > 8;
  __device__ __forceinline__ void row(int j, double lam, double& al, double& be, double& ga, double& de) const {
    double t0, t1, t2, t3;
    btcs_row(j > 0 ? y[j > 0 ? j - 1 : 0] : yl, r, D, t0, t1, al);            // p_{j-1}
    btcs_row(y[j], r, D, t2, be, t3);                                         // d_j
    btcs_row(j < M - 1 ? y[j < M - 1 ? j + 1 : j] : yr, r, D, ga, t0, t1);    // l_{j+1}
    de = lam;
  }
};

// The values beyond a lane's slots of a state: the last of the lane before and the first of the lane after, around
// the L lanes; a slot 0 without a row takes the former.
template <int NT, int M>
__device__ __forceinline__ void neighbours(double (&x)[M], double* ends, int L, bool own, bool dummy, double& xl,
                                           double& xr) {
  const int t = static_cast<int>(threadIdx.x);
  if (own) {
    ends[t] = dummy ? x[M > 1 ? 1 : 0] : x[0];
    ends[NT + t] = x[M - 1];
  }
  wg_barrier<true>();
  xl = xr = 0.0;
  if (own) {
    xl = ends[NT + (t > 0 ? t - 1 : L - 1)];
    xr = ends[t < L - 1 ? t + 1 : 0];
    if (dummy) x[0] = xl;
  }
}

// Reverse steps k = k_hi - 1 down to k_lo of one system or window (u^k at state(k); lam' at lam_in, lam to lam_out, by
// node).  PCR: the PCR steps of a window's solve (0: a whole system).
template <int NT, int MC, int M, bool FULL, bool WINDOW, typename Lay, typename State>
__device__ __forceinline__ void reverse_steps(const AdjSpace<NT, MC>& ws, const InstDesc& d, const Lay& lay,
                                              const SlotLane& l, bool end_first, bool end_last, int pcr,
                                              const State& state, int k_lo, int k_hi,
                                              const double* __restrict__ lam_in, double* __restrict__ lam_out, int lo,
                                              int hi, double* __restrict__ slot) {
  double al[M], ga[M], de[M], X[M], Y[M], V[2 * ((M + 1) / 2)];
  double xl, xr, yl, yr;
#pragma unroll
  for (int j = 0; j < M; ++j) de[j] = X[j] = Y[j] = 0.0;
  {
    double V0[2 * ((M + 1) / 2)], V1[2 * ((M + 1) / 2)];   // (all in flight at once)
    fetch<M>(lam_in, lay, V0);
    fetch<M>(state(k_hi), lay, V1);
    fetch<M>(state(k_hi - 1), lay, V);
    spread<M>(V0, ws.region, lay, de);
    spread<M>(V1, ws.region, lay, X);
  }
  neighbours<NT>(X, ws.ends, lay.L, l.own, l.dummy, xl, xr);
  wg_barrier<true>();                          // ends read before they are written again
  double g = slot ? *slot : 0.0;
  for (int k = k_hi - 1; k >= k_lo; --k) {
    spread<M>(V, ws.region, lay, Y);
    if (k > k_lo) fetch<M>(state(k - 1), lay, V);   // in flight behind this step's solve
    neighbours<NT>(Y, ws.ends, lay.L, l.own, l.dummy, yl, yr);
    double ia = 0.0, ib = 1.0, ic = 0.0, id = 0.0, y, yp;
    if (l.own) slot_eliminate<M, FULL>(TransposedRows<M>{Y, yl, yr, d.r, d.D}, l, al, ga, de, ia, ib, ic, id);
    constexpr int f1 = M > 2 ? 1 : 0;
    const bool f = !FULL && l.dummy;
    if constexpr (WINDOW)
      window_solve<NT, true>(ws.iface, lay.L, pcr, l.own, f ? al[f1] : al[0], f ? ga[f1] : ga[0], f ? de[f1] : de[0],
                             al[M - 2], ga[M - 2], de[M - 2], ia, ib, ic, id, y, yp);
    else
      interface_solve<double, NT, true>(ws.iface, lay.L, f ? al[f1] : al[0], f ? ga[f1] : ga[0],
                                        f ? de[f1] : de[0], al[M - 2], ga[M - 2], de[M - 2], ia, ib, ic, id, y, yp);
    // finish: mu_j, lam_j = (1 - G) mu_j and the terms of dJ/dD
    if (end_first) xl = d.a;
    if (end_last) xr = d.b;
#pragma unroll
    for (int j = 0; j < M; ++j) {
      const double mu = slot_value<M>(j, al, ga, de, yp, y);
      const double xm = j > 0 ? X[j > 0 ? j - 1 : 0] : xl, xp = j < M - 1 ? X[j < M - 1 ? j + 1 : j] : xr;
      const double G = Y[j] >= 0.0 ? d.r * (X[j] - xm) : d.r * (xp - X[j]);
      de[j] = (1.0 - G) * mu;
      const double term = __builtin_fma(-mu, (2.0 * X[j] - xm) - xp, g);
      g = j == 0 && l.dummy ? g : term;
    }
#pragma unroll
    for (int j = 0; j < M; ++j) X[j] = Y[j];
    xl = yl;
    xr = yr;
  }
  put_rows<M>(de, ws.region, lay, lo, hi, lam_out);
  if (slot) *slot = g;
}

// The same of a whole system on 1024 lanes, whose 128 registers hold the elimination and no states beside it: each step
// reads u^k for its rows and, once mu stands where the elimination was, u^(k+1) for the finish, with nothing in flight
// behind the solve.  (256 systems of 16384 rows, us per reverse step: 26.5; 49 with both states and a prefetch in
// registers as above, most of them spilled.)
template <int NT, int MC, int M, bool FULL, typename Lay, typename State>
__device__ __forceinline__ void reverse_steps_lean(const AdjSpace<NT, MC>& ws, const InstDesc& d, const Lay& lay,
                                                   const SlotLane& l, const State& state, int k_lo, int k_hi,
                                                   const double* __restrict__ lam_in, double* __restrict__ lam_out,
                                                   double* __restrict__ slot) {
  double de[M];
  auto read = [&](const double* src, double (&out)[M]) {
    double V[2 * ((M + 1) / 2)];
#pragma unroll
    for (int j = 0; j < M; ++j) out[j] = 0.0;    // (or the last step's values are carried for lanes without rows)
    fetch<M>(src, lay, V);
    spread<M>(V, ws.region, lay, out);
  };
  read(lam_in, de);
  double g = *slot;
  for (int k = k_hi - 1; k >= k_lo; --k) {
    unsigned up = 0;                             // bit j: y_j >= 0
    double y, yp;
    {
      double al[M], ga[M], Y[M], yl, yr, ia, ib, ic, id;
      read(state(k), Y);
      neighbours<NT>(Y, ws.ends, lay.L, true, l.dummy, yl, yr);
#pragma unroll
      for (int j = 0; j < M; ++j) up |= Y[j] >= 0.0 ? 1u << j : 0u;
      up = static_cast<unsigned>(opaque_lane(static_cast<int>(up)));   // (formed here, not from Y kept)
      slot_eliminate<M, FULL>(TransposedRows<M>{Y, yl, yr, d.r, d.D}, l, al, ga, de, ia, ib, ic, id);
      const bool f = !FULL && l.dummy;
      interface_solve<double, NT, true>(ws.iface, lay.L, f ? al[1] : al[0], f ? ga[1] : ga[0], f ? de[1] : de[0],
                                        al[M - 2], ga[M - 2], de[M - 2], ia, ib, ic, id, y, yp);
#pragma unroll
      for (int j = 0; j < M; ++j) de[j] = slot_value<M>(j, al, ga, de, yp, y);   // mu
    }
    __builtin_amdgcn_sched_barrier(0);
    double X[M], xl, xr;
    read(state(k + 1), X);
    neighbours<NT>(X, ws.ends, lay.L, true, l.dummy, xl, xr);   // (the solve's barriers follow the last read of ends)
    if (l.first) xl = d.a;
    if (l.last) xr = d.b;
#pragma unroll
    for (int j = 0; j < M; ++j) {
      const double xm = j > 0 ? X[j > 0 ? j - 1 : 0] : xl, xp = j < M - 1 ? X[j < M - 1 ? j + 1 : j] : xr;
      const double G = up >> j & 1u ? d.r * (X[j] - xm) : d.r * (xp - X[j]);
      const double term = __builtin_fma(-de[j], (2.0 * X[j] - xm) - xp, g);
      g = j == 0 && l.dummy ? g : term;
      de[j] = (1.0 - G) * de[j];
    }
    wg_barrier<true>();                          // ends read before they are written again
  }
  put_rows<M>(de, ws.region, lay, 0, lay.R, lam_out);
  *slot = g;
}

template <int NT, int MC>
struct AdjWholeRun {
  const AdjSpace<NT, MC>& ws;
  const InstDesc& d;
  int R, P;
  const double *u0, *useg, *lamp;
  int64_t ustride;
  int k_lo, k_hi;
  double *lam, *slot;
  template <int M, bool FULL>
  __device__ __forceinline__ void run() const {
    const int t = static_cast<int>(threadIdx.x);
    const bool dir = d.bc == kDirichlet;
    const WholeLayout<M> lay(d, R, P);
    const SlotLane l = slot_lane<M, FULL>(t, R, P, dir);
    auto state = [&](int k) { return (k == 0 ? u0 : useg + static_cast<int64_t>(k - 1) * ustride) + d.off; };
    if constexpr (NT == 1024)
      reverse_steps_lean<NT, MC, M, FULL>(ws, d, lay, l, state, k_lo, k_hi, lamp + d.off, lam + d.off, slot + t);
    else
      reverse_steps<NT, MC, M, FULL, false>(ws, d, lay, l, l.first, l.last, 0, state, k_lo, k_hi, lamp + d.off,
                                            lam + d.off, 0, R, l.own ? slot + t : nullptr);
  }
};

// Whole systems of one width class, one workgroup each.  `code` (optional): those whose windows' bound failed.
template <int NT, int MC>
__global__ __launch_bounds__(NT, NT == 1024 ? 4 : 2) void adj_btcs_whole_kernel(
    const InstDesc* __restrict__ inst, const SysDesc* __restrict__ systems, const int32_t* __restrict__ slot_begin,
    const double* __restrict__ u0, const double* __restrict__ useg, int64_t ustride, int k_lo, int k_hi,
    const double* __restrict__ lamp, double* __restrict__ lam, double* __restrict__ gslot,
    const int* __restrict__ code) {
  using IS = InterfaceSpace<double, NT>;
  using AS = AdjSpace<NT, MC>;
  __shared__ double iface_lds[IS::kBytes / sizeof(double)];
  __shared__ uint64_t iface_votes[2 * IS::kVoteWords];
  __shared__ double regions[(NT / 64) * AS::kRegion];
  __shared__ double ends[2 * NT];
  const AS ws{IS{iface_lds, iface_lds + 3 * NT, iface_votes},
              regions + __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6) * AS::kRegion, ends};
  ws.iface.clear_votes();
  const SysDesc sys = systems[blockIdx.x];
  if (code && code[sys.inst] != 0) return;     // its windows hold
  const InstDesc d = inst[sys.inst];
  const bool dir = d.bc == kDirichlet;
  if (dir && threadIdx.x == 0) {               // Dirichlet end nodes carry none
    lam[d.off] = 0.0;
    lam[d.off + d.n - 1] = 0.0;
  }
  double* slot = gslot + slot_begin[sys.inst];
  if (sys.rows == 1) {                         // a single Dirichlet unknown
    if (threadIdx.x == 0) {
      double v = lamp[d.off + 1], g = *slot;
      for (int k = k_hi - 1; k >= k_lo; --k) {
        const double y = (k == 0 ? u0 : useg + static_cast<int64_t>(k - 1) * ustride)[d.off + 1];
        const double x = (useg + static_cast<int64_t>(k) * ustride)[d.off + 1];
        double t0, be, t1;
        btcs_row(y, d.r, d.D, t0, be, t1);
        const double mu = v / be, G = y >= 0.0 ? d.r * (x - d.a) : d.r * (d.b - x);
        v = (1.0 - G) * mu;
        g = __builtin_fma(-mu, (2.0 * x - d.a) - d.b, g);
      }
      lam[d.off + 1] = v;
      *slot = g;
    }
    return;
  }
  with_slots<NT, MC>(sys.rows, sys.chunks,
                     AdjWholeRun<NT, MC>{ws, d, sys.rows, sys.chunks, u0, useg, lamp, ustride, k_lo, k_hi, lam, slot});
}

// Launch `launch` of a segment of `len` reverse steps on windows: kAdjDeepHalo / 2^S steps with S of the window's instance
// (0: left to other kernels), from lam[launch & 1] to the other.
__global__ __launch_bounds__(kDeepLanes, 2) void adj_btcs_deep_kernel(
    const InstDesc* __restrict__ inst, const ChunkWin* __restrict__ wins, const int* __restrict__ code,
    const int32_t* __restrict__ slot_begin, const double* __restrict__ u0, const double* __restrict__ useg,
    int64_t ustride, int len, int launch, const double* __restrict__ lamp, double* __restrict__ lam,
    double* __restrict__ gslot) {
  constexpr int NT = kDeepLanes, M = kChunkRows;
  using IS = InterfaceSpace<double, NT>;
  using AS = AdjSpace<NT, M>;
  __shared__ double iface_lds[IS::kBytes / sizeof(double)];
  __shared__ uint64_t iface_votes[2 * IS::kVoteWords];
  __shared__ double regions[(NT / 64) * AS::kRegion];
  __shared__ double ends[2 * NT];
  const AS ws{IS{iface_lds, iface_lds + 3 * NT, iface_votes},
              regions + __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6) * AS::kRegion, ends};
  ws.iface.clear_votes();
  const ChunkWin w = wins[blockIdx.x];
  const int pcr = code[w.inst];
  if (pcr <= 0) return;
  int done;
  const int steps = deep_steps<kAdjDeepHalo>(w, pcr, launch, len, done);
  if (steps == 0) return;
  const InstDesc d = inst[w.inst];
  const bool dir = d.bc == kDirichlet;
  const WindowLayout lay(d, w);
  const int t = static_cast<int>(threadIdx.x);
  const bool first = t == 0, last = t == w.chunks - 1;
  const bool end_first = dir && first && w.first == 0, end_last = dir && last && w.first + w.chunks == lay.ch.P;
  const SlotLane l{0, t < w.chunks, lay.dummy(t), first, last, first ? 0.0 : -1.0};
  const int c = w.first + t < lay.ch.P ? w.first + t : w.first + t - lay.ch.P;
  const bool kept = t >= w.lo && t < w.lo + w.count;
  auto state = [&](int k) { return (k == 0 ? u0 : useg + static_cast<int64_t>(k - 1) * ustride) + d.off; };
  reverse_steps<NT, M, M, false, true>(ws, d, lay, l, end_first, end_last, pcr, state, len - done - steps, len - done,
                                       lamp + d.off, lam + d.off, lay.row(w.lo), lay.row(w.lo + w.count),
                                       kept ? gslot + slot_begin[w.inst] + c : nullptr);
  if (end_first) lam[d.off] = 0.0;             // Dirichlet end nodes carry none
  if (end_last) lam[d.off + d.n - 1] = 0.0;
}

// lam of the instances whose last launch left it in `lam`, to lam_next.
__global__ __launch_bounds__(256) void adj_btcs_settle_kernel(const InstDesc* __restrict__ inst,
                                                              const ChunkWin* __restrict__ wins,
                                                              const int* __restrict__ code, int len,
                                                              const double* __restrict__ lam,
                                                              double* __restrict__ lam_next) {
  const ChunkWin w = wins[blockIdx.x];
  const int pcr = code[w.inst];
  if (pcr <= 0) return;
  const int per = kAdjDeepHalo >> pcr;
  if ((len + per - 1) / per & 1) return;
  const InstDesc d = inst[w.inst];
  const WindowLayout lay(d, w);
  const int lo = lay.row(w.lo), hi = lay.row(w.lo + w.count);
  for (int k = lo + static_cast<int>(threadIdx.x); k < hi; k += 256) lam_next[d.off + lay.node(k)] = lam[d.off + lay.node(k)];
  if (d.bc == kDirichlet && threadIdx.x == 0) {
    if (w.first + w.lo == 0) lam_next[d.off] = 0.0;
    if (w.first + w.lo + w.count == lay.ch.P) lam_next[d.off + d.n - 1] = 0.0;
  }
}

}  // namespace

hipError_t launch_adj_btcs_deep(const burgers_ctx* ctx, const BtcsPlan& plan, const int32_t* slot_begin,
                                const double* u0, const double* useg, int64_t ustride, int len, double* lam,
                                double* lam_next, double* gslot) {
  if (plan.n_deep <= 0 || len <= 0) return hipSuccess;
  const InstDesc* inst = ctx->inst.as<InstDesc>();
  const ChunkWin* wins = plan.deep->as<ChunkWin>();
  const int* code = deep_code(plan.deep_words.as<int>(), ctx->count);
  const unsigned n = static_cast<unsigned>(plan.n_deep);
  constexpr int kFewest = kAdjDeepHalo >> kMaxPcr;
  double* bufs[2] = {lam, lam_next};
  for (int j = 0; j < (len + kFewest - 1) / kFewest; ++j)
    adj_btcs_deep_kernel<<<n, kDeepLanes, 0, ctx->stream>>>(inst, wins, code, slot_begin, u0, useg, ustride, len, j,
                                                            bufs[j & 1], bufs[(j & 1) ^ 1], gslot);
  adj_btcs_settle_kernel<<<n, 256, 0, ctx->stream>>>(inst, wins, code, len, lam, lam_next);
  return hipGetLastError();
}

hipError_t launch_adj_btcs_whole(const burgers_ctx* ctx, const WgGroup& g, const int32_t* slot_begin, const double* u0,
                                 const double* useg, int64_t ustride, int k_lo, int k_hi, const double* lamp,
                                 double* lam, double* gslot, const int* code) {
  if (g.n <= 0 || k_hi <= k_lo) return hipSuccess;
  const unsigned n = static_cast<unsigned>(g.n);
  auto go = [&](auto kernel, int lanes) {
    kernel<<<n, lanes, 0, ctx->stream>>>(ctx->inst.as<InstDesc>(), g.sys->as<SysDesc>(), slot_begin, u0, useg, ustride,
                                         k_lo, k_hi, lamp, lam, gslot, code);
  };
  switch (g.shape.lanes) {
    case 64: go(adj_btcs_whole_kernel<64, 8>, 64); break;
    case 128: go(adj_btcs_whole_kernel<128, 8>, 128); break;
    case 256: go(adj_btcs_whole_kernel<256, 8>, 256); break;
    case 512:
      if (g.shape.chunk == 16) go(adj_btcs_whole_kernel<512, 16>, 512);
      else go(adj_btcs_whole_kernel<512, 8>, 512);
      break;
    default: go(adj_btcs_whole_kernel<1024, 16>, 1024); break;
  }
  return hipGetLastError();
}

}  // namespace burgers
