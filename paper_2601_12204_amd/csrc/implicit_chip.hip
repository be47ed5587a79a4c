// Crank-Nicolson and Newton systems of up to 8192 rows held on chip for every step of a call, one
// workgroup per system, by the interface partition of the resident BTCS solver (interface.hpp).  HBM sees
// the state once per call instead of once per step (Crank-Nicolson) or nine times per step (Newton: four
// iterations that each read the iterate twice, the old state once or twice and write the iterate, after a
// pass that copies the state).
//
// What bounds them: vector issue in binary64 and the barriers of the interface solve, as for BTCS.  Both
// keep a second state beside the elimination's three arrays (the old state u^n; for Newton the iterate),
// so a lane takes at most 8 rows (16 rows with a second state would need more than the 128 registers that
// let four waves share a SIMD).
#include "interface.hpp"
#include "internal.hpp"
#include "newton_check.hpp"
#include "stencil.hpp"

#pragma clang fp contract(off)

namespace burgers {
namespace {

// Crank-Nicolson: (I + N/2) y = u^n, the BTCS solve with r and D halved (inst: that table), then
// u^{n+1} = 2y - u^n, with y rounded to the state type as the per-step solver stores it.
template <typename S, int NT>
struct CnRun {
  const InterfaceSpace<double, NT>& ws;
  const InstDesc& d;
  int R, P;
  S* x;
  int steps;
  template <int M, bool FULL>
  __device__ __forceinline__ void run() const {
    using T = double;
    const SlotLane l = slot_lane<M, FULL>(static_cast<int>(threadIdx.x), R, P, d.bc == kDirichlet);
    const SlotRows rows{d.r, d.D, d.a, d.b};
    T old[M], al[M], ga[M], de[M];
#pragma unroll
    for (int j = 0; j < M; ++j) old[j] = l.own ? static_cast<T>(x[l.base + j]) : T(0);
    for (int step = 0; step < steps; ++step) {
#pragma unroll
      for (int j = 0; j < M; ++j) de[j] = old[j];
      T y, yp;
      slot_step<NT, M, FULL>(ws, rows, l, P, al, ga, de, y, yp);
#pragma unroll
      for (int j = 0; j < M; ++j) {
        const T v = static_cast<T>(static_cast<S>(slot_value<M>(j, al, ga, de, yp, y)));
        old[j] = static_cast<T>(static_cast<S>(2.0 * v - old[j]));
      }
    }
    if (l.own) {
#pragma unroll
      for (int j = 0; j < M; ++j)
        if (j > 0 || !l.dummy) x[l.base + j] = static_cast<S>(old[j]);
    }
  }
};

template <typename S, int NT>
__global__ __launch_bounds__(NT, 4) void cn_resident_kernel(const InstDesc* __restrict__ inst,
                                                            const SysDesc* __restrict__ systems, S* __restrict__ u,
                                                            int steps) {
  using T = double;
  using IS = InterfaceSpace<T, NT>;
  __shared__ T iface_lds[IS::kBytes / sizeof(T)];
  __shared__ uint64_t iface_votes[2 * IS::kVoteWords];
  const IS ws{iface_lds, iface_lds + 3 * NT, iface_votes};
  ws.clear_votes();
  const SysDesc sys = systems[blockIdx.x];
  const InstDesc d = inst[sys.inst];
  const bool dir = d.bc == kDirichlet;
  S* __restrict__ x = u + d.off + (dir ? 1 : 0);
  if (dir && threadIdx.x == 0) {
    u[d.off] = static_cast<S>(d.a);
    u[d.off + d.n - 1] = static_cast<S>(d.b);
  }
  if (sys.rows == 1) {   // a single Dirichlet unknown
    if (threadIdx.x == 0) {
      T v = static_cast<T>(x[0]);
      for (int step = 0; step < steps; ++step) {
        T al, be, ga;
        btcs_row(v, d.r, d.D, al, be, ga);
        const T y = static_cast<T>(static_cast<S>(((v - al * d.a) - ga * d.b) / be));
        v = static_cast<T>(static_cast<S>(2.0 * y - v));
      }
      x[0] = static_cast<S>(v);
    }
    return;
  }
  with_slots<NT, 8>(sys.rows, sys.chunks, CnRun<S, NT>{ws, d, sys.rows, sys.chunks, x, steps});
}

// Rows of a Newton iteration for a lane's slots: the Jacobian row of eq. 11 at the iterate x and the
// right-hand side -F; xl and xr are the iterate's values beside the slots (a slot 0 that is no row holds the
// value before the chunk).  Evaluated in the association of the per-step Newton kernels, so that the
// dominance check decides alike.  A Dirichlet value does not move: the end rows drop that coupling.
template <int M, bool FULL>
struct NewtonSlotRows {
  const double (&x)[M];
  const double (&u)[M];
  double xl, xr, half_r, D;
  const SlotLane& l;
  int& bad;
  static constexpr double a = 0.0, b = 0.0;
  static constexpr bool kInOrder = true;
  __device__ __forceinline__ void row(int j, double, double& al, double& be, double& ga, double& de) const {
    const double xm = j > 0 ? x[j > 0 ? j - 1 : 0] : xl;
    const double xp = j < M - 1 ? x[j + 1 < M ? j + 1 : j] : xr;
    const double hx = half_r * x[j];
    const double F = (x[j] - u[j]) + (hx * (xp - xm) - D * fma_exact(-2.0, x[j], xp + xm));
    al = -hx - D;
    be = (1.0 + 2.0 * D) + half_r * (xp - xm);
    ga = hx - D;
    de = -F;
    if (j == 0) al = l.first ? 0.0 : al;
    if (j == M - 1) ga = l.last ? 0.0 : ga;
    const bool lost = newton_row_not_dominant(al, be, ga);
    bad |= (j == 0 && !FULL ? lost && !l.dummy : lost) ? 1 : 0;
    asm volatile("" : "+v"(bad));   // (decided here: sunk below the solve, the check would hold every row's terms)
  }
};

// The last increments of a step against the iterate, per group of 64 consecutive unknowns (the group that
// one wave of the per-step kernel holds).  A lane whose own rows of a group pass among themselves cannot
// make the group fail, so the groups' maxima are formed (in LDS, by atomic maxima of the non-negative
// values' bit patterns) only when some lane's rows do not: a vote and one barrier per step otherwise.
template <int NT>
struct IncrementSpace {
  static constexpr int kGroups = NT * 8 / 64 + 1;
  unsigned long long* inc;     // kGroups
  unsigned long long* scale;   // kGroups
  uint64_t* votes;             // 2 x kVoteWords (step parity), one byte per wave, zero at the start
};

template <int NT, int M, bool FULL>
__device__ __forceinline__ void check_increments(const IncrementSpace<NT>& w, int parity, const SlotLane& l,
                                                 const double (&delta)[M], const double (&x)[M],
                                                 const double (&u)[M], double tol, int* flags) {
  constexpr int kV = InterfaceSpace<double, NT>::kVoteWords, kGroups = IncrementSpace<NT>::kGroups;
  const int tid = threadIdx.x;
  const int g0 = l.base >> 6;
  double inc[2] = {0.0, 0.0}, scale[2] = {0.0, 0.0};   // of group g0 and of the next one
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const bool row = l.own && (FULL || j > 0 || !l.dummy);
    const bool second = ((l.base + j) >> 6) != g0;
    const bool finite = __builtin_isfinite(delta[j]) && __builtin_isfinite(x[j]);
    const double i = finite ? __builtin_fabs(delta[j]) : __builtin_inf();
    const double c = finite ? __builtin_fmax(__builtin_fabs(x[j]), __builtin_fabs(u[j])) : 0.0;
    inc[0] = __builtin_fmax(inc[0], row && !second ? i : 0.0);
    inc[1] = __builtin_fmax(inc[1], row && second ? i : 0.0);
    scale[0] = __builtin_fmax(scale[0], row && !second ? c : 0.0);
    scale[1] = __builtin_fmax(scale[1], row && second ? c : 0.0);
  }
  const bool doubt = !(inc[0] <= tol * scale[0]) || !(inc[1] <= tol * scale[1]);
  const bool wave_doubt = __ballot(doubt) != 0;
  if ((tid & 63) == 0) reinterpret_cast<unsigned char*>(w.votes + parity * kV)[tid >> 6] = wave_doubt ? 1 : 0;
  __syncthreads();
  uint64_t any = 0;
#pragma unroll
  for (int k = 0; k < kV; ++k) any |= w.votes[parity * kV + k];
  if (any == 0) return;
  for (int g = tid; g < kGroups; g += NT) {
    w.inc[g] = 0;
    w.scale[g] = 0;
  }
  __syncthreads();
  if (l.own) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (g0 + q < kGroups) {
        atomicMax(&w.inc[g0 + q], __builtin_bit_cast(unsigned long long, inc[q]));
        atomicMax(&w.scale[g0 + q], __builtin_bit_cast(unsigned long long, scale[q]));
      }
    }
  }
  __syncthreads();
  for (int g = tid; g < kGroups; g += NT)
    if (!(__builtin_bit_cast(double, w.inc[g]) <= tol * __builtin_bit_cast(double, w.scale[g]))) flags[1] = 1;
  __syncthreads();
}

// Fully implicit steps (eqs. 10-14): kNewtonIters Newton iterations each, the old state and the iterate in
// registers.  A lane follows the iterate's two neighbours of its slots by itself: the solve gives it
// y_{t-1} (the increment of the row before its chunk) and the next chunk's first row and unknown, whose
// increment it forms exactly as that chunk's lane does, so no further exchange is needed.
template <typename S, int NT>
struct NewtonRun {
  const InterfaceSpace<double, NT>& ws;
  const IncrementSpace<NT>& incs;
  const InstDesc& d;
  int R, P;
  S* xg;
  int steps;
  int* flags;
  template <int M, bool FULL>
  __device__ __forceinline__ void run() const {
    using T = double;
    const bool dir = d.bc == kDirichlet;
    const SlotLane l = slot_lane<M, FULL>(static_cast<int>(threadIdx.x), R, P, dir);
    const T half_r = d.r / 2.0, tol = newton_increment_tol<S>();
    T old[M], x[M], al[M], ga[M], de[M];
    // (the Dirichlet values beside the first and last unknown are read in binary64)
    T xl = d.a, xr = d.b;
#pragma unroll
    for (int j = 0; j < M; ++j) old[j] = l.own ? static_cast<T>(xg[l.base + j]) : T(0);
    if (l.own && !l.first) xl = static_cast<T>(xg[l.base == 0 ? R - 1 : l.base - 1]);
    if (l.own && !l.last) xr = static_cast<T>(xg[l.base + M == R ? 0 : l.base + M]);
    int bad = 0;
    // (every lane's reads of the state end before the first solve's barriers, its writes follow the last)
    for (int step = 0; step < steps; ++step) {
#pragma unroll
      for (int j = 0; j < M; ++j) x[j] = old[j];
#pragma unroll 1
      for (int it = 0; it < kNewtonIters; ++it) {
        T y, yp;
        NextChunk<T> next{};
        slot_step<NT, M, FULL>(ws, NewtonSlotRows<M, FULL>{x, old, xl, xr, half_r, d.D, l, bad}, l, P, al, ga, de, y,
                               yp, &next);
        // increments (into de), the new iterate and its neighbours
#pragma unroll
        for (int j = 0; j < M; ++j) {
          de[j] = slot_value<M>(j, al, ga, de, yp, y);
          x[j] = static_cast<T>(static_cast<S>(x[j] + de[j]));
        }
        if (!l.first) xl = static_cast<T>(static_cast<S>(xl + yp));
        if (!l.last)
          xr = static_cast<T>(static_cast<S>(
              xr + __builtin_fma(-next.ga, next.y, __builtin_fma(-next.al, y, next.de))));
      }
      check_increments<NT, M, FULL>(incs, step & 1, l, de, x, old, tol, flags);
#pragma unroll
      for (int j = 0; j < M; ++j) old[j] = x[j];
    }
    if (bad && l.own) flags[0] = 1;
    if (l.own) {
#pragma unroll
      for (int j = 0; j < M; ++j)
        if (FULL || j > 0 || !l.dummy) xg[l.base + j] = static_cast<S>(old[j]);
    }
  }
};

template <typename S, int NT>
__global__ __launch_bounds__(NT, 4) void newton_resident_kernel(const InstDesc* __restrict__ inst,
                                                                const SysDesc* __restrict__ systems,
                                                                S* __restrict__ u, int steps,
                                                                int* __restrict__ flags) {
  using T = double;
  using IS = InterfaceSpace<T, NT>;
  using Inc = IncrementSpace<NT>;
  __shared__ T iface_lds[IS::kBytes / sizeof(T)];
  __shared__ uint64_t iface_votes[2 * IS::kVoteWords], inc_votes[2 * IS::kVoteWords];
  __shared__ unsigned long long groups[2 * Inc::kGroups];
  const IS ws{iface_lds, iface_lds + 3 * NT, iface_votes};
  const Inc incs{groups, groups + Inc::kGroups, inc_votes};
  ws.clear_votes();
  if (threadIdx.x < 2 * IS::kVoteWords) inc_votes[threadIdx.x] = 0;   // (ordered by the first solve's barriers)
  const SysDesc sys = systems[blockIdx.x];
  const InstDesc d = inst[sys.inst];
  const bool dir = d.bc == kDirichlet;
  S* __restrict__ xg = u + d.off + (dir ? 1 : 0);
  if (dir && threadIdx.x == 0) {
    u[d.off] = static_cast<S>(d.a);
    u[d.off + d.n - 1] = static_cast<S>(d.b);
  }
  if (sys.rows == 1) {   // a single Dirichlet unknown
    if (threadIdx.x == 0) {
      const T half_r = d.r / 2.0, tol = newton_increment_tol<S>();
      T old[1] = {static_cast<T>(xg[0])};
      const SlotLane l{0, true, false, true, true};
      int bad = 0;
      for (int step = 0; step < steps; ++step) {
        T x[1] = {old[0]};
        for (int it = 0; it < kNewtonIters; ++it) {
          const NewtonSlotRows<1, true> rows{x, old, d.a, d.b, half_r, d.D, l, bad};
          T al, be, ga, de;
          rows.row(0, 0.0, al, be, ga, de);
          const T delta = de / be;
          x[0] = static_cast<T>(static_cast<S>(x[0] + delta));
          if (it == kNewtonIters - 1 &&
              !(__builtin_fabs(delta) <= tol * __builtin_fmax(__builtin_fabs(x[0]), __builtin_fabs(old[0]))))
            flags[1] = 1;
        }
        old[0] = x[0];
      }
      if (bad) flags[0] = 1;
      xg[0] = static_cast<S>(old[0]);
    }
    return;
  }
  with_slots<NT, 8>(sys.rows, sys.chunks, NewtonRun<S, NT>{ws, incs, d, sys.rows, sys.chunks, xg, steps, flags});
}

template <typename S>
void cn_launch(int lanes, unsigned n, hipStream_t st, const InstDesc* inst, const SysDesc* sys, S* u, int steps) {
  switch (lanes) {
    case 64: cn_resident_kernel<S, 64><<<n, 64, 0, st>>>(inst, sys, u, steps); break;
    case 128: cn_resident_kernel<S, 128><<<n, 128, 0, st>>>(inst, sys, u, steps); break;
    case 256: cn_resident_kernel<S, 256><<<n, 256, 0, st>>>(inst, sys, u, steps); break;
    case 512: cn_resident_kernel<S, 512><<<n, 512, 0, st>>>(inst, sys, u, steps); break;
    default: cn_resident_kernel<S, 1024><<<n, 1024, 0, st>>>(inst, sys, u, steps); break;
  }
}

template <typename S>
void newton_launch(int lanes, unsigned n, hipStream_t st, const InstDesc* inst, const SysDesc* sys, S* u, int steps,
                   int* flags) {
  switch (lanes) {
    case 64: newton_resident_kernel<S, 64><<<n, 64, 0, st>>>(inst, sys, u, steps, flags); break;
    case 128: newton_resident_kernel<S, 128><<<n, 128, 0, st>>>(inst, sys, u, steps, flags); break;
    case 256: newton_resident_kernel<S, 256><<<n, 256, 0, st>>>(inst, sys, u, steps, flags); break;
    case 512: newton_resident_kernel<S, 512><<<n, 512, 0, st>>>(inst, sys, u, steps, flags); break;
    default: newton_resident_kernel<S, 1024><<<n, 1024, 0, st>>>(inst, sys, u, steps, flags); break;
  }
}

}  // namespace

hipError_t launch_cn_resident(const burgers_ctx* ctx, const InstDesc* half, const WgGroup& g, void* u, int steps) {
  if (g.n <= 0 || steps <= 0) return hipSuccess;
  const unsigned n = static_cast<unsigned>(g.n);
  if (ctx->dtype == BURGERS_F64)
    cn_launch<double>(g.shape.lanes, n, ctx->stream, half, g.sys->as<SysDesc>(), static_cast<double*>(u), steps);
  else
    cn_launch<float>(g.shape.lanes, n, ctx->stream, half, g.sys->as<SysDesc>(), static_cast<float*>(u), steps);
  return hipGetLastError();
}

hipError_t launch_newton_resident(const burgers_ctx* ctx, const WgGroup& g, void* u, int steps, int* flags) {
  if (g.n <= 0 || steps <= 0) return hipSuccess;
  const unsigned n = static_cast<unsigned>(g.n);
  const InstDesc* inst = ctx->inst.as<InstDesc>();
  if (ctx->dtype == BURGERS_F64)
    newton_launch<double>(g.shape.lanes, n, ctx->stream, inst, g.sys->as<SysDesc>(), static_cast<double*>(u), steps, flags);
  else
    newton_launch<float>(g.shape.lanes, n, ctx->stream, inst, g.sys->as<SysDesc>(), static_cast<float*>(u), steps, flags);
  return hipGetLastError();
}

// At most 8 rows a lane at every size (see the registers above): 8192 rows on 1024 lanes.
WidthClass chip_width_class(int rows) {
  int lanes = 64;
  while (lanes * 8 < rows) lanes *= 2;
  return WidthClass{lanes, 8};
}

}  // namespace burgers
