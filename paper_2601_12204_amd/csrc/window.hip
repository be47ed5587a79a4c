// BTCS and Crank-Nicolson systems of more than 16384 rows on truncated windows: several steps per launch
// (btcs_deep_kernel) or one (btcs_window_kernel), with the same results to the bit.
//
// A system is cut into chunks of 16 rows (some of 15 where the rows do not divide), at the same rows for every
// window, step and launch.  A window is a run of up to 512 (256) chunks, one per lane, solved
// as a plain system by the interface partition: beyond its two ends the unknowns are taken as zero (at a
// Dirichlet end of the system: the boundary value).  An interface row whose couplings have fallen below
// 2^-54 of its diagonal drops them there and then, and the PCR takes at most S steps (strides 1 to
// 2^(S-1), S <= 4), so a chunk's solution depends on the 2^S chunks on either side and on nothing else: chunks
// that far inside a window are the same in every window that holds them, whatever steps it has taken before.
// A window of several steps therefore only loses 2^S chunks at either end with each, and how a call's steps
// are spread over launches, windows or calls does not show in the results.
//
// Error of a kept row.  Dropping couplings a and c of a row changes its right-hand side by at most (|a| + |c|)
// max|x|.  After s PCR steps they join interface unknowns 2^s chunks, n_s >= 16 2^s - 1 rows, apart, and the influence
// of one of those unknowns on the other is a solution of the rows between that is 1 at one end and 0 at the other:
// with a lower coupling -l_i, an upper one -p_i and d_i - l_i - p_i = 1 in every row, v = theta^k over the distance k
// is above it whenever -l_i + d_i theta - p_i theta^2 >= 0, that is for any theta from the smaller root of that
// quadratic on, which for the BTCS rows (c = r u_i, the couplings D + max(c,0) and D - min(c,0)) is at most
//     g(C) = 2 (D + C) / (1 + 2D + C + sqrt((1 + C)^2 + 4D)),   C = r max|u_i|
// (g increases with C).  So |a| + |c| <= 2 theta^(n_s).  With theta^257 <= 2^-56 that is below 2^-54 after four steps:
// the S-th step cuts nothing that is not negligible by then, and the kept rows are within about 2^-53 max|u^n| of the
// exact ones after every step: a row's couplings are dropped once, for 2^-54 max|u^n|, and reach other rows through
// couplings that add up to 0.3 over the PCR steps.  A smaller S serves a theta with theta^(n_S) <= 2^-56, for the same
// results to the bit.  By the maximum principle max|u| does not grow, so the bound at the start of a call holds for
// all of its steps (up to rounding, which the slack of the limits covers); the state of a Crank-Nicolson step, 2y - u,
// has no such bound: those systems are checked, and stepped, once per launch.
//
// This is the truncation that the whole systems' PCR makes too when it drops couplings below 2^-54 (the decay of
// the inverse of a diagonally dominant tridiagonal matrix, behind truncated SPIKE solvers).  Systems beyond the bound
// are solved exactly by the partition levels.
#include <cmath>

#include "interface.hpp"
#include "internal.hpp"
#include "windows.hpp"

#pragma clang fp contract(off)

namespace burgers {
namespace {

constexpr int kMaxS = kMaxPcr;
constexpr int kWatched = 8;   // beside the PCR steps of an instance's code: a pool's, beyond the bound at the tick's start

// The largest theta for S PCR steps, with slack for rounding (of its own evaluation, and for S < 4 of the growth of
// max|u| by rounding over a call's steps: S = 4 has it in hand).
// S < 4 asks for n_S rows where one instance alone is stepped, and otherwise for a little more: instances run side by
// side, each as many steps a launch as its S allows, so one of a smaller S than the others makes every launch longer
// where the chip is not full.  At ten times the CFL step diffusion alone gives a theta of 0.537: within 63 rows for S = 2
// (0.540), not within 60 (0.524).  (One grid of 2^24 rows, 128 steps: 3.39 ms with 63 rows, 3.60 with 60; 87 problems of
// up to 30484 nodes, 78 steps: 1.50 and 1.42.)
struct ThetaLimits {
  double of[kMaxS];     // S = 1 .. kMaxS: theta^rows <= 2^-56
  double rows[kMaxS];   // 16 2^S - 1 or 15 2^S; S = 4: 257
};
ThetaLimits theta_limits(bool alone = false) {
  ThetaLimits t;
  for (int s = 1; s <= kMaxS; ++s) {
    t.rows[s - 1] = s == kMaxS ? 257 : alone ? (kChunkRows << s) - 1 : (kChunkRows - 1) << s;
    t.of[s - 1] = std::exp2(-56.0 / t.rows[s - 1]) * (1.0 - (s < kMaxS ? 1e-9 : 1e-12));
  }
  return t;
}

// One step per launch.  Every window evaluates the bound from its own rows and flags its instance when it
// fails; the partition levels then redo that instance's step (the old state is still in u).
//
// Bound by HBM and the latency of load, solve and store in turn: 16 x 256 rows per window, so that four
// workgroups a CU overlap them (2^24 rows: 46.4 us, binary32 40.1; with chunks at fixed rows of the window, before a
// chunk's rows were the same in every window, 45.9 and 38.6).
template <typename S, int NT>
__global__ __launch_bounds__(NT, 4) void btcs_window_kernel(
    const InstDesc* __restrict__ inst, const ChunkWin* __restrict__ wins, const S* __restrict__ u,
    S* __restrict__ out, int* __restrict__ flag_now, int* __restrict__ flag_next, double theta_lim) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[WindowSpace<S, NT>::kBytes];
  __shared__ uint64_t iface_votes[2 * InterfaceSpace<double, NT>::kVoteWords];
  __shared__ double wave_max[NT / 64];
  const InterfaceSpace<double, NT> ws{reinterpret_cast<double*>(smem), reinterpret_cast<double*>(smem) + 3 * NT,
                                      iface_votes};
  ws.clear_votes();
  S* stage = reinterpret_cast<S*>(smem);
  const ChunkWin w = wins[blockIdx.x];
  const InstDesc d = inst[w.inst];
  const Frame f(system_rows(d), w);
  const S* __restrict__ x = u + d.off + (d.bc == kDirichlet ? 1 : 0);
  S* __restrict__ y = out + d.off + (d.bc == kDirichlet ? 1 : 0);
  const double M = workgroup_max<NT>(window_load<S, NT, true>(x, stage, f), wave_max);   // (its barrier: the stage is written)
  if (threadIdx.x == 0) {
    flag_next[w.inst] = 0;                     // the next step's slot (its last readers have finished)
    flag_next[-1] = 0;
    if (!(theta_bound(d, M) <= theta_lim)) {
      flag_now[w.inst] = 1;
      flag_now[-1] = 1;
    }
  }
  window_advance<S, NT>(ws, stage, f, w, d, 1, kMaxS, [](const auto&) {});
  window_kept<NT, kStepHalo>(f, w, [&](int k, int i) {
    const S val = stage[padded(i)];
    y[k] = w.cn ? static_cast<S>(2.0 * static_cast<double>(val) - static_cast<double>(x[k])) : val;
  });
  window_ends<S>(f, w, d, out);
}

// Up to kDeepHalo / 2^S steps of each window with the rows on chip, S of its instance (code; 0: the instance
// is left to the partition levels).  A launch beyond an instance's last step does nothing for it.
// WATCH (pools): an instance whose code says so (kWatched) is stepped with the bound checked at every step, from the
// rows it keeps; the steps that fail it are told by its sticky word.
//
// Bound by vector issue like the whole systems on chip (whole.hip), with 512 / (512 - 2 kDeepHalo) of the rows' work, and
// by the window's load and store once per launch, which the CU's other workgroup covers in part.
template <typename S, bool WATCH>
__global__ __launch_bounds__(kDeepLanes, 4) void btcs_deep_kernel(
    const InstDesc* __restrict__ inst, const ChunkWin* __restrict__ wins, const int* __restrict__ code,
    const S* __restrict__ u, S* __restrict__ out, int launch, int nsteps, int* __restrict__ sticky, double theta_lim) {
  constexpr int NT = kDeepLanes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[WindowSpace<S, NT>::kBytes];
  __shared__ uint64_t iface_votes[2 * InterfaceSpace<double, NT>::kVoteWords];
  const InterfaceSpace<double, NT> ws{reinterpret_cast<double*>(smem), reinterpret_cast<double*>(smem) + 3 * NT,
                                      iface_votes};
  ws.clear_votes();
  S* stage = reinterpret_cast<S*>(smem);
  const ChunkWin w = wins[blockIdx.x];
  if (w.count <= 0) return;                    // an empty slot of a resident pool
  const int word = code[w.inst], pcr = WATCH ? word & ~kWatched : word;
  if (pcr <= 0) return;
  int done;
  const int steps = deep_steps(w, pcr, launch, nsteps, done);
  if (steps == 0) return;
  const InstDesc d = inst[w.inst];
  const Frame f(system_rows(d), w);
  const int dir = d.bc == kDirichlet ? 1 : 0;
  window_load<S, NT, false>(u + d.off + dir, stage, f);
  __syncthreads();
  window_advance<S, NT>(ws, stage, f, w, d, steps, pcr, [&](const double (&rows)[kChunkRows]) {
    if constexpr (WATCH) {
      const int t = opaque_lane(static_cast<int>(threadIdx.x));
      if ((word & kWatched) && t >= w.lo && t < w.lo + w.count) {
        Magnitude<double> m;
#pragma unroll
        for (int j = 0; j < kChunkRows; ++j) m.take(rows[j]);
        if (!(theta_bound(d, m.value()) <= theta_lim)) sticky[w.inst] = 1;
      }
    }
  });
  S* __restrict__ y = out + d.off + dir;
  window_kept<NT, kDeepHalo>(f, w, [&](int k, int i) { y[k] = stage[padded(i)]; });
  window_ends<S>(f, w, d, out);
}

// The kept rows of the instances whose last launch left them in `work`, back to u.
template <typename S>
__global__ __launch_bounds__(256) void btcs_settle_kernel(const InstDesc* __restrict__ inst,
                                                          const ChunkWin* __restrict__ wins,
                                                          const int* __restrict__ code, const S* __restrict__ work,
                                                          S* __restrict__ u, int nsteps) {
  const ChunkWin w = wins[blockIdx.x];
  if (w.count <= 0) return;
  const int pcr = code[w.inst] & ~kWatched;
  if (pcr <= 0) return;
  const int per = kDeepHalo >> pcr, total = w.limit > 0 && w.limit < nsteps ? w.limit : nsteps;
  if (((total + per - 1) / per & 1) == 0) return;
  const InstDesc d = inst[w.inst];
  const Frame f(system_rows(d), w);
  const int64_t o = d.off + (d.bc == kDirichlet ? 1 : 0);
  int c = w.first + w.lo;
  if (c >= f.ch.P) c -= f.ch.P;
  const int first = f.ch.base(c), count = f.ch.rows(c, w.count);   // (kept chunks of a window do not wrap)
  for (int i = threadIdx.x; i < count; i += 256) u[o + first + i] = work[o + first + i];
  window_ends<S>(f, w, d, u);
}

// max|u| of every windowed instance over its windows' kept rows, into top[inst] (the bits of a non-negative
// binary64 value, which order like integers).
template <typename S>
__global__ __launch_bounds__(256) void btcs_top_kernel(const InstDesc* __restrict__ inst,
                                                       const ChunkWin* __restrict__ wins, const S* __restrict__ u,
                                                       unsigned long long* __restrict__ top) {
  __shared__ double wave_max[4];
  const ChunkWin w = wins[blockIdx.x];
  if (w.count <= 0) return;
  const InstDesc d = inst[w.inst];
  const Frame f(system_rows(d), w);
  const S* __restrict__ x = u + d.off + (d.bc == kDirichlet ? 1 : 0);
  int c = w.first + w.lo;
  if (c >= f.ch.P) c -= f.ch.P;
  const int first = f.ch.base(c), count = f.ch.rows(c, w.count);
  Magnitude<S> m;
#pragma unroll 8
  for (int i = threadIdx.x; i < count; i += 256) m.take(x[first + i]);
  const double M = workgroup_max<256>(m.value(), wave_max);
  if (threadIdx.x == 0) atomicMax(top + w.inst, __builtin_bit_cast(unsigned long long, M));
}

// Every windowed instance's PCR steps for a call from its bound, and the flags of those beyond it (flags[-1]:
// any), which the partition levels take.  `fresh` (a pool's): there are none, so such an instance steps on, watched, and
// its sticky word (zero from the first tick of its slot's request, fresh, on) tells if a step fails the bound.
// `transposed`: the adjoint's bound.  Leaves `top` cleared for the next call.
__global__ __launch_bounds__(256) void btcs_decide_kernel(const InstDesc* __restrict__ inst,
                                                          const int32_t* __restrict__ members, int n,
                                                          unsigned long long* __restrict__ top,
                                                          int* __restrict__ beyond, int64_t count,
                                                          int* __restrict__ code, int* __restrict__ flags, int* __restrict__ sticky,
                                                          ThetaLimits lim, const int32_t* __restrict__ fresh,
                                                          int transposed) {
  const bool pool = fresh != nullptr;
  bool failed = false;
  for (int k = threadIdx.x; k < n; k += 256) {
    const int i = members[k];
    const InstDesc d = inst[i];
    double M = __builtin_bit_cast(double, top[i]);
    top[i] = 0;
    if (d.bc == kDirichlet) M = __builtin_fmax(M, __builtin_fmax(__builtin_fabs(d.a), __builtin_fabs(d.b)));
    for (int q = 0; q < 3; ++q) beyond[static_cast<int64_t>(q) * count + i] = 0;
    const double theta = theta_bound(d, M), coupling = __builtin_fmax(d.D + d.r * M, 1.0);
    int s = 0;
#pragma unroll
    for (int q = kMaxS; q >= 1; --q) {
      bool holds = theta <= lim.of[q - 1];
      if (transposed)
        holds = holds && (theta == 0.0 || lim.rows[q - 1] * log2(theta) + log2(coupling) <= (q < kMaxS ? -56.0 : -55.0));
      s = holds ? q : s;
    }
    if (pool) {
      if (fresh[i]) sticky[i] = 0;
      code[i] = s == 0 ? kMaxS | kWatched : s;
      flags[i] = 0;
    } else {
      code[i] = s;
      flags[i] = s == 0 ? 1 : 0;
      failed = failed || s == 0;
    }
  }
  const int any = __syncthreads_or(failed);
  if (threadIdx.x == 0) flags[-1] = any ? 1 : 0;
}

template <typename S>
hipError_t deep_launch(const burgers_ctx* ctx, const BtcsPlan& plan, S* u, S* work, int64_t nsteps) {
  const InstDesc* inst = ctx->inst.as<InstDesc>();
  const ChunkWin* wins = plan.deep->as<ChunkWin>();
  const int* code = deep_code(plan.deep_words.as<int>(), ctx->count);
  const unsigned n = static_cast<unsigned>(plan.n_deep);
  S* bufs[2] = {u, work};
  // as many launches as instances with the fewest steps per launch need
  constexpr int kFewest = kDeepHalo >> kMaxS;
  const int64_t launches = (nsteps + kFewest - 1) / kFewest;
  auto kernel = plan.pool ? btcs_deep_kernel<S, true> : btcs_deep_kernel<S, false>;
  int* sticky = win_sticky(plan.win_flags.as<int>(), ctx->count);
  const double lim = btcs_window_limit();
  for (int64_t j = 0; j < launches; ++j)
    kernel<<<n, kDeepLanes, 0, ctx->stream>>>(inst, wins, code, bufs[j & 1], bufs[(j & 1) ^ 1], static_cast<int>(j),
                                              static_cast<int>(nsteps), sticky, lim);
  btcs_settle_kernel<S><<<n, 256, 0, ctx->stream>>>(inst, wins, code, work, u, static_cast<int>(nsteps));
  return hipGetLastError();
}

template <typename S>
hipError_t step_launch(const burgers_ctx* ctx, const BtcsPlan& plan, const InstDesc* inst, const S* u, S* out,
                       int* now, int* next) {
  const unsigned n = static_cast<unsigned>(plan.n_win);
  const double lim = btcs_window_limit();
  const ChunkWin* wins = plan.win->as<ChunkWin>();
  if (plan.win_rows == kChunkRows * 512)
    btcs_window_kernel<S, 512><<<n, 512, 0, ctx->stream>>>(inst, wins, u, out, now, next, lim);
  else
    btcs_window_kernel<S, 256><<<n, 256, 0, ctx->stream>>>(inst, wins, u, out, now, next, lim);
  return hipGetLastError();
}

// Windows of `lanes` chunks that lose `halo` chunks at either end, over a system of R rows.
void chunk_windows(int32_t i, int32_t R, bool periodic, int lanes, int halo, bool cn, std::vector<ChunkWin>& out) {
  const int64_t P = (static_cast<int64_t>(R) + kChunkRows - 1) / kChunkRows, kept = lanes - 2 * halo;
  const int64_t n = (P + kept - 1) / kept, per = (P + n - 1) / n;   // evenly: a window's idle waves cost nothing
  for (int64_t c = 0; c < P; c += per) {
    const int64_t count = std::min(per, P - c);
    const int64_t left = periodic ? halo : std::min<int64_t>(halo, c);
    const int64_t right = periodic ? halo : std::min<int64_t>(halo, P - c - count);
    out.push_back(ChunkWin{i, static_cast<int32_t>((c - left + P) % P), static_cast<uint16_t>(left + count + right),
                           static_cast<uint16_t>(left), static_cast<int32_t>(count), cn ? 1 : 0, 0});
  }
}

}  // namespace

void btcs_step_windows(int32_t i, int32_t R, bool periodic, int rows, bool cn, std::vector<ChunkWin>& out) {
  chunk_windows(i, R, periodic, rows / kChunkRows, kStepHalo, cn, out);
}

void btcs_deep_windows(int32_t i, int32_t R, bool periodic, std::vector<ChunkWin>& out, bool adjoint) {
  chunk_windows(i, R, periodic, kDeepLanes, adjoint ? kAdjDeepHalo : kDeepHalo, false, out);
}

double btcs_window_limit() { return theta_limits().of[kMaxS - 1]; }
double btcs_window_theta(const InstDesc& d, double M) { return theta_bound(d, M); }

int64_t btcs_deep_windows_max(int64_t rows) {
  const int64_t P = (rows + kChunkRows - 1) / kChunkRows, kept = kDeepLanes - 2 * kDeepHalo;
  return (P + kept - 1) / kept;
}

hipError_t launch_btcs_windows(const burgers_ctx* ctx, const BtcsPlan& plan, const InstDesc* inst, const void* u,
                               void* out, int* now, int* next) {
  if (ctx->dtype == BURGERS_F64)
    return step_launch<double>(ctx, plan, inst, static_cast<const double*>(u), static_cast<double*>(out), now, next);
  return step_launch<float>(ctx, plan, inst, static_cast<const float*>(u), static_cast<float*>(out), now, next);
}

hipError_t launch_btcs_bound(const burgers_ctx* ctx, const BtcsPlan& plan, const void* u, const int32_t* fresh) {
  const InstDesc* inst = ctx->inst.as<InstDesc>();
  const ChunkWin* wins = plan.deep->as<ChunkWin>();
  const unsigned n = static_cast<unsigned>(plan.n_deep);
  unsigned long long* top = plan.deep_words.as<unsigned long long>();
  if (ctx->dtype == BURGERS_F64)
    btcs_top_kernel<double><<<n, 256, 0, ctx->stream>>>(inst, wins, static_cast<const double*>(u), top);
  else
    btcs_top_kernel<float><<<n, 256, 0, ctx->stream>>>(inst, wins, static_cast<const float*>(u), top);
  btcs_decide_kernel<<<1, 256, 0, ctx->stream>>>(inst, plan.deep_inst->as<int32_t>(), static_cast<int>(plan.n_deep_inst),
                                                 top, deep_beyond(plan.deep_words.as<int>(), ctx->count), ctx->count,
                                                 deep_code(plan.deep_words.as<int>(), ctx->count),
                                                 win_flag_slot(plan.win_flags.as<int>(), ctx->count, 0),
                                                 win_sticky(plan.win_flags.as<int>(), ctx->count),
                                                 theta_limits(plan.n_deep_inst == 1 && !plan.transposed),
                                                 fresh, plan.transposed ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_btcs_deep(const burgers_ctx* ctx, const BtcsPlan& plan, void* u, void* work, int64_t nsteps) {
  if (ctx->dtype == BURGERS_F64)
    return deep_launch<double>(ctx, plan, static_cast<double*>(u), static_cast<double*>(work), nsteps);
  return deep_launch<float>(ctx, plan, static_cast<float*>(u), static_cast<float*>(work), nsteps);
}

}  // namespace burgers
