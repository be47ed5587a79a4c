// BTCS systems of up to 16384 rows solved whole, one workgroup each, in slots (interface.hpp): on chip for
// every step of a call (btcs_resident_kernel, also recording every state for the adjoint) and one step per
// launch through HBM (btcs_whole_kernel).  Both run the same operations in the same order, so they agree
// bitwise.
//
// What bounds them: vector issue in binary64 (25 instructions per row and step over all, counted at 8192 rows on 512
// lanes, 87% of the slots: five of them the row's assembly, one a quarter-rate reciprocal), and the interface solve, 100
// to 150 of a lane's instructions and four or five barriers a step, which the other workgroups of a CU cover in part.
#include "interface.hpp"
#include "internal.hpp"
#include "staging.hpp"
#include "stencil.hpp"

#pragma clang fp contract(off)

namespace burgers {
namespace {

// Stores one step's rows of a system at x (its first unknown; REC of the resident solver): the lane holds
// its slots in de.  Each wave passes its lanes' slots through a region of LDS of its own, half the wave at a
// time (32 lanes of M slots, one of padding per lane), and stores the rows among them in order, 64
// consecutive slots per instruction.  The region is private to the wave, so no workgroup barrier is
// needed; a wave's LDS accesses are performed in order, which the wavefront-scope fences keep the
// compiler from reordering.
template <typename S, int NT, int M, bool FULL>
__device__ __forceinline__ void record_rows(const double (&de)[M], double* lds, int R, int P, S* __restrict__ x) {
  constexpr int kHalf = 32, kSlots = kHalf * M;
  // (the lane index is formed here, at every step, so that no address of the stores below is kept live
  // across the solve)
  const int lt = opaque_lane(static_cast<int>(threadIdx.x));
  const int lane = lt & 63, wave = lt >> 6;
  double* region = lds + wave * kHalf * (M + 1);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if ((lane >> 5) == h) {
#pragma unroll
      for (int j = 0; j < M; ++j) region[(M + 1) * (lane & 31) + j] = de[j];
    }
    wave_sync();
#pragma unroll 2   // (fully unrolled, the loads held for the stores spill across the solve)
    for (int i = 0; i < (kSlots + 63) / 64; ++i) {
      const int q = lane + 64 * i;
      const int owner = 64 * wave + kHalf * h + q / M, j = q % M;   // the slot's lane and place there
      const double v = region[(M + 1) * (q / M < kHalf ? q / M : 0) + j];
      const SlotLane o = slot_lane<M, FULL>(owner, R, P, false);
      if ((kSlots % 64 == 0 || q < kSlots) && o.own && (j > 0 || !o.dummy)) x[o.base + j] = static_cast<S>(v);
    }
    wave_sync();
  }
}

// Every step of a launch on one system, M slots a lane: x its first unknown in the state buffer.  The state
// is rounded through S once per step as the per-step kernel's store would round it.
template <typename S, int NT, int M, bool FULL, bool REC>
__device__ __forceinline__ void resident_body(const InterfaceSpace<double, NT>& ws, double* rec_lds, const InstDesc& d,
                                              int R, int P, S* __restrict__ x, int steps, S* __restrict__ xr,
                                              int64_t rstride) {
  using T = double;
  const bool dir = d.bc == kDirichlet;
  const SlotLane l = slot_lane<M, FULL>(static_cast<int>(threadIdx.x), R, P, dir);
  const SlotRows rows{d.r, d.D, d.a, d.b};
  T al[M], ga[M], de[M];   // de carries the state between steps
  // (a slot 0 that is no row reads the row before; its value is never used)
#pragma unroll
  for (int j = 0; j < M; ++j) de[j] = l.own ? static_cast<T>(x[l.base + j]) : T(0);
  for (int step = 0; step < steps; ++step) {
    T y, yp;
    slot_step<NT, M, FULL, REC>(ws, rows, l, P, al, ga, de, y, yp);
#pragma unroll
    for (int j = 0; j < M; ++j) de[j] = static_cast<T>(static_cast<S>(slot_value<M>(j, al, ga, de, yp, y)));
    if constexpr (REC) record_rows<S, NT, M, FULL>(de, rec_lds, R, P, xr + step * rstride);
  }
  if constexpr (!REC) {
    if (l.own) {
#pragma unroll
      for (int j = 0; j < M; ++j)
        if (j > 0 || !l.dummy) x[l.base + j] = static_cast<S>(de[j]);
    }
  }
}

template <typename S, int NT, bool REC>
struct ResidentRun {
  const InterfaceSpace<double, NT>& ws;
  double* rec_lds;
  const InstDesc& d;
  int R, P;
  S* x;
  int steps;
  S* xr;
  int64_t rstride;
  template <int M, bool FULL>
  __device__ __forceinline__ void run() const {
    resident_body<S, NT, M, FULL, REC>(ws, rec_lds, d, R, P, x, steps, xr, rstride);
  }
};

// Resident solver: one workgroup keeps one system in registers for all steps of a launch; the state buffer
// is read once and written once (in place).
// REC: the source u is only read, and the state after each step k (1 <= k <= steps) is stored at
// rec + (k - 1) rstride (Dirichlet boundary values included) instead of the final one in place; the
// step's barriers then wait for LDS only, so those stores stay in flight across the next steps.
template <typename S, int NT, int MC, bool REC = false>
__global__ __launch_bounds__(NT, MC == 16 ? 4 : 1) void btcs_resident_kernel(
    const InstDesc* __restrict__ inst, const SysDesc* __restrict__ systems, S* __restrict__ u,
    int steps, S* __restrict__ rec, int64_t rstride) {
  using T = double;
  using IS = InterfaceSpace<T, NT>;
  constexpr int kRecSlots = REC ? (NT / 64) * 32 * (MC + 1) : 1;
  __shared__ T iface_lds[IS::kBytes / sizeof(T)];
  __shared__ uint64_t iface_votes[2 * IS::kVoteWords];
  __shared__ T rec_lds[kRecSlots];
  const IS ws{iface_lds, iface_lds + 3 * NT, iface_votes};
  ws.clear_votes();
  const SysDesc sys = systems[blockIdx.x];
  if (sys.rows <= 0) return;                   // an empty slot of a resident pool
  if (sys.limit > 0 && sys.limit < steps) steps = sys.limit;
  const InstDesc d = inst[sys.inst];
  const bool dir = d.bc == kDirichlet;
  S* __restrict__ x = u + d.off + (dir ? 1 : 0);
  S* __restrict__ xr = REC ? rec + d.off + (dir ? 1 : 0) : nullptr;
  if (dir && threadIdx.x == 0) {
    if constexpr (REC) {
      for (int step = 0; step < steps; ++step) {
        rec[step * rstride + d.off] = static_cast<S>(d.a);
        rec[step * rstride + d.off + d.n - 1] = static_cast<S>(d.b);
      }
    } else {
      u[d.off] = static_cast<S>(d.a);
      u[d.off + d.n - 1] = static_cast<S>(d.b);
    }
  }
  if (sys.rows == 1) {   // a single Dirichlet unknown
    if (threadIdx.x == 0) {
      T v = static_cast<T>(x[0]);
      for (int step = 0; step < steps; ++step) {
        T al, be, ga;
        btcs_row(v, d.r, d.D, al, be, ga);
        const T de = (v - al * d.a) - ga * d.b;
        v = static_cast<T>(static_cast<S>(de / be));
        if constexpr (REC) xr[step * rstride] = static_cast<S>(v);
      }
      if constexpr (!REC) x[0] = static_cast<S>(v);
    }
    return;
  }
  with_slots<NT, MC>(sys.rows, sys.chunks,
                     ResidentRun<S, NT, REC>{ws, rec_lds, d, sys.rows, sys.chunks, x, steps, xr, rstride});
}

// One step of a system whose rows are staged in LDS (row k at padded(k)): solved in slots, the new rows
// written back to the stage (which the interface solve's LDS overlays meanwhile).
template <typename S, int NT>
struct WholeRun {
  const InterfaceSpace<double, NT>& ws;
  const InstDesc& d;
  int R, P;
  S* stage;
  template <int M, bool FULL>
  __device__ __forceinline__ void run() const {
    const SlotLane l = slot_lane<M, FULL>(static_cast<int>(threadIdx.x), R, P, d.bc == kDirichlet);
    double al[M], ga[M], de[M];
#pragma unroll
    for (int j = 0; j < M; ++j) de[j] = l.own ? static_cast<double>(stage[padded(l.base + j)]) : 0.0;
    __syncthreads();                           // every lane's rows read: the interface LDS overlays them
    double y, yp;
    slot_step<NT, M, FULL>(ws, SlotRows{d.r, d.D, d.a, d.b}, l, P, al, ga, de, y, yp);
    __syncthreads();                           // the interface unknowns read before the rows are rewritten
    if (l.own) {
#pragma unroll
      for (int j = 0; j < M; ++j)
        if (j > 0 || !l.dummy) stage[padded(l.base + j)] = static_cast<S>(slot_value<M>(j, al, ga, de, yp, y));
    }
  }
};

// One step of one system per workgroup through HBM: the rows staged through LDS (coalesced loads), solved,
// and stored coalesced, with the Dirichlet boundary nodes.  EXACT: every system has NT x MC rows.  (Compiled with the
// ragged bodies, that one spilled beside them: 1024 x 8192 rows, binary64, 31.2 us a step, 27.6 alone.)
template <typename S, int NT, int MC, bool EXACT = false>
__global__ __launch_bounds__(NT, MC == 16 ? 4 : 1) void btcs_whole_kernel(const InstDesc* __restrict__ inst,
                                                                          const SysDesc* __restrict__ systems,
                                                                          const S* __restrict__ u,
                                                                          S* __restrict__ out) {
  using T = double;
  using IS = InterfaceSpace<T, NT>;
  constexpr int kStageBytes = padded_size(NT * MC) * static_cast<int>(sizeof(S));
  constexpr int kBytes = kStageBytes > IS::kBytes ? kStageBytes : IS::kBytes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kBytes];
  __shared__ uint64_t iface_votes[2 * IS::kVoteWords];
  const IS iws{reinterpret_cast<T*>(smem), reinterpret_cast<T*>(smem) + 3 * NT, iface_votes};
  iws.clear_votes();
  S* stage = reinterpret_cast<S*>(smem);
  const SysDesc sys = systems[blockIdx.x];
  const InstDesc d = inst[sys.inst];
  const bool dir = d.bc == kDirichlet;
  const int R = sys.rows, tid = threadIdx.x;
  const int64_t o = d.off + (dir ? 1 : 0);
  if (dir && tid == 0) {
    out[d.off] = static_cast<S>(d.a);
    out[d.off + d.n - 1] = static_cast<S>(d.b);
  }
  if (!EXACT && R == 1) {   // a single Dirichlet unknown
    if (tid == 0) {
      const T v = static_cast<T>(u[o]);
      T al, be, ga;
      btcs_row(v, d.r, d.D, al, be, ga);
      const T y = ((v - al * d.a) - ga * d.b) / be;
      out[o] = sys.cn ? static_cast<S>(2.0 * static_cast<T>(static_cast<S>(y)) - v) : static_cast<S>(y);
    }
    return;
  }
  stage_in<S, NT, MC>(stage, u + o, R);
  __syncthreads();
  if constexpr (EXACT) WholeRun<S, NT>{iws, d, NT * MC, NT, stage}.template run<MC, true>();
  else with_slots<NT, MC>(R, sys.chunks, WholeRun<S, NT>{iws, d, R, sys.chunks, stage});
  __syncthreads();
  if (sys.cn) stage_out_cn<S, NT, MC>(stage, u + o, out + o, R);
  else stage_out<S, NT, MC>(stage, out + o, R);
}

template <typename S, bool REC>
void resident_launch(const burgers_ctx* ctx, const WgGroup& g, S* u, int steps, S* rec, int64_t rstride) {
  const InstDesc* inst = ctx->inst.as<InstDesc>();
  const SysDesc* sys = g.sys->as<SysDesc>();
  const unsigned n = static_cast<unsigned>(g.n);
  hipStream_t st = ctx->stream;
  const bool hi = g.shape.chunk == 16;
  switch (g.shape.lanes) {
    case 64: btcs_resident_kernel<S, 64, 8, REC><<<n, 64, 0, st>>>(inst, sys, u, steps, rec, rstride); break;
    case 128: btcs_resident_kernel<S, 128, 8, REC><<<n, 128, 0, st>>>(inst, sys, u, steps, rec, rstride); break;
    case 256: btcs_resident_kernel<S, 256, 8, REC><<<n, 256, 0, st>>>(inst, sys, u, steps, rec, rstride); break;
    case 512:
      if (hi) btcs_resident_kernel<S, 512, 16, REC><<<n, 512, 0, st>>>(inst, sys, u, steps, rec, rstride);
      else btcs_resident_kernel<S, 512, 8, REC><<<n, 512, 0, st>>>(inst, sys, u, steps, rec, rstride);
      break;
    default:
      if (hi) btcs_resident_kernel<S, 1024, 16, REC><<<n, 1024, 0, st>>>(inst, sys, u, steps, rec, rstride);
      else btcs_resident_kernel<S, 1024, 8, REC><<<n, 1024, 0, st>>>(inst, sys, u, steps, rec, rstride);
      break;
  }
}

template <typename S>
void whole_launch(const WgGroup& g, hipStream_t st, const InstDesc* inst, const S* u, S* out) {
  const SysDesc* sys = g.sys->as<SysDesc>();
  const unsigned n = static_cast<unsigned>(g.n);
  auto go = [&](auto kernel, int lanes) { kernel<<<n, lanes, 0, st>>>(inst, sys, u, out); };
  const bool hi = g.shape.chunk == 16;
  switch (g.shape.lanes) {
    case 64: go(btcs_whole_kernel<S, 64, 8>, 64); break;
    case 128: go(btcs_whole_kernel<S, 128, 8>, 128); break;
    case 256: go(btcs_whole_kernel<S, 256, 8>, 256); break;
    case 512:
      if (hi) go(g.exact ? btcs_whole_kernel<S, 512, 16, true> : btcs_whole_kernel<S, 512, 16>, 512);
      else go(btcs_whole_kernel<S, 512, 8>, 512);
      break;
    default:
      if (hi) go(g.exact ? btcs_whole_kernel<S, 1024, 16, true> : btcs_whole_kernel<S, 1024, 16>, 1024);
      else go(btcs_whole_kernel<S, 1024, 8>, 1024);
      break;
  }
}

}  // namespace

hipError_t launch_btcs_resident(const burgers_ctx* ctx, const WgGroup& group, void* u, int steps) {
  if (group.n <= 0 || steps <= 0) return hipSuccess;
  if (ctx->dtype == BURGERS_F64) resident_launch<double, false>(ctx, group, static_cast<double*>(u), steps, nullptr, 0);
  else resident_launch<float, false>(ctx, group, static_cast<float*>(u), steps, nullptr, 0);
  return hipGetLastError();
}

// The resident solver recording every step (the adjoint's recompute of a checkpoint segment).
hipError_t launch_btcs_record(const burgers_ctx* ctx, const WgGroup& group, const void* src, void* rec,
                              int64_t rstride, int steps) {
  if (group.n <= 0 || steps <= 0) return hipSuccess;
  if (ctx->dtype != BURGERS_F64) return hipErrorInvalidValue;
  // (the recording kernels only read the source)
  resident_launch<double, true>(ctx, group, static_cast<double*>(const_cast<void*>(src)), steps,
                                static_cast<double*>(rec), rstride);
  return hipGetLastError();
}

hipError_t launch_btcs_whole(const burgers_ctx* ctx, const InstDesc* inst, const WgGroup& group, const void* u,
                             void* out) {
  if (group.n <= 0) return hipSuccess;
  if (ctx->dtype == BURGERS_F64)
    whole_launch<double>(group, ctx->stream, inst, static_cast<const double*>(u), static_cast<double*>(out));
  else
    whole_launch<float>(group, ctx->stream, inst, static_cast<const float*>(u), static_cast<float*>(out));
  return hipGetLastError();
}

}  // namespace burgers
