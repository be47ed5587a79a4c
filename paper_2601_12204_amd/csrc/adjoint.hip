// Discrete adjoint of the two steppers (binary64), for gradients of a loss of the final state with
// respect to the initial state and the viscosity.  The paper obtains such gradients by reverse-mode AD
// through its solvers (Sec. 2.7.1 and 2.7.3); here the derivatives of the discrete steps are written
// out by hand.  The upwind switch is differentiated on its u_i >= 0 branch at u_i = 0, dt is a
// constant, and nu enters through D = nu dt/dx^2 only.  Dirichlet boundary nodes are constants.
//
// Explicit step (Sec. 2.3, eq. 21): the adjoint of u' = E(u) is the transpose of the 3-point Jacobian,
// a gather stencil.  BTCS step (Sec. 2.4, eq. 23): x = A(y)^{-1} y gives
//   mu = A(y)^{-T} lam',   lam = (1 - G) mu,   G_i = r [H (x_i - x_{i-1}) + (1 - H)(x_{i+1} - x_i)],
//   dJ/dD += -sum_i mu_i (2 x_i - x_{i-1} - x_{i+1}),
// with the Dirichlet values standing in as x_0 = a, x_{n-1} = b.  A^T is tridiagonal with the neighbours'
// coefficients (sub p_{i-1}, super l_{i+1}, the cyclic corners swapped).  adjoint_btcs.hip solves it on chip; here are
// the explicit reverse steps and, for the BTCS systems of more than 16384 rows that are beyond the windows' bound, the
// array path: A^T assembled with unit diagonal into binary64 arrays, solved by the partition levels, and finished.
//
// dJ/dD is accumulated in a fixed order, whatever the grouping of steps into launches: per 16 nodes of an explicit
// instance and per chunk of a BTCS system over all steps, per tile of nodes and step on the array path.
#include "internal.hpp"
#include "stencil.hpp"
#include "wave.hpp"

#pragma clang fp contract(off)

namespace burgers {
namespace {

constexpr int kAdjThreads = 256;
constexpr int kAdjLaneNodes = 4;                          // BTCS tiles: consecutive nodes per lane
constexpr int kAdjTile = kAdjThreads * kAdjLaneNodes;     // nodes of one BTCS adjoint tile (one dJ/dD slot)

// Sum over the workgroup in a fixed order (a butterfly within each wave, lane 0's result, then the waves
// in order), so that the per-tile partials of dJ/dD are deterministic.  Valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v = v + __shfl_xor(v, m, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double tot = red[0];
#pragma unroll
  for (int w = 1; w < kAdjThreads / 64; ++w) tot = tot + red[w];
  return tot;
}

// ---- Explicit reverse steps ---------------------------------------------------------------------------
// lam^k = (dE/du at u^k)^T lam^(k+1).  With beta_i = max(r u_i + D, D) and alpha_i = beta_i - r u_i, the weights of the
// forward update u' = u + alpha (u_p - u) - beta (u - u_m), a node hands q_i = beta_i lam_i to its left neighbour and
// p_i = alpha_i lam_i to its right one:
//   lam'_i = lam_i - p_i - q_i - r s_i lam_i + q_{i+1} + p_{i-1},   s_i = u_i >= 0 ? u_i - u_{i-1} : u_{i+1} - u_i.
//
// A wave holds lam over a window of up to 1024 nodes (16 consecutive ones per lane) in registers for a run of
// reverse steps, and passes end values between lanes by whole-wave DPP moves: a step needs no LDS and no barrier.
// Of the states only every kAdjGroup-th is recorded and read; the ones between are computed again in registers,
// by the forward kernels' operations (so to the bit), and used in turn.  Windows keep their middle nodes and carry
// kAdjHalo nodes on either side (a short periodic instance's halo goes around it several times); an error at a
// window's edge travels one node per reverse step, after kAdjGroup - 1 nodes of the first states' own, so a launch
// takes at most kAdjRun = kAdjHalo - (kAdjGroup - 1) steps, rounded down to whole groups.
//
// dJ/dD, the sum over nodes and steps of lam^(k+1)_j (u_{j+1} + u_{j-1} - 2 u_j), is accumulated per lane over its 16
// nodes and all steps, in a slot per 16 nodes of the instance that carries the sum from launch to launch.  Lanes hold
// the same 16 nodes in every window that keeps them, so the gradient does not depend on how the steps are grouped into
// launches (the checkpoint interval).
//
// Bound by vector issue: 31 instructions per node and step (counted, 92% of the slots; 26 per node of a window, about 4.5
// of them the states' second computation, and one in six of a window's nodes halo or beyond it).  (256 x 16384 nodes, us per reverse step, the recording of the states on another stream included: 7 here;
// 18 with every state recorded and read, 8 + 8 bytes per node and step, by workgroups of 256 lanes with
// an exchange and a barrier a step.)
constexpr int kAdjChunk = 16;
constexpr int kAdjRegion = 32 * (kAdjChunk + 1);   // a half-wave's chunks, padded by one per chunk
static_assert(64 * kAdjChunk == kAdjWinNodes && kAdjChunk == kAdjSumNodes, "window layout");
static_assert(kAdjRun % kAdjGroup == 0 && kAdjRun + kAdjGroup - 1 <= kAdjHalo, "run of a launch");

__device__ __forceinline__ int fresh_lane() { return opaque_lane(static_cast<int>(threadIdx.x) & 63); }

__device__ __forceinline__ double from_left(double x) { return wave_move<0x13C>(x); }
__device__ __forceinline__ double from_right(double x) { return wave_move<0x134>(x); }

// Instance nodes of the window nodes lane, lane + 64, lane + 128, ...: an instance shorter than the window is gone
// around as often as it takes (beyond a Dirichlet window's end the nodes are any).
struct NodeWalk {
  int g, step, n;
  __device__ __forceinline__ NodeWalk(const AdjWindow& w, int nodes, int lane) : g(w.first + lane), n(nodes) {
    step = n >= 64 ? 64 : 64 % n;
    if (g >= n) g = n >= 64 ? g - n : g % n;
  }
  __device__ __forceinline__ int next() {
    const int now = g;
    g += step;
    g = g >= n ? g - n : g;
    return now;
  }
};

// Window nodes of src (the instance's first node) for the lane's chunk [16 t, 16 t + 16), in two steps so
// that the loads can be issued long before their values are needed: window_fetch loads 64 consecutive window
// nodes per instruction into v; window_spread passes them to the lanes' chunks, half the wave at a time, through the
// wave's region of LDS.
__device__ __forceinline__ void window_fetch(const double* __restrict__ src, const AdjWindow& w, int n,
                                             double (&v)[kAdjChunk]) {
  const int lane = fresh_lane();
  if (w.first + kAdjWinNodes <= n) {           // (uniform) one address
    const double* __restrict__ p = src + w.first;
#pragma unroll
    for (int i = 0; i < kAdjChunk; ++i) v[i] = p[lane + 64 * i];
    return;
  }
  NodeWalk at(w, n, lane);
#pragma unroll
  for (int i = 0; i < kAdjChunk; ++i) v[i] = src[at.next()];
}

__device__ __forceinline__ void window_spread(const double (&v)[kAdjChunk], double* region, double (&out)[kAdjChunk]) {
  const int lane = fresh_lane();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int i = 0; i < 8; ++i) region[apad(lane) + 68 * i] = v[8 * h + i];   // (apad(lane + 64 i))
    wave_sync();
    if ((lane >> 5) == h) {
#pragma unroll
      for (int j = 0; j < kAdjChunk; ++j) out[j] = region[17 * (lane & 31) + j];   // (apad)
    }
    wave_sync();
  }
}

// The lane's chunk to the window's kept nodes of dst (the instance's first node), the way back.
__device__ __forceinline__ void window_store(const double (&x)[kAdjChunk], const AdjWindow& w, int n, double* region,
                                             double* __restrict__ dst) {
  const int lane = fresh_lane();
  NodeWalk at(w, n, lane);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if ((lane >> 5) == h) {
#pragma unroll
      for (int j = 0; j < kAdjChunk; ++j) region[17 * (lane & 31) + j] = x[j];   // (apad)
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = 512 * h + lane + 64 * i, node = at.next();
      const double v = region[apad(lane) + 68 * i];
      if (k >= w.lo && k < w.lo + w.count) dst[node] = v;
    }
    wave_sync();
  }
}

// What a lane knows of its chunk.  EDGE: the window holds a Dirichlet node or keeps part of a chunk.
struct AdjLane {
  double r, D;
  bool first;   // node 0 of a Dirichlet instance is the chunk's first
  int last;     // place of its node n - 1 in the chunk, or none (negative or beyond)
  int kept;     // kept nodes: a prefix of the chunk
  template <bool EDGE>
  __device__ __forceinline__ bool fixed(int j) const {
    return EDGE && ((j == 0 && first) || j == last);
  }
};

// The state after u.
template <bool EDGE>
__device__ __forceinline__ void adj_forward(const double (&u)[kAdjChunk], double (&x)[kAdjChunk], const AdjLane& l) {
  const double left = from_left(u[kAdjChunk - 1]), right = from_right(u[0]);
#pragma unroll
  for (int j = 0; j < kAdjChunk; ++j) {
    const double um = j > 0 ? u[j > 0 ? j - 1 : 0] : left;
    const double up = j < kAdjChunk - 1 ? u[j < kAdjChunk - 1 ? j + 1 : j] : right;
    const double v = upwind_central(u[j], um, up, l.r, l.D);
    x[j] = l.fixed<EDGE>(j) ? u[j] : v;
    if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
}

// lam at the step from u, in place, and its terms of dJ/dD.
template <bool EDGE>
__device__ __forceinline__ void adj_back(double (&u)[kAdjChunk], double (&lam)[kAdjChunk], double& g, const AdjLane& l) {
  constexpr int M = kAdjChunk;
  // (opaque, or the compiler keeps adj_forward's differences and weights of u for this and spills)
#pragma unroll
  for (int j = 0; j < M; ++j) asm volatile("" : "+v"(u[j]));
  const double left = from_left(u[M - 1]), right = from_right(u[0]);
  auto weights = [&](int j, double& p, double& q) {
    const double be = __builtin_fmax(__builtin_fma(l.r, u[j], l.D), l.D);
    p = __builtin_fma(-l.r, u[j], be) * lam[j];
    q = be * lam[j];
    if (l.fixed<EDGE>(j)) p = q = 0.0;
  };
  double p, q, pl, ql;
  weights(M - 1, pl, ql);
  weights(0, p, q);
  double pm = from_left(pl);                 // p of the node before
  const double q_right = from_right(q);
  double dm = u[0] - left;                   // u_j - u_{j-1}
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const double um = j > 0 ? u[j > 0 ? j - 1 : 0] : left, up = j < M - 1 ? u[j < M - 1 ? j + 1 : j] : right;
    const double dp = up - u[j];
    double pn = 0.0, qn = q_right;
    if (j + 2 < M) weights(j + 1, pn, qn);
    else if (j + 2 == M) {
      pn = pl;
      qn = ql;
    }
    const double own = u[j] >= 0.0 ? dm : dp, lj = lam[j];
    double t = (lj - p) - q;
    t = __builtin_fma(-own, l.r * lj, t);
    t = (t + qn) + pm;
    const double lap = fma_exact(-2.0, u[j], up + um);   // (rounded as eq. 4 reads, like the oracle's)
    if constexpr (EDGE) g = j < l.kept ? __builtin_fma(lj, lap, g) : g;
    else g = __builtin_fma(lj, lap, g);
    lam[j] = l.fixed<EDGE>(j) ? 0.0 : t;
    pm = p;
    p = pn;
    q = qn;
    dm = dp;
    // (a few nodes at a time, or the scheduler forms every node's terms up front and spills)
    if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
}

// Reverse steps k = k_hi - 1 down to k_lo (a multiple of kAdjGroup) of a segment: the states u^k with k a multiple of
// kAdjGroup at u0 for k = 0, else at useg + (k - 1) ustride; lam^(k_hi) from lamp, lam^(k_lo) to lam (the kept
// nodes).  One window per wave.
template <bool EDGE>
__global__ __launch_bounds__(256, 2) void adj_explicit_kernel(
    const InstDesc* __restrict__ inst, const AdjWindow* __restrict__ wins, int n_wins, const double* __restrict__ u0,
    const double* __restrict__ useg, int64_t ustride, int k_lo, int k_hi, const double* __restrict__ lamp,
    double* __restrict__ lam, double* __restrict__ gslot) {
  constexpr int M = kAdjChunk;
  __shared__ double lds[4 * kAdjRegion];
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int index = 4 * static_cast<int>(blockIdx.x) + wave;
  if (index >= n_wins) return;
  double* region = lds + wave * kAdjRegion;
  const AdjWindow w = wins[index];
  const InstDesc d = inst[w.inst];
  const int n = d.n, at = M * (static_cast<int>(threadIdx.x) & 63);
  const bool dir = EDGE && d.bc == kDirichlet;
  const AdjLane l{d.r, d.D, dir && w.first + at == 0, dir ? n - 1 - w.first - at : -1,
                  at >= w.lo ? w.lo + w.count - at : 0};
  const int slot = w.slot0 + (at - w.lo) / M;
  double g = l.kept > 0 ? gslot[slot] : 0.0;
  auto state = [&](int k) { return (k == 0 ? u0 : useg + static_cast<int64_t>(k - 1) * ustride) + d.off; };
  auto ends = [&](double (&x)[M], double a, double b) {   // the fixed nodes' values
    if constexpr (EDGE) {
#pragma unroll
      for (int j = 0; j < M; ++j) {
        if (j == 0 && l.first) x[j] = a;
        if (j == l.last) x[j] = b;
      }
    }
  };
  double L[M], U0[M], U1[M], U2[M], U3[M], V[M];
  window_fetch(lamp + d.off, w, n, V);
  window_spread(V, region, L);
  ends(L, 0.0, 0.0);
  static_assert(kAdjGroup == 4, "a group's states");
  int k = (k_hi - 1) / kAdjGroup * kAdjGroup;
  window_fetch(state(k), w, n, V);
  for (int top = k_hi - k; k >= k_lo; k -= kAdjGroup, top = kAdjGroup) {   // steps k + top - 1 .. k
    window_spread(V, region, U0);
    ends(U0, d.a, d.b);
    if (top > 1) adj_forward<EDGE>(U0, U1, l);
    if (top > 2) adj_forward<EDGE>(U1, U2, l);
    if (top > 3) adj_forward<EDGE>(U2, U3, l);
    // the next group's state is in flight during this one's reverse steps
    if (k > k_lo) window_fetch(state(k - kAdjGroup), w, n, V);
    if (top > 3) adj_back<EDGE>(U3, L, g, l);
    if (top > 2) adj_back<EDGE>(U2, L, g, l);
    if (top > 1) adj_back<EDGE>(U1, L, g, l);
    adj_back<EDGE>(U0, L, g, l);
  }
  window_store(L, w, n, region, lam + d.off);
  if (l.kept > 0) gslot[slot] = g;
}

// Row k of A(y)^T, normalised by its diagonal, and the right-hand side lamp / d, for every unknown of
// the tile's instance; written at t.sys_off of the adjoint arrays.
__global__ __launch_bounds__(kAdjThreads) void adj_btcs_assemble_kernel(
    const InstDesc* __restrict__ inst, const AdjTile* __restrict__ tiles, const double* __restrict__ u,
    const double* __restrict__ lamp, double* __restrict__ LA, double* __restrict__ LC,
    double* __restrict__ LD, const int* __restrict__ only) {
  if (only && only[-1] == 0) return;          // every instance is within its windows' bound
  const AdjTile t = tiles[blockIdx.x];
  if (only && only[t.inst] == 0) return;      // this instance's windows held
  const InstDesc d = inst[t.inst];
  const int n = t.n;
  const bool periodic = t.bc == kPeriodic;
  const int first = periodic ? 0 : 1;
  const int m = periodic ? n : n - 2;
  for (int q = 0; q < kAdjLaneNodes; ++q) {
  const int node = t.start + static_cast<int>(threadIdx.x) + q * kAdjThreads;
  const int k = node - first;   // unknown index of this node
  if (node >= n || k < 0 || k >= m) continue;
  const double* __restrict__ y = u + t.off;
  double sub, diag, sup, tmp1, tmp2;
  btcs_row(y[first + k], d.r, d.D, sub, diag, sup);
  double sub_t = 0.0, sup_t = 0.0;   // p_{k-1} and l_{k+1}
  if (periodic || k > 0) {
    const int km = k == 0 ? m - 1 : k - 1;
    btcs_row(y[first + km], d.r, d.D, tmp1, tmp2, sub_t);
  }
  if (periodic || k < m - 1) {
    const int kp = k == m - 1 ? 0 : k + 1;
    btcs_row(y[first + kp], d.r, d.D, sup_t, tmp1, tmp2);
  }
  const int64_t o = t.sys_off + k;
  LA[o] = sub_t / diag;
  LC[o] = sup_t / diag;
  LD[o] = lamp[t.off + first + k] / diag;
  }
}

// lam = (1 - G) mu and the tile's partial -mu . (L x); boundary nodes get zero.
__global__ __launch_bounds__(kAdjThreads) void adj_btcs_finish_kernel(
    const InstDesc* __restrict__ inst, const AdjTile* __restrict__ tiles, const double* __restrict__ u,
    const double* __restrict__ x, const double* __restrict__ X, double* __restrict__ lam,
    double* __restrict__ gslot, const int* __restrict__ only) {
  __shared__ double red[kAdjThreads / 64];
  if (only && only[-1] == 0) return;          // every instance is within its windows' bound
  const AdjTile t = tiles[blockIdx.x];
  if (only && only[t.inst] == 0) return;
  const InstDesc d = inst[t.inst];
  const int n = t.n;
  const bool periodic = t.bc == kPeriodic;
  double g = 0.0;
  for (int q = 0; q < kAdjLaneNodes; ++q) {
  const int j = t.start + static_cast<int>(threadIdx.x) + q * kAdjThreads;
  if (j < n) {
    double out = 0.0;
    if (periodic || (j > 0 && j < n - 1)) {
      const double* __restrict__ xs = x + t.off;
      const int first = periodic ? 0 : 1;
      const double mu = X[t.sys_off + (j - first)];
      const double xm = periodic ? xs[j == 0 ? n - 1 : j - 1] : (j == 1 ? d.a : xs[j - 1]);
      const double xp = periodic ? xs[j == n - 1 ? 0 : j + 1] : (j == n - 2 ? d.b : xs[j + 1]);
      const double xj = xs[j];
      const double G = u[t.off + j] >= 0.0 ? d.r * (xj - xm) : d.r * (xp - xj);
      out = (1.0 - G) * mu;
      g = g - mu * ((2.0 * xj - xm) - xp);
    }
    lam[t.off + j] = out;
  }
  }
  const double tot = block_sum(g, red);
  if (threadIdx.x == 0) gslot[t.slot] = gslot[t.slot] + tot;
}

// grad_nu[i] = (sum of instance i's slots) * dt/dx^2, a workgroup per instance: each lane's every 256th slot in
// order, then the lanes in a fixed order.
__global__ __launch_bounds__(kAdjThreads) void adj_nu_kernel(const InstDesc* __restrict__ inst,
                                                             const int32_t* __restrict__ slot_begin,
                                                             const double* __restrict__ gslot,
                                                             double* __restrict__ grad_nu) {
  __shared__ double red[kAdjThreads / 64];
  const int i = blockIdx.x;
  double s = 0.0;
  for (int k = slot_begin[i] + static_cast<int>(threadIdx.x); k < slot_begin[i + 1]; k += kAdjThreads) s = s + gslot[k];
  s = block_sum(s, red);
  if (threadIdx.x == 0) grad_nu[i] = s * inst[i].dtdx2;
}

// Dirichlet boundary nodes carry no gradient.
__global__ void zero_ends_kernel(const InstDesc* __restrict__ inst, double* __restrict__ g, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const InstDesc d = inst[i];
  if (d.bc == kDirichlet) {
    g[d.off] = 0.0;
    g[d.off + d.n - 1] = 0.0;
  }
}

__global__ void fill_kernel(double* __restrict__ p, int64_t n, double v) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

}  // namespace

int adjoint_tile_nodes() { return kAdjTile; }

hipError_t launch_adj_explicit(const burgers_ctx* ctx, const AdjWindow* wins, int64_t n_wins, int64_t n_inner,
                               const double* u0, const double* useg, int64_t ustride, int k_lo, int k_hi,
                               const double* lamp, double* lam, double* gslot) {
  if (n_wins <= 0 || k_hi <= k_lo) return hipSuccess;
  const int inner = static_cast<int>(n_inner), edge = static_cast<int>(n_wins - n_inner);
  if (inner > 0)
    adj_explicit_kernel<false><<<static_cast<unsigned>((inner + 3) / 4), 256, 0, ctx->stream>>>(
        ctx->inst.as<InstDesc>(), wins, inner, u0, useg, ustride, k_lo, k_hi, lamp, lam, gslot);
  if (edge > 0)
    adj_explicit_kernel<true><<<static_cast<unsigned>((edge + 3) / 4), 256, 0, ctx->stream>>>(
        ctx->inst.as<InstDesc>(), wins + n_inner, edge, u0, useg, ustride, k_lo, k_hi, lamp, lam, gslot);
  return hipGetLastError();
}

hipError_t launch_adj_btcs_assemble(const burgers_ctx* ctx, const AdjTile* tiles, int64_t n_tiles,
                                    const double* u, const double* lamp, double* LA, double* LC, double* LD,
                                    const int* only) {
  if (n_tiles <= 0) return hipSuccess;
  adj_btcs_assemble_kernel<<<static_cast<unsigned>(n_tiles), kAdjThreads, 0, ctx->stream>>>(
      ctx->inst.as<InstDesc>(), tiles, u, lamp, LA, LC, LD, only);
  return hipGetLastError();
}

hipError_t launch_adj_btcs_finish(const burgers_ctx* ctx, const AdjTile* tiles, int64_t n_tiles,
                                  const double* u, const double* x, const double* X, double* lam,
                                  double* gslot, const int* only) {
  if (n_tiles <= 0) return hipSuccess;
  adj_btcs_finish_kernel<<<static_cast<unsigned>(n_tiles), kAdjThreads, 0, ctx->stream>>>(
      ctx->inst.as<InstDesc>(), tiles, u, x, X, lam, gslot, only);
  return hipGetLastError();
}

hipError_t launch_adj_nu(const burgers_ctx* ctx, const int32_t* slot_begin, const double* gslot,
                         double* grad_nu) {
  adj_nu_kernel<<<static_cast<unsigned>(ctx->count), kAdjThreads, 0, ctx->stream>>>(ctx->inst.as<InstDesc>(), slot_begin,
                                                                                    gslot, grad_nu);
  return hipGetLastError();
}

hipError_t launch_zero_dirichlet_ends(const burgers_ctx* ctx, double* g) {
  const int count = static_cast<int>(ctx->count);
  zero_ends_kernel<<<(count + 255) / 256, 256, 0, ctx->stream>>>(ctx->inst.as<InstDesc>(), g, count);
  return hipGetLastError();
}

hipError_t launch_fill(const burgers_ctx* ctx, double* p, int64_t n, double v) {
  if (n <= 0) return hipSuccess;
  fill_kernel<<<static_cast<unsigned>((n + 255) / 256), 256, 0, ctx->stream>>>(p, n, v);
  return hipGetLastError();
}

}  // namespace burgers
