// BTCS step (Sec. 2.4, eq. 23) for gfx950: one tridiagonal solve A(u^n) u^{n+1} = u^n per step, cyclic
// for periodic instances, with the Dirichlet boundary values moved to the right-hand side.
//
// Thomas' recurrence is serial, so the solve is split by the partition method:
//   1. Each thread owns a contiguous chunk of rows.  Eliminating the chunk's interior expresses every
//      row through the chunk's first unknown F and last unknown E, and leaves two rows per chunk that
//      couple only F_k, E_k and the neighbouring chunks' E_{k-1}, F_{k+1}: a tridiagonal system of
//      2P rows over (F_0, E_0, F_1, E_1, ...), cyclic whenever the original one is.
//   2. That reduced system is solved by cyclic parallel cyclic reduction (PCR) in LDS when it is small,
//      or reduced again by the same chunk elimination in a further level (long systems).
//   3. Each chunk recovers its interior rows from F and E.
// Rows are assembled on the fly from u^n (no coefficient arrays in HBM).  The reduced systems have
// unit diagonals and |sub| + |super| < 1, since A is strictly diagonally dominant (row sums 1), so no
// pivoting is needed at any level.
//
// Arithmetic is binary64 for both state types; a binary32 state is widened on load and rounded once per
// step on store.  A binary32 partition solve drifts by a systematic bias of a few ulp per step, which
// over 10^3 steps exceeds the serial binary32 solve's own error; the binary64 solve keeps the binary32
// path within its one rounding per step of the exact discrete solution.  Binary64 instructions issue at
// half the binary32 rate on gfx950, but the solve is bound by its pivot chain's latency and its barriers
// rather than by issue rate: a binary32-state step takes about as long as a binary64 one.
#include <algorithm>
#include <cmath>

#include "interface.hpp"
#include "internal.hpp"
#include "newton_check.hpp"
#include "staging.hpp"
#include "stencil.hpp"
#include "windows.hpp"

#pragma clang fp contract(off)

namespace burgers {
namespace {

constexpr int kWgThreads = 512;   // threads of the whole-system solver
constexpr int kWgChunk = 16;      // longest chunk a thread of the whole-system solver eliminates
constexpr int kWgRows = kWgThreads * kWgChunk;            // longest system of the exact 512 x 16 kernels
constexpr int kWholeRows = 2 * kWgRows;                   // longest system solved whole (1024 lanes x 16)
constexpr int kRedRows = kReduceBlock * kRedChunk;        // rows one partition workgroup stages

// Row sources of the chunk elimination.  row() returns row k as assembled; boundary() then folds the
// Dirichlet values into the reduced rows of the chunk that holds the first or last row of the system
// (only level-0 systems of Dirichlet instances have such values; every other source has none).

// Rows of a reduced system stored with unit diagonal.
template <typename T>
struct ArrayRows {
  const T* __restrict__ A;
  const T* __restrict__ C;
  const T* __restrict__ Dv;
  __device__ __forceinline__ void row(int, int k, int, T& al, T& be, T& ga, T& de) const {
    al = A[k];
    be = T(1);
    ga = C[k];
    de = Dv[k];
  }
  __device__ __forceinline__ void boundary(int, int, int, T&, T&, T&, T&) const {}
};

// Rows of a reduced system preloaded into registers: a lane issues all its loads before the elimination
// starts instead of waiting for one row's loads at every step of the pivot chain.
template <typename T, int M>
struct RegRows {
  T a[M], c[M], d[M];
  __device__ __forceinline__ void load(const T* __restrict__ A, const T* __restrict__ C,
                                       const T* __restrict__ D, int s, int m) {
#pragma unroll
    for (int j = 0; j < M; ++j) {
      if (j < m) {
        a[j] = A[s + j];
        c[j] = C[s + j];
        d[j] = D[s + j];
      }
    }
  }
  __device__ __forceinline__ void row(int j, int, int, T& al, T& be, T& ga, T& de) const {
    al = a[j];
    be = T(1);
    ga = c[j];
    de = d[j];
  }
  __device__ __forceinline__ void boundary(int, int, int, T&, T&, T&, T&) const {}
};

// Rows of a level-0 system whose old values sit in LDS (staged coalesced from HBM); row k is held at
// padded(k - base).
template <typename S>
struct LdsRows {
  const S* st;
  int base;
  double r, D;
  DirichletEnds ends;
  __device__ __forceinline__ void row(int, int k, int, double& al, double& be, double& ga, double& de) const {
    const double ui = static_cast<double>(st[padded(k - base)]);
    btcs_row(ui, r, D, al, be, ga);
    de = ui;
  }
  __device__ __forceinline__ void boundary(int s, int m, int R, double& AF, double& DF, double& CE,
                                           double& DE) const {
    ends.apply(s, m, R, AF, DF, CE, DE);
  }
};

template <typename S>
struct LdsDst {
  S* st;
  int base;
  __device__ __forceinline__ void write(int, int k, double v) const { st[padded(k - base)] = static_cast<S>(v); }
};

// Reduced systems of at least this many rows are read and written by the workgroup solver through LDS
// (coalesced); smaller ones lane by lane, which saves the transposes' barriers.
constexpr int kCoalesceRows = 2048;

// Rows held coalesced (lane t: rows t + j NT) to the lanes' chunks (lane t < P: rows s..s+m-1) through
// the LDS buffer `st`; ends with a barrier, so the next call may reuse the buffer.
template <typename T, int NT, int MC>
__device__ __forceinline__ void stage_transpose(T* st, const T (&v)[MC], int R, int P, int s, int m, T (&out)[MC]) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int j = 0; j < MC; ++j) {
    const int i = tid + j * NT;
    if (i < R) st[padded(i)] = v[j];
  }
  __syncthreads();
  if (tid < P) {
#pragma unroll
    for (int j = 0; j < MC; ++j)
      if (j < m) out[j] = st[padded(s + j)];
  }
  __syncthreads();
}

// Chunk elimination.  Rows s..s+m-1 (2 <= m <= M) of a system with R rows.  On return, for
// 1 <= j <= m-2, row j reads  x_j + al[j] F + ga[j] E = de[j]  with F = x_0, E = x_{m-1}, and the two
// reduced rows are
//   F row:  AF * E_prev + F + CF * E      = DF
//   E row:  AE * F      + E + CE * F_next = DE.
template <typename T, int M, typename Src>
__device__ __forceinline__ void chunk_eliminate(const Src& src, int s, int m, int R, T (&al)[M],
                                                T (&ga)[M], T (&de)[M], T& AF, T& CF, T& DF, T& AE,
                                                T& CE, T& DE) {
  T a0, b0, c0, d0;
  src.row(0, s, R, a0, b0, c0, d0);
  // forward: x_j + al[j] x_0 + ga[j] x_{j+1} = de[j]
#pragma unroll
  for (int j = 1; j < M; ++j) {
    if (j < m) {
      T aj, bj, cj, dj;
      src.row(j, s + j, R, aj, bj, cj, dj);
      // (binary64 only: one reciprocal per pivot; in binary32, scaling all three coefficients by one
      // rounded reciprocal biases the row enough to accumulate over many steps)
      if (j == 1) {
        const T inv = recip(bj);
        al[1] = aj * inv;
        ga[1] = cj * inv;
        de[1] = dj * inv;
      } else {
        const T inv = recip(__builtin_fma(-aj, ga[j - 1], bj));
        const T ai = aj * inv;
        al[j] = -(ai * al[j - 1]);
        ga[j] = cj * inv;
        de[j] = __builtin_fma(-ai, de[j - 1], dj * inv);
      }
      if (j == m - 1) {
        AE = al[j];
        CE = ga[j];
        DE = de[j];
      }
    }
  }
  // backward: x_j + al[j] x_0 + ga[j] x_{m-1} = de[j]  (row m-2 already has this form)
#pragma unroll
  for (int j = M - 3; j >= 1; --j) {
    if (j <= m - 3) {
      const T g = ga[j];
      de[j] = __builtin_fma(-g, de[j + 1], de[j]);
      al[j] = __builtin_fma(-g, al[j + 1], al[j]);
      ga[j] = -(g * ga[j + 1]);
    }
  }
  // row 0 with x_1 eliminated (for m == 2, x_1 is E itself)
  T a1 = T(0), g1 = T(-1), d1 = T(0);
  if (m > 2) {
    a1 = al[1];
    g1 = ga[1];
    d1 = de[1];
  }
  const T inv0 = recip(__builtin_fma(-c0, a1, b0));
  const T ci = c0 * inv0;
  AF = a0 * inv0;
  CF = -(ci * g1);
  DF = __builtin_fma(-ci, d1, d0 * inv0);
  src.boundary(s, m, R, AF, DF, CE, DE);
}

// Interior rows from the chunk's end values.
template <typename T, int M, typename Dst>
__device__ __forceinline__ void chunk_recover(const Dst& dst, int s, int m, const T (&al)[M],
                                              const T (&ga)[M], const T (&de)[M], T F, T E) {
  dst.write(0, s, F);
#pragma unroll
  for (int j = 1; j < M; ++j) {
    if (j < m - 1) dst.write(j, s + j, __builtin_fma(-ga[j], E, __builtin_fma(-al[j], F, de[j])));
    if (j == m - 1) dst.write(j, s + j, E);
  }
}

template <typename S>
struct PtrDst {
  S* __restrict__ x;
  __device__ __forceinline__ void write(int, int k, double v) const { x[k] = static_cast<S>(v); }
};

// Workspace of pcr_pairs in LDS: two buffers of three arrays (sub, super, rhs) of 2 NT rows, and one flag
// per wave for each buffer.
template <typename T, int NT>
struct PcrSpace {
  static constexpr int kRows = 2 * NT;
  static constexpr int kWaves = (NT + 63) / 64;
  T* rows;     // 2 buffers x 3 arrays x kRows
  int* flags;  // 2 buffers x kWaves
  static constexpr int kBytes = 2 * 3 * kRows * static_cast<int>(sizeof(T));
};

// Cyclic PCR on the 2P reduced rows of P chunks (P a power of two, P <= NT), every row normalised to a
// unit diagonal:  A_i x_{i-s} + x_i + C_i x_{i+s} = D_i.  Lane t < P owns rows 2t (its chunk's F row) and
// 2t+1 (its E row) and keeps them in registers; each step publishes them to LDS, F rows at [0, P) and E
// rows at [P, 2P), so the partners of either row at any distance sit at consecutive positions across
// the wave.  Indices wrap modulo 2P; a non-cyclic system simply carries zero corner couplings.  After
// log2(2P) steps every row couples only to itself and the solution is D / (1 + A + C); the reduction
// stops earlier once every coupling of every row is negligible, and the solution is then D.
// The steps alternate between the two buffers, so one barrier per step orders both the reads after the
// writes and the next step's writes after the reads.  Each wave's vote on stopping rides in the same
// buffer as its rows.  On return F and E hold the solution of rows 2t and 2t+1.
template <typename T, int NT>
__device__ __forceinline__ void pcr_pairs(const PcrSpace<T, NT>& w, int P, T fa, T fc, T fd, T ea, T ec, T ed,
                                          T& F, T& E) {
  constexpr int kR = PcrSpace<T, NT>::kRows;
  constexpr int kW = PcrSpace<T, NT>::kWaves;
  const int t = threadIdx.x;
  const bool own = t < P;
  const int mask = P - 1;
  if (own) {
    T* A = w.rows;
    A[t] = fa; A[kR + t] = fc; A[2 * kR + t] = fd;
    A[P + t] = ea; A[kR + P + t] = ec; A[2 * kR + P + t] = ed;
  }
  __syncthreads();
  int b = 0;
  bool done = false;
  for (int s = 1; s < 2 * P && !done; s <<= 1) {
    const T* A = w.rows + b * 3 * kR;
    const T* C = A + kR;
    const T* D = C + kR;
    bool live = false;
    if (own) {
      T nfa, nfc, nfd, nea, nec, ned;
      if (s == 1) {   // F row: partners E_{t-1} and E_t; E row: partners F_t and F_{t+1}
        const int m = P + ((t - 1) & mask), p = (t + 1) & mask;
        pcr_combine(fa, fc, fd, A[m], C[m], D[m], ea, ec, ed, nfa, nfc, nfd);
        pcr_combine(ea, ec, ed, fa, fc, fd, A[p], C[p], D[p], nea, nec, ned);
      } else {        // rows 2t -+ s and 2t+1 -+ s: the same kind of row, s/2 lanes away
        const int h = s >> 1;
        const int m = (t - h) & mask, p = (t + h) & mask;
        pcr_combine(fa, fc, fd, A[m], C[m], D[m], A[p], C[p], D[p], nfa, nfc, nfd);
        pcr_combine(ea, ec, ed, A[P + m], C[P + m], D[P + m], A[P + p], C[P + p], D[P + p], nea, nec, ned);
      }
      fa = nfa; fc = nfc; fd = nfd;
      ea = nea; ec = nec; ed = ned;
      live = (__builtin_fabs(fa) + __builtin_fabs(fc)) > kNegligible ||
             (__builtin_fabs(ea) + __builtin_fabs(ec)) > kNegligible;
      T* nA = w.rows + (1 - b) * 3 * kR;
      nA[t] = fa; nA[kR + t] = fc; nA[2 * kR + t] = fd;
      nA[P + t] = ea; nA[kR + P + t] = ec; nA[2 * kR + P + t] = ed;
    }
    const bool wave_live = __ballot(live) != 0;
    if ((t & 63) == 0) w.flags[(1 - b) * kW + (t >> 6)] = wave_live ? 1 : 0;
    __syncthreads();
    b = 1 - b;
    int any = 0;
#pragma unroll
    for (int k = 0; k < kW; ++k) any |= w.flags[b * kW + k];
    done = any == 0;
  }
  if (!done) {   // ran all log2(2P) steps: the remaining couplings point at the row itself
    fd = fd / ((T(1) + fa) + fc);
    ed = ed / ((T(1) + ea) + ec);
  }
  F = fd;
  E = ed;
}

// Reduced systems of the partition levels (rows (A, 1, C, D) in HBM), one workgroup each: chunk elimination
// to two rows per lane, PCR in LDS, recovery to X.  (They are few and large: their rows preloaded in
// registers matter more than a second workgroup per CU.)
template <int NT, int MC, bool EXACT>
__device__ __forceinline__ void reduced_solve(const PcrSpace<double, NT>& pcr, double* tstage, const SysDesc& sys,
                                              const double* __restrict__ LA, const double* __restrict__ LC,
                                              const double* __restrict__ LD, double* __restrict__ LX) {
  using T = double;                          // (tstage: one coefficient array at a time)
  const int R = sys.rows, P = sys.chunks;
  const int tid = threadIdx.x;
  const ArrayRows<T> asrc{LA + sys.in_off, LC + sys.in_off, LD + sys.in_off};
  const PtrDst<T> adst{LX + sys.in_off};
  if (R == 1) {   // a single Dirichlet unknown
    if (tid == 0) {
      T al, be, ga, de;
      asrc.row(0, 0, 1, al, be, ga, de);
      adst.write(0, 0, de / be);
    }
    return;
  }

  T al[MC], ga[MC], de[MC];
  int s = 0, m = 0;
  if (tid < P) {
    chunk_span(tid, R, P, s, m);
    if constexpr (EXACT) {
      s = tid * MC;
      m = MC;
    }
  }
  T AF = T(0), CF = T(0), DF = T(0), AE = T(0), CE = T(0), DE = T(0);
  if (R >= kCoalesceRows) {
    // One workgroup reads the whole reduced system: coalesced loads of the three arrays (every load in
    // flight at once), then each array transposed through LDS into the lanes' chunks.
    T va[MC], vc[MC], vd[MC];
#pragma unroll
    for (int j = 0; j < MC; ++j) {
      const int i = tid + j * NT;
      if (i < R) {
        va[j] = asrc.A[i];
        vc[j] = asrc.C[i];
        vd[j] = asrc.Dv[i];
      }
    }
    RegRows<T, MC> rr;
    stage_transpose<T, NT, MC>(tstage, va, R, P, s, m, rr.a);
    stage_transpose<T, NT, MC>(tstage, vc, R, P, s, m, rr.c);
    stage_transpose<T, NT, MC>(tstage, vd, R, P, s, m, rr.d);
    if (tid < P) chunk_eliminate<T, MC>(rr, s, m, R, al, ga, de, AF, CF, DF, AE, CE, DE);
  } else if (tid < P) {   // small systems: the lanes' own rows straight from HBM, all loads up front
    RegRows<T, MC> rr;
    rr.load(asrc.A, asrc.C, asrc.Dv, s, m);
    chunk_eliminate<T, MC>(rr, s, m, R, al, ga, de, AF, CF, DF, AE, CE, DE);
  }
  T F = T(0), E = T(0);
  // (PCR's last barrier follows its last read of the rows, so the staging buffer is free on return)
  pcr_pairs<T, NT>(pcr, P, AF, CF, DF, AE, CE, DE, F, E);
  if (R >= kCoalesceRows) {   // through LDS again, for a coalesced store
    if (tid < P) chunk_recover<T, MC>(LdsDst<T>{tstage, 0}, s, m, al, ga, de, F, E);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < MC; ++j) {
      const int i = tid + j * NT;
      if (i < R) adst.x[i] = tstage[padded(i)];
    }
  } else {
    if (tid < P) chunk_recover<T, MC>(adst, s, m, al, ga, de, F, E);
  }
}

// One system per workgroup.  `only` (optional): the systems of instances whose entry is 1; only[-1] is zero when there
// is none.
template <int NT, int MC, bool EXACT = false>
__global__ __launch_bounds__(NT, MC == 16 ? 2 : 1) void btcs_reduced_kernel(
    const SysDesc* __restrict__ systems, const double* __restrict__ LA, const double* __restrict__ LC,
    const double* __restrict__ LD, double* __restrict__ LX, const int* __restrict__ only) {
  using T = double;
  using Pcr = PcrSpace<T, NT>;
  constexpr int kStageBytes = padded_size(NT * MC) * static_cast<int>(sizeof(T));
  constexpr int kBytes = kStageBytes > Pcr::kBytes ? kStageBytes : Pcr::kBytes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kBytes];
  __shared__ int pcr_flags[2 * Pcr::kWaves];
  const Pcr pcr{reinterpret_cast<T*>(smem), pcr_flags};
  if (only && only[-1] == 0) return;
  const SysDesc sys = systems[blockIdx.x];
  if (only && only[sys.inst] != 1) return;
  reduced_solve<NT, MC, EXACT>(pcr, reinterpret_cast<T*>(smem), sys, LA, LC, LD, LX);
}

// Per-step whole-system solver for systems of exactly NT x MC rows whose first row is 16-byte aligned,
// persistent and pipelined through LDS.  Each workgroup walks a strided share of the systems with two
// staging buffers: while it solves system k (its rows in registers), the rows of system k + 1 stream from
// HBM straight into the other buffer (global_load_lds, which holds no registers) and the stores of
// system k - 1 drain, so the only wait for memory comes after the solve, at the top of the next system.
// Loads and stores of a system go out as 16-byte chunks, every wave instruction covering 1 KB of
// consecutive chunks.  In LDS the chunks are swizzled: chunk q = H t + h (lane t's h-th chunk of its
// H = MC * sizeof(S) / 16) sits at H t + (h ^ f(t)), f(t) = (t / (16 / H)) mod H, so that 16 lanes
// reading either their own chunks (one h each) or 16 consecutive chunks touch 16 different 16-byte bank
// groups.  The interface solve's LDS overlays the buffer of the system being solved (its rows are in
// registers by then).  Same operations in the same order as btcs_whole_kernel<S, NT, MC>:
// bitwise the same results.
template <typename S>
struct Chunk16;
template <>
struct Chunk16<double> {
  typedef double type __attribute__((ext_vector_type(2)));
};
template <>
struct Chunk16<float> {
  typedef float type __attribute__((ext_vector_type(4)));
};

template <typename S, int NT, int MC>
struct StreamLayout {
  using V = typename Chunk16<S>::type;
  static constexpr int kPer = 16 / static_cast<int>(sizeof(S));               // elements per chunk
  static constexpr int kLane = MC / kPer;                                     // H: chunks of a lane's rows
  static constexpr int kWaves = NT / 64;
  static constexpr int kShift = kLane == 8 ? 1 : kLane == 4 ? 2 : 3;          // log2(16 / H)
  static_assert(kLane == 2 || kLane == 4 || kLane == 8, "a lane's rows must be 2, 4 or 8 chunks");
  static constexpr int kBuf = (NT * MC * static_cast<int>(sizeof(S)) > InterfaceSpace<double, NT>::kBytes
                                   ? NT * MC * static_cast<int>(sizeof(S))
                                   : InterfaceSpace<double, NT>::kBytes);
  // LDS position of chunk q (an involution: the XOR leaves q / H unchanged)
  __device__ static __forceinline__ int swz(int q) { return q ^ (((q / kLane) >> kShift) & (kLane - 1)); }
  // Issue the loads of a system's rows (src: its first row) into the buffer buf: instruction k of wave w
  // fills the LDS chunks 64 (k kWaves + w) + lane, each lane fetching the chunk that belongs there.
  __device__ static __forceinline__ void load_async(unsigned char* buf, const S* src) {
    const int lane = static_cast<int>(threadIdx.x) & 63, wave = static_cast<int>(threadIdx.x) >> 6;
    const unsigned char* s = reinterpret_cast<const unsigned char*>(src);
#pragma unroll
    for (int k = 0; k < kLane; ++k) {
      const int p0 = (k * kWaves + wave) * 64;
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(s + 16 * swz(p0 + lane)),
          (__attribute__((address_space(3))) void*)(buf + 16 * p0), 16, 0, 0);
    }
  }
  // Coalesced stores of a system's new rows from buf (dst: its first row).
  __device__ static __forceinline__ void store(const unsigned char* buf, S* dst) {
    const int lane = static_cast<int>(threadIdx.x) & 63, wave = static_cast<int>(threadIdx.x) >> 6;
    const V* b = reinterpret_cast<const V*>(buf);
    V* d = reinterpret_cast<V*>(dst);
#pragma unroll
    for (int k = 0; k < kLane; ++k) {
      const int q = (k * kWaves + wave) * 64 + lane;
      d[q] = b[swz(q)];
    }
  }
};

// vmcnt(0) with the other counters left alone: every vector memory access of this wave is complete,
// including the LDS writes of global_load_lds (which the compiler does not track).
__device__ __forceinline__ void wait_vector_memory() { __builtin_amdgcn_s_waitcnt(0x0F70); }

template <typename S, int NT, int MC>
__global__ __launch_bounds__(NT, 2) void btcs_stream_kernel(const InstDesc* __restrict__ inst,
                                                            const SysDesc* __restrict__ systems, int n_sys,
                                                            const S* __restrict__ u, S* __restrict__ out) {
  using T = double;
  using L = StreamLayout<S, NT, MC>;
  using V = typename L::V;
  constexpr int W = NT * MC, H = L::kLane, E = L::kPer;
  using IS = InterfaceSpace<T, NT>;
  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * L::kBuf];
  __shared__ uint64_t iface_votes[2 * IS::kVoteWords];
  const int tid = threadIdx.x;
  int b = blockIdx.x;
  if (b >= n_sys) return;
  if (tid < 2 * IS::kVoteWords) iface_votes[tid] = 0;
  SysDesc sys = systems[b];
  InstDesc d = inst[sys.inst];
  L::load_async(smem, u + d.off + (d.bc == kDirichlet ? 1 : 0));
  // lane tid's chunks in LDS: H tid + (h ^ f(tid))
  const int own = H * tid, fx = (tid >> L::kShift) & (H - 1);
  int cur = 0;
  S* prev_dst = nullptr;                       // rows of the previous system, still to be stored
  for (;;) {
    wait_vector_memory();
    __syncthreads();                           // this system's rows have landed; last system's results written
    unsigned char* bc = smem + cur * L::kBuf;
    unsigned char* bn = smem + (cur ^ 1) * L::kBuf;
    if (prev_dst) L::store(bn, prev_dst);
    const bool dir = d.bc == kDirichlet;
    T al[MC], ga[MC], de[MC];
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const V v = reinterpret_cast<const V*>(bc)[own + (h ^ fx)];
#pragma unroll
      for (int e = 0; e < E; ++e) de[h * E + e] = static_cast<T>(v[e]);
    }
    __syncthreads();                           // every read of both buffers done: bn takes the next rows
    const int nb = b + static_cast<int>(gridDim.x);
    SysDesc nsys{};
    InstDesc nd{};
    if (nb < n_sys) {
      nsys = systems[nb];
      nd = inst[nsys.inst];
      L::load_async(bn, u + nd.off + (nd.bc == kDirichlet ? 1 : 0));
    }
    if (dir && tid == 0) {
      out[d.off] = static_cast<S>(d.a);
      out[d.off + d.n - 1] = static_cast<S>(d.b);
    }
    const IS iws{reinterpret_cast<T*>(bc), reinterpret_cast<T*>(bc) + 3 * NT, iface_votes};
    T y, yp;
    slot_step<NT, MC, true, true>(iws, SlotRows{d.r, d.D, d.a, d.b}, slot_lane<MC, true>(tid, W, NT, dir), NT, al, ga,
                                  de, y, yp);
    wg_barrier<true>();                        // the interface unknowns read before bc takes the results
#pragma unroll
    for (int h = 0; h < H; ++h) {
      V v;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int j = h * E + e;
        v[e] = static_cast<S>(j < MC - 1 ? __builtin_fma(-ga[j], y, __builtin_fma(-al[j], yp, de[j])) : y);
      }
      reinterpret_cast<V*>(bc)[own + (h ^ fx)] = v;
    }
    S* dst = out + d.off + (dir ? 1 : 0);
    if (nb >= n_sys) {
      __syncthreads();
      L::store(bc, dst);
      break;
    }
    prev_dst = dst;
    b = nb;
    sys = nsys;
    d = nd;
    cur ^= 1;
  }
}

// Rows of a Newton iteration (fully implicit central-convection step, eqs. 10-14) for the whole system of
// one instance: the Jacobian row of eq. 11 at the iterate x (staged in LDS, unknown k at padded(k)) and
// the right-hand side -F, with the old state u read from HBM.  The increment of a Dirichlet neighbour is
// zero, so the end rows simply drop that coupling.  A row that is not strictly diagonally dominant is
// noted in `bad` (kept per lane, branch-free, and reported once after the elimination).
template <typename S>
struct NewtonRows {
  const double* st;
  const S* __restrict__ u;
  double half_r, D, a, b;
  bool periodic;
  int* flags;
  mutable bool bad = false;
  __device__ __forceinline__ void row(int, int k, int R, double& al, double& be, double& ga, double& de) const {
    const double xm = k > 0 ? st[padded(k - 1)] : (periodic ? st[padded(R - 1)] : a);
    const double xp = k < R - 1 ? st[padded(k + 1)] : (periodic ? st[padded(0)] : b);
    const double xi = st[padded(k)];
    const double F = (xi - static_cast<double>(u[k])) + (half_r * xi * (xp - xm) - D * ((xp + xm) - 2.0 * xi));
    al = -(half_r * xi) - D;
    be = (1.0 + 2.0 * D) + half_r * (xp - xm);
    ga = half_r * xi - D;
    de = -F;
    if (!periodic) {
      if (k == 0) al = 0.0;
      if (k == R - 1) ga = 0.0;
    }
    bad = bad || newton_row_not_dominant(al, be, ga);
  }
  __device__ __forceinline__ void boundary(int, int, int, double&, double&, double&, double&) const {}
};

// Eliminate the Jacobian's chunks, PCR, recover the increment into the staging buffer and add it to the
// iterate in HBM (FULL: every lane holds MC rows).  On the last iteration the increments are checked
// against the iterate.
template <bool FULL, typename S, int NT, int MC>
__device__ __forceinline__ void newton_solve(const PcrSpace<double, NT>& pcr, double* stage, const NewtonRows<S>& rows,
                                             S* __restrict__ xs, int R, int P, bool last) {
  using T = double;
  const int tid = threadIdx.x;
  T al[MC], ga[MC], de[MC];
  T AF = T(0), CF = T(0), DF = T(0), AE = T(0), CE = T(0), DE = T(0);
  int s = 0, m = 0;
  if (tid < P) {
    chunk_span(tid, R, P, s, m);
    if constexpr (FULL) {
      s = tid * MC;
      m = MC;
    }
    chunk_eliminate<T, MC>(rows, s, m, R, al, ga, de, AF, CF, DF, AE, CE, DE);
    if (rows.bad) rows.flags[0] = 1;
  }
  __syncthreads();                             // the PCR rows overlay the staged iterate
  T F = T(0), E = T(0);
  pcr_pairs<T, NT>(pcr, P, AF, CF, DF, AE, CE, DE, F, E);   // ends its use of the rows with a barrier
  if (tid < P) chunk_recover<T, MC>(PtrDst<T>{stage}, s, m, al, ga, de, F, E);   // increments, unpadded
  __syncthreads();
#pragma unroll
  for (int j = 0; j < MC; ++j) {
    const int i = tid + j * NT;
    T delta = T(0), xn = T(0), uo = T(0);
    if (i < R) {
      delta = stage[i];
      const S v = static_cast<S>(static_cast<T>(xs[i]) + delta);
      xs[i] = v;
      xn = static_cast<T>(v);
      if (last) uo = static_cast<T>(rows.u[i]);
    }
    if (last) newton_check_increment(i < R, delta, xn, uo, newton_increment_tol<S>(), rows.flags);
  }
}

// One Newton iteration for systems of up to NT x MC rows, one workgroup per system: stage the iterate,
// eliminate the Jacobian's chunks, PCR, recover the increment into the staging buffer and add it to the
// iterate in HBM (x is the output state buffer, updated in place).
template <typename S, int NT, int MC>
__global__ __launch_bounds__(NT, MC == 16 ? 4 : 1) void newton_wg_kernel(const InstDesc* __restrict__ inst,
                                                                         const SysDesc* __restrict__ systems,
                                                                         const S* __restrict__ u, S* __restrict__ x,
                                                                         int last, int* __restrict__ flags) {
  using T = double;
  using Pcr = PcrSpace<T, NT>;
  constexpr int kStageBytes = padded_size(NT * MC) * static_cast<int>(sizeof(T));
  constexpr int kBytes = kStageBytes > Pcr::kBytes ? kStageBytes : Pcr::kBytes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kBytes];
  __shared__ int pcr_flags[2 * Pcr::kWaves];
  const Pcr pcr{reinterpret_cast<T*>(smem), pcr_flags};
  T* stage = reinterpret_cast<T*>(smem);
  const SysDesc sys = systems[blockIdx.x];
  const InstDesc d = inst[sys.inst];
  const bool dir = d.bc == kDirichlet;
  const int R = sys.rows, P = sys.chunks;
  const int tid = threadIdx.x;
  const int64_t o = d.off + (dir ? 1 : 0);
  S* __restrict__ xs = x + o;
#pragma unroll
  for (int j = 0; j < MC; ++j) {
    const int i = tid + j * NT;
    if (i < R) stage[padded(i)] = static_cast<T>(xs[i]);
  }
  __syncthreads();
  const NewtonRows<S> rows{stage, u + o, d.r / 2.0, d.D, d.a, d.b, !dir, flags};
  if (R == 1) {   // a single Dirichlet unknown
    if (tid == 0) {
      T al, be, ga, de;
      rows.row(0, 0, 1, al, be, ga, de);
      if (rows.bad) flags[0] = 1;
      const T delta = de / be;
      const S v = static_cast<S>(stage[0] + delta);
      xs[0] = v;
      if (last && !(__builtin_fabs(delta) <= newton_increment_tol<S>() *
                    __builtin_fmax(__builtin_fabs(static_cast<T>(v)), __builtin_fabs(static_cast<T>(rows.u[0])))))
        flags[1] = 1;
    }
    return;
  }
  // every lane's chunk full (NT x MC rows): the chunk size as a constant, so no row is selected at a
  // run-time index
  if (R == NT * MC && P == NT) newton_solve<true, S, NT, MC>(pcr, stage, rows, xs, R, P, last != 0);
  else newton_solve<false, S, NT, MC>(pcr, stage, rows, xs, R, P, last != 0);
}

constexpr int kSpikeWaves = kReduceBlock / 64;

// One row of a block's interface system in spike form: unit diagonal, couplings a (row i - s) and c
// (row i + s), right-hand side d, and the spike columns p (on the previous block's last unknown L) and q
// (on the next block's first unknown Rt).
struct SpikeRow {
  double a, c, d, p, q;
};

// One PCR step of row r with its partners m (distance -s) and p (distance +s), as pcr_combine, also
// carried through the two spike columns.
__device__ __forceinline__ SpikeRow spike_combine(const SpikeRow& r, const SpikeRow& m, const SpikeRow& p) {
  const double inv = recip(__builtin_fma(-r.c, p.a, __builtin_fma(-r.a, m.c, 1.0)));
  const double a = r.a * inv, c = r.c * inv;
  SpikeRow n;
  n.a = -(a * m.a);
  n.c = -(c * p.c);
  n.d = __builtin_fma(-c, p.d, __builtin_fma(-a, m.d, r.d * inv));
  n.p = __builtin_fma(-c, p.p, __builtin_fma(-a, m.p, r.p * inv));
  n.q = __builtin_fma(-c, p.q, __builtin_fma(-a, m.q, r.q * inv));
  return n;
}

// The block's two rows in the partition form (tridiagonal over the first and last unknowns of all
// blocks), from the spike form of its first and last unknowns,
//   x_0 + P_0 L + Q_0 Rt = D_0,   x_e + P_e L + Q_e Rt = D_e:
//   F row:  (P_0 - k P_e) L + x_0 - k x_e = D_0 - k D_e,        k = Q_0 / Q_e
//   E row:  -h x_0 + x_e + (Q_e - h Q_0) Rt = D_e - h D_0,     h = P_e / P_0
// A block with no left (right) neighbour coupling has P = 0 (Q = 0) throughout; then h = 0 (k = 0).
__device__ __forceinline__ void partition_rows(double P0, double Q0, double D0, double Pe, double Qe, double De,
                                               double& AF, double& CF, double& DF, double& AE, double& CE,
                                               double& DE) {
  const double k = Qe != 0.0 ? Q0 / Qe : 0.0;
  const double h = P0 != 0.0 ? Pe / P0 : 0.0;
  AF = __builtin_fma(-k, Pe, P0);
  CF = -k;
  DF = __builtin_fma(-k, De, D0);
  AE = -h;
  CE = __builtin_fma(-h, Q0, Qe);
  DE = __builtin_fma(-h, D0, De);
}

// ---- Interface partition inside a block of a long system ------------------------------------------
// Within a block, chunk t's interior rows lie between the interface unknowns y_{t-1} and y_t as in the
// whole-system solver.  The block's first chunk has L (the previous block's last unknown, row rs - 1)
// on its left, and its last chunk's interface row couples to Rt (the next block's first unknown, row
// re).  Both stay symbolic as spike columns, so PCR over the block's Pb interface rows (one per lane,
// rows outside the block taken as zero) leaves  y_t + P_t L + Q_t Rt = D_t.  The block's first unknown
// is its first chunk's first interior row, x = de_0 - al_0 L - ga_0 y_0, and its last is y_{Pb-1}.

// LDS of a block's interface solve (it overlays the staged rows once every chunk has been read): the
// exchanged first interior rows, two buffers of the interface rows' five columns, and the waves' votes.
struct BlockIfaceSpace {
  static constexpr int kN = kReduceBlock;
  static constexpr int kBytes = (3 + 2 * 5) * kN * 8;
  double* xchg;   // 3 x kN
  double* rows;   // 2 buffers x 5 columns x kN
  int* flags;     // 2 x kSpikeWaves
  __device__ __forceinline__ SpikeRow load(int b, int i) const {
    const double* r = rows + b * 5 * kN;
    return SpikeRow{r[i], r[kN + i], r[2 * kN + i], r[3 * kN + i], r[4 * kN + i]};
  }
  __device__ __forceinline__ void store(int b, int i, const SpikeRow& v) const {
    double* r = rows + b * 5 * kN;
    r[i] = v.a; r[kN + i] = v.c; r[2 * kN + i] = v.d; r[3 * kN + i] = v.p; r[4 * kN + i] = v.q;
  }
};

// Lane t < Pb passes its chunk's first interior row (al0, ga0, de0), its last interior row (alL, gaL,
// deL) and its interface row (ia, ib, ic, id).  On return r is the lane's final spike row and the
// result is the buffer that holds every lane's final row.  Starts by writing the LDS (the caller
// synchronises after its last read of what the space overlays) and ends with a barrier.
__device__ __forceinline__ int block_iface_solve(const BlockIfaceSpace& w, int Pb, double al0, double ga0,
                                                 double de0, double alL, double gaL, double deL, double ia,
                                                 double ib, double ic, double id, SpikeRow& r) {
  constexpr int kN = BlockIfaceSpace::kN;
  const int t = threadIdx.x;
  const bool own = t < Pb;
  const SpikeRow zero{0.0, 0.0, 0.0, 0.0, 0.0};
  if (own) {
    w.xchg[t] = al0;
    w.xchg[kN + t] = ga0;
    w.xchg[2 * kN + t] = de0;
  }
  __syncthreads();
  r = zero;
  if (own) {
    const bool next = t + 1 < Pb;
    const double nal = next ? w.xchg[t + 1] : 0.0;
    const double nga = next ? w.xchg[kN + t + 1] : 0.0;
    const double nde = next ? w.xchg[2 * kN + t + 1] : 0.0;
    const double inv = recip(__builtin_fma(-ic, nal, __builtin_fma(-ia, gaL, ib)));
    const double lower = -(ia * alL) * inv;   // on y_{t-1}, which is L for the block's first chunk
    r.a = t > 0 ? lower : 0.0;
    r.p = t > 0 ? 0.0 : lower;
    r.c = next ? -(ic * nga) * inv : 0.0;     // on y_{t+1}, or directly on Rt for the last chunk
    r.q = next ? 0.0 : ic * inv;
    r.d = __builtin_fma(-ic, nde, __builtin_fma(-ia, deL, id)) * inv;
    w.store(0, t, r);
  }
  __syncthreads();
  int b = 0;
  bool done = false;
  for (int s = 1; s < Pb && !done; s <<= 1) {
    bool live = false;
    if (own) {
      r = spike_combine(r, t >= s ? w.load(b, t - s) : zero, t + s < Pb ? w.load(b, t + s) : zero);
      live = (__builtin_fabs(r.a) + __builtin_fabs(r.c)) > kNegligible;
      w.store(1 - b, t, r);
    }
    const bool wave_live = __ballot(live) != 0;
    if ((t & 63) == 0) w.flags[(1 - b) * kSpikeWaves + (t >> 6)] = wave_live ? 1 : 0;
    __syncthreads();
    b = 1 - b;
    int any = 0;
#pragma unroll
    for (int k = 0; k < kSpikeWaves; ++k) any |= w.flags[b * kSpikeWaves + k];
    done = any == 0;
  }
  return b;
}

// A block's chunks eliminated (rows staged in LDS) and its interface system solved; returns the buffer
// of the final rows.  al/ga/de keep the chunk's interior rows for the recovery.
template <bool FULL, typename S>
__device__ __forceinline__ int block_iface_step(const BlockIfaceSpace& w, const S* stage, const InstDesc& d,
                                                const SysDesc& sys, const ChunkBlock& cb, int rs, int Pb, int& s,
                                                int& m, double (&al)[kRedChunk], double (&ga)[kRedChunk],
                                                double (&de)[kRedChunk], SpikeRow& r) {
  using T = double;
  const bool dir = d.bc == kDirichlet;
  const int tid = threadIdx.x;
  T ia = T(0), ib = T(1), ic = T(0), id = T(0), alL = T(0), gaL = T(0), deL = T(0);
  s = 0;
  m = 0;
  if (tid < Pb) {
    chunk_span(cb.chunk0 + tid, sys.rows, sys.chunks, s, m);
    if constexpr (FULL) m = kRedChunk;         // the value chunk_span gives, as a constant
    interface_eliminate<T, kRedChunk>(LdsRows<S>{stage, rs, d.r, d.D, DirichletEnds{d.a, d.b, dir}}, s, m,
                                             sys.rows, al, ga, de, ia, ib, ic, id);
#pragma unroll
    for (int j = 0; j < kRedChunk; ++j) {
      if (j == m - 2) {
        alL = al[j];
        gaL = ga[j];
        deL = de[j];
      }
    }
  }
  __syncthreads();                             // every chunk read before the interface LDS overlays the stage
  return block_iface_solve(w, Pb, tid < Pb ? al[0] : T(0), tid < Pb ? ga[0] : T(0), tid < Pb ? de[0] : T(0), alL,
                           gaL, deL, ia, ib, ic, id, r);
}

// Rows [rs, re) of the chunks a partition workgroup owns: chunk k spans chunk_span(k).
__device__ __forceinline__ void block_rows(const SysDesc& sys, int c0, int& rs, int& re) {
  int m;
  chunk_span(c0, sys.rows, sys.chunks, rs, m);
  const int c1 = c0 + kReduceBlock;
  if (c1 >= sys.chunks) {
    re = sys.rows;
  } else {
    chunk_span(c1, sys.rows, sys.chunks, re, m);
  }
}

// Every chunk of the block holds kRedChunk rows (all blocks but those holding a system's shorter last
// chunks): the block kernels then take a body in which the row counts are compile-time constants, so
// that no row index is selected at run time.
__device__ __forceinline__ bool block_full(const SysDesc& sys, int c0, int Pb) {
  const int q = sys.rows / sys.chunks, rho = sys.rows - q * sys.chunks;
  return Pb == kReduceBlock && (q == kRedChunk || (q == kRedChunk - 1 && c0 + Pb <= rho));
}

// One chunk of a partition level held in arrays (FULL: every chunk of the workgroup has kRedChunk rows,
// so the row count is a constant): eliminate it and store its two reduced rows ...
template <bool FULL>
__device__ __forceinline__ void array_reduce_chunk(const SysDesc& sys, int k, double* __restrict__ LA,
                                                   double* __restrict__ LC, double* __restrict__ LD) {
  using T = double;
  T al[kRedChunk], ga[kRedChunk], de[kRedChunk];
  T AF, CF, DF, AE, CE, DE;
  int s, m;
  chunk_span(k, sys.rows, sys.chunks, s, m);
  if constexpr (FULL) m = kRedChunk;
  RegRows<T, kRedChunk> rows;
  rows.load(LA + sys.in_off, LC + sys.in_off, LD + sys.in_off, s, m);
  chunk_eliminate<T, kRedChunk>(rows, s, m, sys.rows, al, ga, de, AF, CF, DF, AE, CE, DE);
  const int64_t o = sys.red_off + 2 * static_cast<int64_t>(k);
  LA[o] = AF; LC[o] = CF; LD[o] = DF;
  LA[o + 1] = AE; LC[o + 1] = CE; LD[o + 1] = DE;
}

// ... and, once the reduced unknowns are solved, eliminate it again and recover its rows.
template <bool FULL>
__device__ __forceinline__ void array_backsub_chunk(const SysDesc& sys, int k, const double* __restrict__ LA,
                                                    const double* __restrict__ LC, const double* __restrict__ LD,
                                                    double* __restrict__ LX) {
  using T = double;
  T al[kRedChunk], ga[kRedChunk], de[kRedChunk];
  T AF, CF, DF, AE, CE, DE;
  int s, m;
  chunk_span(k, sys.rows, sys.chunks, s, m);
  if constexpr (FULL) m = kRedChunk;
  const int64_t o = sys.red_off + 2 * static_cast<int64_t>(k);
  const T F = LX[o];
  const T E = LX[o + 1];
  RegRows<T, kRedChunk> rows;
  rows.load(LA + sys.in_off, LC + sys.in_off, LD + sys.in_off, s, m);
  chunk_eliminate<T, kRedChunk>(rows, s, m, sys.rows, al, ga, de, AF, CF, DF, AE, CE, DE);
  chunk_recover<T, kRedChunk>(PtrDst<T>{LX + sys.in_off}, s, m, al, ga, de, F, E);
}

// Partition level of a reduced system held in (A, C, D) arrays, forward half: every thread eliminates
// one chunk and stores its two reduced rows.
__global__ __launch_bounds__(kReduceBlock, 2) void btcs_array_reduce_kernel(
    const SysDesc* __restrict__ systems, const ChunkBlock* __restrict__ blocks, double* __restrict__ LA,
    double* __restrict__ LC, double* __restrict__ LD, const int* __restrict__ only) {
  if (only && only[-1] == 0) return;
  const ChunkBlock cb = blocks[blockIdx.x];
  const SysDesc sys = systems[cb.sys];
  if (only && only[sys.inst] != 1) return;
  const int k = cb.chunk0 + static_cast<int>(threadIdx.x);
  if (k >= sys.chunks) return;
  if (block_full(sys, cb.chunk0, min(kReduceBlock, sys.chunks - cb.chunk0))) array_reduce_chunk<true>(sys, k, LA, LC, LD);
  else array_reduce_chunk<false>(sys, k, LA, LC, LD);
}

// Backward half: re-eliminate the chunk and recover its rows from the solved reduced unknowns.
__global__ __launch_bounds__(kReduceBlock, 2) void btcs_array_backsub_kernel(
    const SysDesc* __restrict__ systems, const ChunkBlock* __restrict__ blocks, const double* __restrict__ LA,
    const double* __restrict__ LC, const double* __restrict__ LD, double* __restrict__ LX,
    const int* __restrict__ only) {
  if (only && only[-1] == 0) return;
  const ChunkBlock cb = blocks[blockIdx.x];
  const SysDesc sys = systems[cb.sys];
  if (only && only[sys.inst] != 1) return;
  const int k = cb.chunk0 + static_cast<int>(threadIdx.x);
  if (k >= sys.chunks) return;
  if (block_full(sys, cb.chunk0, min(kReduceBlock, sys.chunks - cb.chunk0))) array_backsub_chunk<true>(sys, k, LA, LC, LD, LX);
  else array_backsub_chunk<false>(sys, k, LA, LC, LD, LX);
}

// Forward half of a block-partition step after the block is staged (FULL: every chunk has kRedChunk rows).
template <bool FULL, typename S>
__device__ __forceinline__ void block_reduce_body(const BlockIfaceSpace& w, const S* stage, const InstDesc& d,
                                                  const SysDesc& sys, const ChunkBlock& cb, int rs, int Pb,
                                                  double* __restrict__ LA, double* __restrict__ LC,
                                                  double* __restrict__ LD) {
  using T = double;
  const int tid = threadIdx.x;
  int s, m;
  T al[kRedChunk], ga[kRedChunk], de[kRedChunk];
  SpikeRow r;
  const int b = block_iface_step<FULL>(w, stage, d, sys, cb, rs, Pb, s, m, al, ga, de, r);
  if (tid == 0) {
    // first unknown: x = de_0 - al_0 L - ga_0 y_0 with y_0 = D_0 - P_0 L - Q_0 Rt; last: y_{Pb-1}
    const SpikeRow e = w.load(b, Pb - 1);
    T AF, CF, DF, AE, CE, DE;
    partition_rows(__builtin_fma(-ga[0], r.p, al[0]), -(ga[0] * r.q), __builtin_fma(-ga[0], r.d, de[0]), e.p, e.q,
                   e.d, AF, CF, DF, AE, CE, DE);
    const int64_t o = sys.red_off + 2 * static_cast<int64_t>(cb.chunk0 / kReduceBlock);
    LA[o] = AF; LC[o] = CF; LD[o] = DF;
    LA[o + 1] = AE; LC[o + 1] = CE; LD[o + 1] = DE;
  }
}

// Block partition, forward half (level 0 of a long system): a workgroup stages its 256 chunks' rows
// (<= 4096) through LDS, eliminates every chunk, solves the block's interface system in spike form and
// stores the block's two partition rows at red_off + 2 * (block index within the system).
template <typename S>
__global__ __launch_bounds__(kReduceBlock, 4) void btcs_block_reduce_kernel(
    const InstDesc* __restrict__ inst, const SysDesc* __restrict__ systems,
    const ChunkBlock* __restrict__ blocks, const S* __restrict__ u, double* __restrict__ LA,
    double* __restrict__ LC, double* __restrict__ LD, const int* __restrict__ only) {
  using T = double;
  constexpr int kStageBytes = padded_size(kRedRows) * static_cast<int>(sizeof(S));
  constexpr int kBytes = kStageBytes > BlockIfaceSpace::kBytes ? kStageBytes : BlockIfaceSpace::kBytes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kBytes];
  __shared__ int iface_flags[2 * kSpikeWaves];
  S* stage = reinterpret_cast<S*>(smem);
  T* lds = reinterpret_cast<T*>(smem);
  const BlockIfaceSpace w{lds, lds + 3 * BlockIfaceSpace::kN, iface_flags};
  if (only && only[-1] == 0) return;         // no instance is left to the partition levels
  const ChunkBlock cb = blocks[blockIdx.x];
  const SysDesc sys = systems[cb.sys];
  if (only && only[sys.inst] != 1) return;   // this instance's windows held
  const InstDesc d = inst[sys.inst];
  const bool dir = d.bc == kDirichlet;
  const int Pb = min(kReduceBlock, sys.chunks - cb.chunk0);
  int rs, re;
  block_rows(sys, cb.chunk0, rs, re);
  stage_in(stage, u + d.off + (dir ? 1 : 0) + rs, re - rs);
  __syncthreads();
  if (block_full(sys, cb.chunk0, Pb)) block_reduce_body<true>(w, stage, d, sys, cb, rs, Pb, LA, LC, LD);
  else block_reduce_body<false>(w, stage, d, sys, cb, rs, Pb, LA, LC, LD);
}


// Backward half of a block-partition step after the block is staged (FULL: every chunk has kRedChunk rows; TOP: returns
// the lane's share of the new rows' largest magnitude).
template <bool FULL, bool TOP, typename S>
__device__ __forceinline__ double block_backsub_body(const BlockIfaceSpace& w, S* stage, const InstDesc& d,
                                                   const SysDesc& sys, const ChunkBlock& cb, int rs, int re,
                                                   int Pb, const S* __restrict__ u, S* __restrict__ out,
                                                   const double* __restrict__ LX) {
  using T = double;
  const bool dir = d.bc == kDirichlet;
  const int tid = threadIdx.x;
  const int blk = cb.chunk0 / kReduceBlock;
  const int nblk = (sys.chunks + kReduceBlock - 1) / kReduceBlock;
  int s, m;
  T al[kRedChunk], ga[kRedChunk], de[kRedChunk];
  SpikeRow r;
  const int b = block_iface_step<FULL>(w, stage, d, sys, cb, rs, Pb, s, m, al, ga, de, r);
  // neighbours' end unknowns; a Dirichlet system's outer blocks have P = 0 or Q = 0 and ignore them
  const T* X = LX + sys.red_off;
  const bool periodic = !dir;
  const T L = blk > 0 ? X[2 * blk - 1] : (periodic ? X[2 * nblk - 1] : T(0));
  const T Rt = blk + 1 < nblk ? X[2 * blk + 2] : (periodic ? X[0] : T(0));
  T y = T(0), yp = T(0);
  if (tid < Pb) {
    y = __builtin_fma(-r.q, Rt, __builtin_fma(-r.p, L, r.d));
    if (tid > 0) {
      const SpikeRow q = w.load(b, tid - 1);
      yp = __builtin_fma(-q.q, Rt, __builtin_fma(-q.p, L, q.d));
    } else {
      yp = L;
    }
  }
  __syncthreads();                             // the interface rows read before the stage is rewritten
  Magnitude<S> top;
  if (tid < Pb) {
    const LdsDst<S> dst{stage, rs};
#pragma unroll
    for (int j = 0; j < kRedChunk; ++j) {
      const double v = j == m - 1 ? y : __builtin_fma(-ga[j], y, __builtin_fma(-al[j], yp, de[j]));
      if (j < m) {
        dst.write(j, s + j, v);
        if constexpr (TOP) top.take(static_cast<S>(v));
      }
    }
  }
  __syncthreads();
  const int64_t o = d.off + (dir ? 1 : 0) + rs;
  if (sys.cn) stage_out_cn(stage, u + o, out + o, re - rs);
  else stage_out(stage, out + o, re - rs);
  if (dir && tid == 0) {
    if (cb.chunk0 == 0) out[d.off] = static_cast<S>(d.a);
    if (cb.chunk0 + kReduceBlock >= sys.chunks) out[d.off + d.n - 1] = static_cast<S>(d.b);
  }
  return top.value();
}

// Block partition, backward half: the block repeats the forward reduction (keeping its chunks'
// elimination in registers), takes its neighbours' solved end unknowns L (the previous block's last)
// and Rt (the next block's first; both cyclically for periodic systems), evaluates every interface
// unknown y_t = D_t - P_t L - Q_t Rt, recovers every chunk and stores the new state coalesced (with
// the Dirichlet nodes).
template <typename S>
__global__ __launch_bounds__(kReduceBlock, 3) void btcs_block_backsub_kernel(
    const InstDesc* __restrict__ inst, const SysDesc* __restrict__ systems,
    const ChunkBlock* __restrict__ blocks, const S* __restrict__ u, S* __restrict__ out,
    const double* __restrict__ LX, const int* __restrict__ only) {
  using T = double;
  constexpr int kStageBytes = padded_size(kRedRows) * static_cast<int>(sizeof(S));
  constexpr int kBytes = kStageBytes > BlockIfaceSpace::kBytes ? kStageBytes : BlockIfaceSpace::kBytes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kBytes];
  __shared__ int iface_flags[2 * kSpikeWaves];
  S* stage = reinterpret_cast<S*>(smem);
  T* lds = reinterpret_cast<T*>(smem);
  const BlockIfaceSpace w{lds, lds + 3 * BlockIfaceSpace::kN, iface_flags};
  if (only && only[-1] == 0) return;         // no instance is left to the partition levels
  const ChunkBlock cb = blocks[blockIdx.x];
  const SysDesc sys = systems[cb.sys];
  if (only && only[sys.inst] != 1) return;   // this instance's windows held
  const InstDesc d = inst[sys.inst];
  const bool dir = d.bc == kDirichlet;
  const int Pb = min(kReduceBlock, sys.chunks - cb.chunk0);
  int rs, re;
  block_rows(sys, cb.chunk0, rs, re);
  stage_in(stage, u + d.off + (dir ? 1 : 0) + rs, re - rs);
  __syncthreads();
  if (block_full(sys, cb.chunk0, Pb)) block_backsub_body<true, false>(w, stage, d, sys, cb, rs, re, Pb, u, out, LX);
  else block_backsub_body<false, false>(w, stage, d, sys, cb, rs, re, Pb, u, out, LX);
}

// Step `step` of a call, from u to out, of the instances beyond the windows' bound (state 1), whose solved unknowns
// are in LX: the backward half of it and (NEXT) the forward half of the next step, whose rows the block still holds in
// LDS.  The windows of one step take the step, and all later ones, of an instance whose state has come within the bound
// (a workgroup takes one of either: the launch mostly finds nothing to do).  beyond tells at s mod 3 if step s's state
// is not within it, from its rows as they are formed.  By the maximum principle an instance within the bound stays
// within it (its boundary values are, or the plan has no such calls), so steps are solved alike however a call is split.
template <typename S, bool NEXT>
__global__ __launch_bounds__(kReduceBlock, 3) void btcs_block_turn_kernel(
    const InstDesc* __restrict__ inst, const SysDesc* __restrict__ systems, const ChunkBlock* __restrict__ blocks,
    int n_blocks, const ChunkWin* __restrict__ wins, int n_wins, const S* __restrict__ u, S* __restrict__ out,
    double* __restrict__ LA, double* __restrict__ LC, double* __restrict__ LD, const double* __restrict__ LX, int* state,
    int* beyond, int64_t count, int64_t step, double theta_lim) {
  using T = double;
  constexpr int NT = kReduceBlock;
  constexpr int kStageBytes = padded_size(kRedRows) * static_cast<int>(sizeof(S));
  constexpr int kBlockBytes = kStageBytes > BlockIfaceSpace::kBytes ? kStageBytes : BlockIfaceSpace::kBytes;
  constexpr int kBytes = kBlockBytes > WindowSpace<S, NT>::kBytes ? kBlockBytes : WindowSpace<S, NT>::kBytes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kBytes];
  __shared__ int iface_flags[2 * kSpikeWaves];
  __shared__ uint64_t iface_votes[2 * InterfaceSpace<T, NT>::kVoteWords];
  __shared__ double wave_max[NT / 64];
  if (state[-1] == 0) return;                    // (one word, before the tables: an idle launch is most of them)
  // (both roles' tables and states read at once: their latencies would add up)
  const int turn = static_cast<int>(blockIdx.x);
  const ChunkWin cw = wins[turn < n_wins ? turn : 0];
  const ChunkBlock cb = blocks[turn < n_blocks ? turn : 0];
  const int* now = beyond + step % 3 * count;
  const SysDesc sys = systems[cb.sys];
  const int win_state = state[cw.inst], win_beyond = now[cw.inst];
  const int sys_state = state[sys.inst], sys_beyond = now[sys.inst];
  S* stage = reinterpret_cast<S*>(smem);
  T* lds = reinterpret_cast<T*>(smem);
  // a window, ...
  if (turn < n_wins && (win_state == 2 || (win_state == 1 && step > 0 && win_beyond == 0))) {
    if (threadIdx.x == 0) state[cw.inst] = 2;    // (other workgroups of the launch find 1 or 2, and decide alike)
    const InstDesc d = inst[cw.inst];
    const InterfaceSpace<T, NT> ws{lds, lds + 3 * NT, iface_votes};
    ws.clear_votes();
    const Frame f(system_rows(d), cw);
    const int dir = d.bc == kDirichlet ? 1 : 0;
    window_load<S, NT, false>(u + d.off + dir, stage, f);
    __syncthreads();
    window_advance<S, NT>(ws, stage, f, cw, d, 1, kMaxPcr, [](const auto&) {});
    S* __restrict__ y = out + d.off + dir;
    window_kept<NT, kStepHalo>(f, cw, [&](int k, int i) { y[k] = stage[padded(i)]; });
    window_ends<S>(f, cw, d, out);
    __syncthreads();                             // (the rows below take their place)
  }
  // ... then a block
  const BlockIfaceSpace w{lds, lds + 3 * BlockIfaceSpace::kN, iface_flags};
  if (turn >= n_blocks || sys_state != 1 || (step > 0 && sys_beyond == 0)) return;
  const InstDesc d = inst[sys.inst];
  const bool dir = d.bc == kDirichlet;
  const int Pb = min(kReduceBlock, sys.chunks - cb.chunk0);
  int rs, re;
  block_rows(sys, cb.chunk0, rs, re);
  stage_in(stage, u + d.off + (dir ? 1 : 0) + rs, re - rs);
  __syncthreads();
  const bool full = block_full(sys, cb.chunk0, Pb);
  const double top = full ? block_backsub_body<true, true>(w, stage, d, sys, cb, rs, re, Pb, u, out, LX)
                          : block_backsub_body<false, true>(w, stage, d, sys, cb, rs, re, Pb, u, out, LX);
  const double M = workgroup_max<NT>(top, wave_max);
  if (threadIdx.x == 0) {
    if (!(theta_bound(d, M) <= theta_lim)) beyond[(step + 1) % 3 * count + sys.inst] = 1;
    if (cb.chunk0 == 0) beyond[(step + 2) % 3 * count + sys.inst] = 0;   // (the last step's, read by the launch before)
  }
  if constexpr (NEXT) {
    if (full) block_reduce_body<true>(w, stage, d, sys, cb, rs, Pb, LA, LC, LD);
    else block_reduce_body<false>(w, stage, d, sys, cb, rs, Pb, LA, LC, LD);
  }
}

// The reduced systems of a partition level, one workgroup each, in the narrowest width that holds the
// level's widest system (small reduced systems leave most of a 512-lane workgroup idle).
void reduced_wg_launch(const BtcsPlan::Level& lv, double* LA, double* LC, double* LD, double* LX, hipStream_t st,
                       const int* only) {
  const SysDesc* sys = lv.wg->as<SysDesc>();
  const unsigned n = static_cast<unsigned>(lv.n_wg);
  switch (lv.wg_lanes) {
    case 64: btcs_reduced_kernel<64, kWgChunk><<<n, 64, 0, st>>>(sys, LA, LC, LD, LX, only); break;
    case 128: btcs_reduced_kernel<128, kWgChunk><<<n, 128, 0, st>>>(sys, LA, LC, LD, LX, only); break;
    case 256: btcs_reduced_kernel<256, kWgChunk><<<n, 256, 0, st>>>(sys, LA, LC, LD, LX, only); break;
    default:
      if (lv.wg_exact)   // the full layout as a constant: no row is selected at a run-time index
        btcs_reduced_kernel<kWgThreads, kWgChunk, true><<<n, kWgThreads, 0, st>>>(sys, LA, LC, LD, LX, only);
      else
        btcs_reduced_kernel<kWgThreads, kWgChunk><<<n, kWgThreads, 0, st>>>(sys, LA, LC, LD, LX, only);
      break;
  }
}

// Workgroups of the persistent per-step kernel: as many as the device holds at once.
template <typename S, int NT, int MC>
int stream_grid(int device) {
  static int cached[64] = {};
  if (device < 0 || device >= 64) return 256;
  if (!cached[device]) {
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus <= 0) cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, btcs_stream_kernel<S, NT, MC>, NT, 0) != hipSuccess ||
        per <= 0)
      per = 1;
    cached[device] = cus * per;
  }
  return cached[device];
}

// The partition levels' launches, forward and back to the level-0 unknowns' interfaces (levels_forward), and
// the last back-substitution into the new state (levels_finish).  `only` (optional): only the instances whose
// entry is 1; only[-1] is zero when there is none.
template <typename S>
void levels_forward(const burgers_ctx* ctx, const BtcsPlan& plan, const InstDesc* inst, const S* u, const int* only) {
  double* LA = ctx->level_a.as<double>();
  double* LC = ctx->level_c.as<double>();
  double* LD = ctx->level_d.as<double>();
  double* LX = ctx->level_x.as<double>();
  hipStream_t st = ctx->stream;
  const int L = static_cast<int>(plan.levels.size());
  // forward: reduce level by level
  for (int l = 0; l < L; ++l) {
    const auto& lv = plan.levels[l];
    if (lv.n_blocks == 0) continue;
    if (l == 0) {
      btcs_block_reduce_kernel<S><<<lv.n_blocks, kReduceBlock, 0, st>>>(
          inst, lv.sys->as<SysDesc>(), lv.blocks->as<ChunkBlock>(), u, LA, LC, LD, only);
    } else {
      btcs_array_reduce_kernel<<<lv.n_blocks, kReduceBlock, 0, st>>>(lv.sys->as<SysDesc>(),
                                                                     lv.blocks->as<ChunkBlock>(), LA, LC, LD, only);
    }
  }
  // backward: whole-system solves of each level, then back-substitution of the reduced systems
  for (int l = L - 1; l >= 1; --l) {
    const auto& lv = plan.levels[l];
    if (lv.n_wg) reduced_wg_launch(lv, LA, LC, LD, LX, st, only);
    if (lv.n_blocks) {
      btcs_array_backsub_kernel<<<lv.n_blocks, kReduceBlock, 0, st>>>(
          lv.sys->as<SysDesc>(), lv.blocks->as<ChunkBlock>(), LA, LC, LD, LX, only);
    }
  }
}

template <typename S>
void levels_finish(const burgers_ctx* ctx, const BtcsPlan& plan, const InstDesc* inst, const S* u, S* out,
                   const int* only) {
  if (plan.levels.empty() || plan.levels[0].n_blocks == 0) return;
  const auto& lv = plan.levels[0];
  btcs_block_backsub_kernel<S><<<lv.n_blocks, kReduceBlock, 0, ctx->stream>>>(
      inst, lv.sys->as<SysDesc>(), lv.blocks->as<ChunkBlock>(), u, out, ctx->level_x.as<double>(), only);
}

// nsteps steps of the instances beyond the windows' bound, the last one's rows in bufs[nsteps & 1] (u, work).  Where
// every system's reduced one is solved whole, a step is two launches: one for those and one that ends the step and
// begins the next.
template <typename S>
void beyond_run(const burgers_ctx* ctx, const BtcsPlan& plan, S* u, S* work, int64_t nsteps) {
  const InstDesc* inst = ctx->inst.as<InstDesc>();
  int* state = win_flag_slot(plan.win_flags.as<int>(), ctx->count, 0);
  int* beyond = deep_beyond(plan.deep_words.as<int>(), ctx->count);
  double* LA = ctx->level_a.as<double>();
  double* LC = ctx->level_c.as<double>();
  double* LD = ctx->level_d.as<double>();
  double* LX = ctx->level_x.as<double>();
  const auto& lv = plan.levels[0];
  const double lim = btcs_window_limit();
  const unsigned n = static_cast<unsigned>(std::max<int64_t>(lv.n_blocks, plan.n_turn));
  const bool two = plan.levels.size() == 2 && plan.levels[1].n_blocks == 0;
  S* bufs[2] = {u, work};
  for (int64_t s = 0; s < nsteps; ++s) {
    const S* from = bufs[s & 1];
    S* to = bufs[(s & 1) ^ 1];
    if (s == 0 || !two) levels_forward<S>(ctx, plan, inst, from, state);
    else reduced_wg_launch(plan.levels[1], LA, LC, LD, LX, ctx->stream, state);
    auto kernel = two && s + 1 < nsteps ? btcs_block_turn_kernel<S, true> : btcs_block_turn_kernel<S, false>;
    kernel<<<n, kReduceBlock, 0, ctx->stream>>>(inst, lv.sys->as<SysDesc>(), lv.blocks->as<ChunkBlock>(), lv.n_blocks,
                                                plan.turn->as<ChunkWin>(), static_cast<int>(plan.n_turn), from, to, LA,
                                                LC, LD, LX, state, beyond, ctx->count, s, lim);
  }
}

template <typename S>
hipError_t launch_step(const burgers_ctx* ctx, const BtcsPlan& plan, const void* uv, void* outv, int64_t step) {
  const S* u = static_cast<const S*>(uv);
  S* out = static_cast<S*>(outv);
  const InstDesc* inst = plan.inst_half && plan.inst_half->ptr ? plan.inst_half->as<InstDesc>()
                                                               : ctx->inst.as<InstDesc>();
  hipStream_t st = ctx->stream;
  // truncated windows of the long systems; the partition levels below then serve only the instances
  // whose windows flagged a failed bound this step
  const int* only = nullptr;
  if (plan.n_win > 0) {
    int* now = win_flag_slot(plan.win_flags.as<int>(), ctx->count, step);
    const hipError_t e = launch_btcs_windows(ctx, plan, inst, u, out, now,
                                             win_flag_slot(plan.win_flags.as<int>(), ctx->count, step + 1));
    if (e != hipSuccess) return e;
    only = now;
  }
  levels_forward<S>(ctx, plan, inst, u, only);
  for (const WgGroup& g : plan.wg_state) {
    if (!g.n) continue;
    const SysDesc* sys = g.sys->as<SysDesc>();
    const unsigned n = static_cast<unsigned>(g.n);
    // the pipelined kernel moves 16-byte chunks: the state buffers must be 16-byte aligned too
    if (g.shape.stream && ((reinterpret_cast<uintptr_t>(u) | reinterpret_cast<uintptr_t>(out)) & 15) == 0) {
      if (g.shape.lanes == 1024)
        btcs_stream_kernel<S, 1024, 8><<<std::min(n, static_cast<unsigned>(stream_grid<S, 1024, 8>(ctx->device))),
                                         1024, 0, st>>>(inst, sys, g.n, u, out);
      else
        btcs_stream_kernel<S, 512, 16><<<std::min(n, static_cast<unsigned>(stream_grid<S, 512, 16>(ctx->device))),
                                         512, 0, st>>>(inst, sys, g.n, u, out);
      continue;
    }
    const hipError_t e = launch_btcs_whole(ctx, inst, g, u, out);
    if (e != hipSuccess) return e;
  }
  levels_finish<S>(ctx, plan, inst, u, out, only);
  return hipGetLastError();
}

__global__ void clear_flags_kernel(int* __restrict__ p, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

}  // namespace

template <typename S>
void newton_launch(const burgers_ctx* ctx, const WgGroup& g, const S* u, S* x, int last, int* flags) {
  const InstDesc* inst = ctx->inst.as<InstDesc>();
  const SysDesc* sys = g.sys->as<SysDesc>();
  const unsigned n = static_cast<unsigned>(g.n);
  hipStream_t st = ctx->stream;
  switch (g.shape.lanes) {   // chunks of at most 8 rows in every class (8192 rows: 1024 lanes)
    case 128: newton_wg_kernel<S, 128, 8><<<n, 128, 0, st>>>(inst, sys, u, x, last, flags); break;
    case 256: newton_wg_kernel<S, 256, 8><<<n, 256, 0, st>>>(inst, sys, u, x, last, flags); break;
    case 512: newton_wg_kernel<S, 512, 8><<<n, 512, 0, st>>>(inst, sys, u, x, last, flags); break;
    default: newton_wg_kernel<S, 1024, 8><<<n, 1024, 0, st>>>(inst, sys, u, x, last, flags); break;
  }
}

hipError_t launch_newton_whole(const burgers_ctx* ctx, const WgGroup& group, const void* u, void* x, bool last,
                               int* flags) {
  if (group.n <= 0) return hipSuccess;
  if (ctx->dtype == BURGERS_F64)
    newton_launch<double>(ctx, group, static_cast<const double*>(u), static_cast<double*>(x), last ? 1 : 0, flags);
  else
    newton_launch<float>(ctx, group, static_cast<const float*>(u), static_cast<float*>(x), last ? 1 : 0, flags);
  return hipGetLastError();
}

// Width class of a system solved whole (btcs_solved_whole), by its rows alone, so that every solver of the
// system (on chip, per step, recording, in a pool) lays it out alike.  Up to 4096 rows a lane takes at most
// 8: fewer registers, so more workgroups per CU, and a shorter serial chain for a batch too small to fill
// the chip.  Beyond, 9 to 16 rows a lane: half the lanes, so half the interface solve's share per row, and
// two workgroups per CU up to 8192 rows (100 steps of the 4097..8191-row systems of a ragged batch of 10^4,
// as 1024 lanes of at most 8 rows: 2980 us).  `threads` = 1024 asks for 1024 lanes of 8 at 8192 rows.
WidthClass btcs_width_class(int rows, int threads) {
  if (rows == kWgRows && threads == 1024) return WidthClass{1024, 8};
  if (rows > kWgRows) return WidthClass{1024, 16};
  if (rows > kWgRows / 2) return WidthClass{512, 16};
  int lanes = 64;
  while (lanes * 8 < rows) lanes *= 2;
  return WidthClass{lanes, 8};
}

// Chunk count of the whole-system and on-chip solvers with `threads` lanes: the largest power of two P <= threads with
// two rows or more per chunk; systems of up to 8192 rows then have chunks of at most 8192 / threads.
int btcs_chunks(int rows, int threads) {
  int P = 1;
  while (2 * P <= threads && 2 * (2 * P) <= rows) P *= 2;
  return P;
}

int btcs_wg_capacity() { return kWgRows; }
int btcs_whole_capacity() { return kWholeRows; }
bool btcs_solved_whole(int64_t rows) { return rows <= kWholeRows; }

int btcs_wg_chunks(int rows) {
  // largest power of two P <= min(threads, rows / 2); rows <= capacity keeps every chunk <= kWgChunk
  int P = 1;
  while (2 * P <= kWgThreads && 2 * (2 * P) <= rows) P *= 2;
  return P;
}

int btcs_reduce_chunk() { return kRedChunk; }

bool btcs_wg_exact(const std::vector<SysDesc>& systems) {
  for (const SysDesc& sd : systems)
    if (sd.rows != kWgRows || sd.chunks != kWgThreads) return false;
  return !systems.empty();
}

int btcs_wg_lanes(const std::vector<SysDesc>& systems) {
  int lanes = 64;
  for (const SysDesc& sd : systems)
    while (lanes < sd.chunks) lanes *= 2;
  return lanes < kWgThreads ? lanes : kWgThreads;
}

// Solve systems stored in (A, C, D) arrays with unit diagonal (all levels array-sourced); the solution
// lands in X at each root system's offset.  levels[0] holds the roots that need partitioning.
hipError_t launch_array_solve(const burgers_ctx* ctx, const BtcsPlan& plan, double* LA, double* LC,
                              double* LD, double* LX, const int* only) {
  hipStream_t st = ctx->stream;
  const int L = static_cast<int>(plan.levels.size());
  for (int l = 0; l < L; ++l) {
    const auto& lv = plan.levels[l];
    if (lv.n_blocks)
      btcs_array_reduce_kernel<<<lv.n_blocks, kReduceBlock, 0, st>>>(lv.sys->as<SysDesc>(),
                                                                     lv.blocks->as<ChunkBlock>(), LA, LC, LD, only);
  }
  for (int l = L - 1; l >= 0; --l) {
    const auto& lv = plan.levels[l];
    if (lv.n_wg) reduced_wg_launch(lv, LA, LC, LD, LX, st, only);
    if (lv.n_blocks)
      btcs_array_backsub_kernel<<<lv.n_blocks, kReduceBlock, 0, st>>>(lv.sys->as<SysDesc>(),
                                                                      lv.blocks->as<ChunkBlock>(), LA, LC, LD, LX,
                                                                      only);
  }
  return hipGetLastError();
}

hipError_t launch_btcs_step(const burgers_ctx* ctx, const BtcsPlan& plan, const void* u, void* out, int64_t step) {
  if (ctx->dtype == BURGERS_F64) return launch_step<double>(ctx, plan, u, out, step);
  return launch_step<float>(ctx, plan, u, out, step);
}

hipError_t launch_btcs_beyond(const burgers_ctx* ctx, const BtcsPlan& plan, void* u, void* work, int64_t nsteps) {
  if (ctx->dtype == BURGERS_F64) beyond_run<double>(ctx, plan, static_cast<double*>(u), static_cast<double*>(work), nsteps);
  else beyond_run<float>(ctx, plan, static_cast<float*>(u), static_cast<float*>(work), nsteps);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && (nsteps & 1))
    e = launch_copy_tiles(ctx, plan.copy->as<Tile>(), plan.n_copy, work, u,
                          win_flag_slot(plan.win_flags.as<int>(), ctx->count, 0));
  return e;
}

hipError_t launch_btcs_window_reset(const burgers_ctx* ctx, const BtcsPlan& plan) {
  if (plan.n_win == 0) return hipSuccess;
  const int64_t n = 2 * (ctx->count + 1);     // both parity slots, not the sticky words
  clear_flags_kernel<<<static_cast<unsigned>((n + 255) / 256), 256, 0, ctx->stream>>>(plan.win_flags.as<int>(), n);
  return hipGetLastError();
}

hipError_t launch_clear_ints(const burgers_ctx* ctx, int* p, int64_t n) {
  if (n <= 0) return hipSuccess;
  clear_flags_kernel<<<static_cast<unsigned>((n + 255) / 256), 256, 0, ctx->stream>>>(p, n);
  return hipGetLastError();
}

}  // namespace burgers
