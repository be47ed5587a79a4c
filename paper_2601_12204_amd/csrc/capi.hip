// C ABI and host runtime of the gfx950 Burgers library: contexts, packed layout, launch plans and the
// stepping loops (ping-pong between the caller's state buffer and the context's second buffer).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <tuple>

#include "internal.hpp"

using burgers::ChunkBlock;
using burgers::DevBuf;
using burgers::InstDesc;
using burgers::SysDesc;
using burgers::Tile;
using burgers::BlockTile;

namespace burgers {

bool explicit_windows(int32_t i, int32_t n, bool periodic, int depth, bool rk4, std::vector<BlockTile>& out) {
  const int cap = explicit_block_capacity();
  // each step consumes one halo node per side per stage
  const int32_t halo = depth * (rk4 ? 4 : 1);
  const int32_t wout = cap - 2 * halo;
  if (wout < 1) return false;
  const int64_t nn = n;
  for (int64_t lo = 0; lo < nn; lo += wout) {
    const int64_t hi = std::min<int64_t>(nn, lo + wout);
    BlockTile bt{i, 0, 0, 0, static_cast<int32_t>(hi - lo), 0, rk4 ? 1 : 0, 0};
    if (periodic) {
      bt.first = static_cast<int32_t>(((lo - halo) % nn + nn) % nn);
      bt.width = static_cast<int32_t>((hi - lo) + 2 * halo);
      bt.lo = halo;
    } else {
      const int64_t first = std::max<int64_t>(0, lo - halo);
      bt.first = static_cast<int32_t>(first);
      bt.width = static_cast<int32_t>(std::min<int64_t>(nn, hi + halo) - first);
      bt.lo = static_cast<int32_t>(lo - first);
    }
    out.push_back(bt);
  }
  return true;
}

}  // namespace burgers

namespace {

// Instance subsets a plan is built for; kSetBtcsHbm holds the BTCS-scheme instances like kSetBtcs but
// steps every one through HBM (the adjoint's out-of-place recompute of a checkpoint segment).
enum SetId { kSetAll = 0, kSetExplicit = 1, kSetBtcs = 2, kSetBtcsHbm = 3 };

bool valid_problem(const burgers_problem& p);
double grid_dx(const burgers_problem& p);

}  // namespace

namespace burgers {

bool problem_valid(const burgers_problem& p) { return valid_problem(p); }

InstDesc inst_desc(const burgers_problem& p, int64_t off) {
  InstDesc d{};
  d.off = off;
  d.n = static_cast<int32_t>(p.n);
  d.bc = p.bc;
  burgers_ratios(&p, &d.r, &d.D);
  const double dxv = grid_dx(p);
  d.dtdx2 = p.dt / (dxv * dxv);
  d.a = p.bc == BURGERS_BC_DIRICHLET ? p.left : 0.0;
  d.b = p.bc == BURGERS_BC_DIRICHLET ? p.right : 0.0;
  return d;
}

// Runs independent chains of launches: over the context's stream and up to three side streams of the context,
// forked from it and joined back with events (under graph capture they become parallel branches of the
// graph).  A process has four hardware queues here, and streams beyond them share one: a stream waiting for an
// event then holds up the others of its queue, so no more are taken than the chains' estimates need (three
// contexts in turn on three side streams each, a small ragged batch: 505 us a call, on one each 358).
// Chains of little work beside the longest stay on one stream: a fork and join cost about as much as they
// would gain.
hipError_t run_tasks(burgers_ctx* ctx, std::vector<Task>& tasks, bool serial) {
  constexpr double kWorthForking = 15.0;   // us
  std::stable_sort(tasks.begin(), tasks.end(), [](const Task& x, const Task& y) { return x.us > y.us; });
  double beside = 0;
  for (size_t k = 1; k < tasks.size(); ++k) beside += tasks[k].us;
  hipError_t e = hipSuccess;
  if (serial || beside < kWorthForking) {
    for (const Task& t : tasks)
      if ((e = t.run()) != hipSuccess) return e;
    return e;
  }
  // into as few streams as finish with the longest chain (or with an even share of all of it)
  constexpr int kStreams = 4;
  const double room = 1.1 * std::max(tasks[0].us, (tasks[0].us + beside) / kStreams);
  double load[kStreams] = {0, 0, 0, 0};
  std::vector<int> place(tasks.size());
  for (size_t k = 0; k < tasks.size(); ++k) {
    int q = 0;
    while (q < kStreams && load[q] + tasks[k].us > room) ++q;
    if (q == kStreams) q = static_cast<int>(std::min_element(load, load + kStreams) - load);
    place[k] = q;
    load[q] += tasks[k].us;
  }
  SideStreams& sides = ctx->sides;
  for (int q = 1; q < kStreams; ++q) {
    if (load[q] == 0) continue;
    if (!sides.stream[q - 1] && (e = hipStreamCreateWithFlags(&sides.stream[q - 1], hipStreamNonBlocking)) != hipSuccess) return e;
    if (!sides.joined[q - 1] &&
        (e = hipEventCreateWithFlags(&sides.joined[q - 1], hipEventDisableTiming)) != hipSuccess)
      return e;
  }
  if (!sides.forked && (e = hipEventCreateWithFlags(&sides.forked, hipEventDisableTiming)) != hipSuccess) return e;
  hipStream_t main = ctx->stream;
  if ((e = hipEventRecord(sides.forked, main)) != hipSuccess) return e;
  for (int q = 1; q < kStreams && e == hipSuccess; ++q)
    if (load[q] > 0) e = hipStreamWaitEvent(sides.stream[q - 1], sides.forked, 0);
  // chains of few launches first: the host is done with them soon, and a chain of many then delays none
  std::vector<size_t> order(tasks.size());
  for (size_t k = 0; k < order.size(); ++k) order[k] = k;
  std::stable_sort(order.begin(), order.end(), [&](size_t x, size_t y) { return tasks[x].launches < tasks[y].launches; });
  for (size_t k : order) {
    if (e != hipSuccess) break;
    if (place[k] > 0) ctx->stream = sides.stream[place[k] - 1];
    e = tasks[k].run();
    ctx->stream = main;
  }
  // (joined after an error too: nothing enqueued may outlive the context's stream order)
  for (int q = 1; q < kStreams; ++q) {
    if (load[q] == 0) continue;
    hipError_t j = hipEventRecord(sides.joined[q - 1], sides.stream[q - 1]);
    if (j == hipSuccess) j = hipStreamWaitEvent(main, sides.joined[q - 1], 0);
    if (e == hipSuccess) e = j;
  }
  return e;
}

}  // namespace burgers

namespace {

bool is_finite(double x) { return std::isfinite(x); }

double grid_dx(const burgers_problem& p) {
  return p.bc == BURGERS_BC_PERIODIC ? p.length / static_cast<double>(p.n)
                                     : p.length / static_cast<double>(p.n - 1);
}

// Largest instance: node indices of a window (first node + up to 8192) and of staged blocks stay within
// 32-bit integers.
constexpr int64_t kMaxNodes = (int64_t{1} << 31) - 65536;

bool valid_problem(const burgers_problem& p) {
  if (p.n < 3 || p.n > kMaxNodes) return false;
  if (!is_finite(p.length) || p.length <= 0) return false;
  if (!is_finite(p.nu) || p.nu < 0) return false;
  if (!is_finite(p.dt) || p.dt <= 0) return false;
  if (p.bc != BURGERS_BC_PERIODIC && p.bc != BURGERS_BC_DIRICHLET) return false;
  if (p.scheme < BURGERS_EXPLICIT || p.scheme > BURGERS_NEWTON) return false;
  if (!is_finite(p.left) || !is_finite(p.right)) return false;
  return true;
}

burgers_status from_hip(hipError_t e) {
  if (e == hipSuccess) return BURGERS_OK;
  if (e == hipErrorOutOfMemory) return BURGERS_E_NOMEM;
  return BURGERS_E_DEVICE;
}

// Record a device error as sticky and translate it.
burgers_status note(burgers_ctx* ctx, hipError_t e) {
  if (e != hipSuccess && ctx->sticky == hipSuccess) ctx->sticky = e;
  return from_hip(e);
}

const std::vector<int32_t>& set_members(const burgers_ctx* ctx, int set) {
  return set == kSetAll ? ctx->set_all : (set == kSetExplicit ? ctx->set_explicit : ctx->set_btcs);
}

bool own_scheme_set(int set) { return set == kSetBtcs || set == kSetBtcsHbm; }

// Copy a host table to a new device buffer, in stream order (a pageable source may be released as soon
// as the call returns).
template <typename T>
hipError_t upload_on(hipStream_t stream, DevBuf& buf, const std::vector<T>& v) {
  hipError_t e = buf.alloc(v.size() * sizeof(T), stream);
  if (e != hipSuccess) return e;
  if (v.empty()) return hipSuccess;
  return hipMemcpyAsync(buf.ptr, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, stream);
}

// Streaming tiles covering every node of the members of one subset.
std::vector<Tile> stream_tiles(const burgers_ctx* ctx, const std::vector<int32_t>& members) {
  const int tile = burgers::explicit_tile_nodes(ctx->dtype);
  std::vector<Tile> tiles;
  for (int32_t i : members) {
    const int32_t n = static_cast<int32_t>(ctx->probs[i].n);
    for (int64_t s = 0; s < n; s += tile)   // 64-bit counter: n may be close to INT32_MAX
      tiles.push_back(Tile{ctx->offsets[i], n, static_cast<int32_t>(s), ctx->probs[i].bc, i});
  }
  return tiles;
}

// Tiles of a subset used to copy its instances back from the second buffer.
hipError_t ensure_copy(burgers_ctx* ctx, int set) {
  if (ctx->copy_tiles.count(set)) return hipSuccess;
  auto tiles = stream_tiles(ctx, set_members(ctx, set));
  auto buf = std::make_unique<DevBuf>();
  hipError_t e = upload_on(ctx->stream, *buf, tiles);
  if (e != hipSuccess) return e;
  ctx->copy_tiles[set] = {std::move(buf), static_cast<int64_t>(tiles.size())};
  return hipSuccess;
}

// Steps per launch of the explicit windows.  Each launch moves a window through HBM once (load and
// store) and recomputes 2 T halo nodes of its 8192 per step; T = 128 balances the two (3% halo work).
constexpr int kDefaultDepth = 128;
constexpr int kMaxDepth = 512;

// Explicit launch plan of one subset under the context's forced path (0 = automatic).
//   path 1: streaming kernel, one step per launch.
//   path 2: whole instances on chip, all steps in one launch (every instance must fit).
//   path 3: temporal blocking with `depth` steps per launch for every instance.
//   automatic: whole instances for those that fit, windows of `depth` steps for longer ones.
burgers_status ensure_explicit(burgers_ctx* ctx, int set) {
  auto it = ctx->explicit_plans.find(set);
  const int want_path = ctx->plan.explicit_path;
  const int want_depth = ctx->plan.tblock_depth > 0 ? ctx->plan.tblock_depth : kDefaultDepth;
  if (it != ctx->explicit_plans.end() && it->second->path == (want_path ? want_path : 0) &&
      it->second->depth == want_depth)
    return BURGERS_OK;
  auto plan = std::make_unique<burgers::ExplicitPlan>();
  plan->path = want_path ? want_path : 0;
  plan->depth = want_depth;
  const auto& members = set_members(ctx, set);
  // instances advanced by their own scheme (burgers_run) take RK4 where they ask for it; a forward-Euler
  // call (burgers_step_explicit) steps every instance with forward Euler
  auto is_rk4 = [&](int32_t i) { return set == kSetExplicit && ctx->probs[i].scheme == BURGERS_RK4; };
  bool any_rk4 = false;
  for (int32_t i : members) any_rk4 = any_rk4 || is_rk4(i);
  if (plan->path == 1 && any_rk4) return BURGERS_E_UNSUPPORTED;   // the streaming kernel is forward Euler only
  hipError_t e;
  auto st = stream_tiles(ctx, members);
  plan->stream = std::make_unique<DevBuf>();
  if ((e = upload_on(ctx->stream, *plan->stream, st)) != hipSuccess) return from_hip(e);
  plan->n_stream = static_cast<int64_t>(st.size());
  if (plan->path != 1) {
    const int cap = burgers::explicit_block_capacity();
    const int T = plan->depth;
    std::vector<BlockTile> whole, win;
    std::vector<int32_t> windowed;
    for (int32_t i : members) {
      const burgers_problem& p = ctx->probs[i];
      const int32_t n = static_cast<int32_t>(p.n);
      const bool periodic = p.bc == BURGERS_BC_PERIODIC;
      const int32_t rk4 = is_rk4(i) ? 1 : 0;
      if (n <= cap) {
        whole.push_back(BlockTile{i, 0, n, 0, n, periodic ? 1 : 0, rk4});
        continue;
      }
      if (plan->path == 2) return BURGERS_E_UNSUPPORTED;
      windowed.push_back(i);
      if (!burgers::explicit_windows(i, n, periodic, T, rk4 != 0, win)) return BURGERS_E_UNSUPPORTED;
    }
    auto fe_first = [](const BlockTile& x, const BlockTile& y) { return x.rk4 < y.rk4; };
    // whole instances: by workgroup width (widest first), then forward Euler before RK4
    auto lanes_of = [](const BlockTile& x) { return burgers::explicit_block_lanes(x.width); };
    std::stable_sort(whole.begin(), whole.end(), [&](const BlockTile& x, const BlockTile& y) {
      const int lx = lanes_of(x), ly = lanes_of(y);
      if (lx != ly) return lx > ly;
      if (x.rk4 != y.rk4) return x.rk4 < y.rk4;
      return lx == 64 && (x.width + 63) / 64 > (y.width + 63) / 64;   // (one wave each: the longest running first)
    });
    plan->whole_classes.clear();
    for (size_t k = 0; k < whole.size();) {
      const int lanes = lanes_of(whole[k]);
      size_t e = k;
      int64_t rk4 = 0;
      while (e < whole.size() && lanes_of(whole[e]) == lanes) rk4 += whole[e++].rk4 ? 1 : 0;
      plan->whole_classes.push_back({lanes, static_cast<int64_t>(k), static_cast<int64_t>(e - k) - rk4, rk4});
      k = e;
    }
    // the classes below the widest packed for one launch per scheme, 512 / lanes instances of a class per
    // workgroup (widest first); the widest class keeps its own kernel, whose step loop compiles to fewer
    // registers than the pack kernel's (4096 instances of 8192 nodes: 61.9 against 63.9 ms).  Instances of one
    // wave are packed only beside others (one launch instead of two that may have to wait for each other);
    // alone they take workgroups of four waves, one per SIMD (64 instances of 1000 nodes, binary64: 0.22 us a
    // step against 0.39 with eight)
    plan->pack_waves = std::any_of(plan->whole_classes.begin(), plan->whole_classes.end(), [](const auto& c) {
      return c.lanes > 64 && c.lanes < burgers::explicit_pack_lanes();
    });
    std::vector<burgers::BlockPack> fe_packs, rk4_packs;
    for (const auto& c : plan->whole_classes) {
      if (c.lanes >= burgers::explicit_pack_lanes() || (c.lanes == 64 && !plan->pack_waves)) continue;
      const int per = burgers::explicit_pack_lanes() / c.lanes;
      auto pack = [&](int64_t first, int64_t count, std::vector<burgers::BlockPack>& out) {
        for (int64_t q = 0; q < count; q += per)
          out.push_back(burgers::BlockPack{static_cast<int32_t>(first + q),
                                           static_cast<int32_t>(std::min<int64_t>(per, count - q)), c.lanes, 0});
      };
      pack(c.offset, c.n_fe, fe_packs);
      pack(c.offset + c.n_fe, c.n_rk4, rk4_packs);
    }
    plan->n_packs_fe = static_cast<int64_t>(fe_packs.size());
    plan->n_packs_rk4 = static_cast<int64_t>(rk4_packs.size());
    fe_packs.insert(fe_packs.end(), rk4_packs.begin(), rk4_packs.end());
    plan->packs = std::make_unique<DevBuf>();
    if ((e = upload_on(ctx->stream, *plan->packs, fe_packs)) != hipSuccess) return from_hip(e);
    std::stable_sort(win.begin(), win.end(), fe_first);
    plan->whole = std::make_unique<DevBuf>();
    plan->win = std::make_unique<DevBuf>();
    plan->win_copy = std::make_unique<DevBuf>();
    auto wc = stream_tiles(ctx, windowed);
    if ((e = upload_on(ctx->stream, *plan->whole, whole)) != hipSuccess || (e = upload_on(ctx->stream, *plan->win, win)) != hipSuccess ||
        (e = upload_on(ctx->stream, *plan->win_copy, wc)) != hipSuccess)
      return from_hip(e);
    plan->n_win = static_cast<int64_t>(win.size());
    plan->n_win_rk4 = std::count_if(win.begin(), win.end(), [](const BlockTile& b) { return b.rk4 != 0; });
    plan->n_win_copy = static_cast<int64_t>(wc.size());
  }
  ctx->explicit_plans[set] = std::move(plan);
  return BURGERS_OK;
}

burgers_status ensure_newton(burgers_ctx* ctx, const std::vector<int32_t>& members);

// Rows a partition level leaves for the next one.  Level 0 (from the state) runs the block partition,
// which reduces each workgroup's 256 chunks to two rows; deeper levels leave two rows per chunk.
int32_t reduced_rows(int level, int32_t chunks) {
  if (level == 0) return 2 * ((chunks + burgers::kReduceBlock - 1) / burgers::kReduceBlock);
  return 2 * chunks;
}

// Implicit launch plan of one instance subset under the context's forced path (0 = automatic).
//   path 1: every step through HBM; whole-system solves for systems of up to 16384 rows, windows or
//           partition levels for longer ones.
//   path 2: systems of up to 8192 rows (or exactly 16384) stay on chip for all steps of a launch (every
//           system must fit).
//   path 3: partition levels for every system of at least 32 rows (shorter ones solved whole).
//   automatic: on chip for systems that fit (BTCS up to 16384 rows, Crank-Nicolson and Newton up to 8192),
//           the others as on path 1.
// Reduced-system rows are carved from the context's level arrays.
burgers_status ensure_btcs(burgers_ctx* ctx, int set) {
  const int want = set == kSetBtcsHbm ? 1 : ctx->plan.btcs_path;
  const int threads = ctx->plan.btcs_block ? ctx->plan.btcs_block : burgers::kResidentThreadsDefault;
  const int longmode = ctx->plan.btcs_long;
  auto found = ctx->btcs.find(set);
  const bool pipelined = ctx->plan.btcs_pipeline == 1;
  if (found != ctx->btcs.end() && found->second->path == want && found->second->threads == threads &&
      found->second->longmode == longmode && found->second->stream_exact == pipelined)
    return BURGERS_OK;
  auto plan = std::make_unique<burgers::BtcsPlan>();
  plan->path = want;
  plan->threads = threads;
  plan->longmode = longmode;
  plan->stream_exact = pipelined;
  const int cap = burgers::btcs_wg_capacity();
  const int chunk = burgers::btcs_reduce_chunk();
  // truncated windows of the long systems (automatic and per-step paths); the partition levels stay as the
  // fallback for failed bounds.  One step per launch: 4096 rows each (8192 when asked); on the automatic path
  // also windows of several steps, where they are all that steps through HBM (see enqueue_stepped)
  plan->win_rows = longmode == 2 ? cap : 4096;
  std::vector<burgers::ChunkWin> windows, deep, turn;
  std::vector<int32_t> windowed;
  bool only_windows = want == 0 && !burgers::tl_arena;
  auto add_windows = [&](int32_t i, int32_t R, bool is_cn) {
    const bool periodic = ctx->probs[i].bc == BURGERS_BC_PERIODIC;
    burgers::btcs_step_windows(i, R, periodic, plan->win_rows, is_cn, windows);
    if (is_cn) return;
    burgers::btcs_deep_windows(i, R, periodic, deep);
    burgers::btcs_step_windows(i, R, periodic, 4096, false, turn);
    windowed.push_back(i);
    // (boundary values beyond the bound may bring an instance within it beyond it again: every step is then judged
    // by itself)
    const burgers::InstDesc& d = ctx->inst_host[i];
    const double edge = std::max(std::abs(d.a), std::abs(d.b));
    only_windows = only_windows && burgers::btcs_window_theta(d, edge) <= burgers::btcs_window_limit() * (1.0 - 1e-9);
  };
  // whole-system systems grouped by width class (lanes, chunk)
  std::map<std::pair<int, int>, std::vector<SysDesc>> wg_state, resident, streamed, cn_chip, newton_chip;
  const int64_t elem = ctx->dtype == BURGERS_F64 ? 8 : 4;
  auto whole = [&](std::map<std::pair<int, int>, std::vector<SysDesc>>& groups, int32_t rows, int32_t i,
                   bool is_cn) {
    const burgers::WidthClass w = burgers::btcs_width_class(rows, threads);
    groups[{w.lanes, w.chunk}].push_back(
        SysDesc{0, -1, rows, burgers::btcs_chunks(rows, w.lanes), i, 0, is_cn ? 1 : 0});
  };
  // Crank-Nicolson and Newton systems of up to 8192 rows, held on chip on the automatic path
  auto on_chip = [&](std::map<std::pair<int, int>, std::vector<SysDesc>>& groups, int32_t rows, int32_t i) {
    const burgers::WidthClass w = burgers::chip_width_class(rows);
    groups[{w.lanes, w.chunk}].push_back(SysDesc{0, -1, rows, burgers::btcs_chunks(rows, w.lanes), i, 0});
  };
  std::vector<int32_t> stepped, cn, newton;
  std::vector<std::vector<SysDesc>> red_sys, wg_sys;
  int64_t rows_used = 0;
  for (int32_t i : set_members(ctx, set)) {
    const burgers_problem& p = ctx->probs[i];
    const int32_t R0 = static_cast<int32_t>(p.bc == BURGERS_BC_PERIODIC ? p.n : p.n - 2);
    const bool fits = burgers::btcs_solved_whole(R0);
    // (Crank-Nicolson instances are those advanced by their own scheme; burgers_step_btcs takes them as BTCS)
    const bool is_cn = own_scheme_set(set) && p.scheme == BURGERS_CN;
    if (is_cn) cn.push_back(i);
    const bool is_newton = own_scheme_set(set) && p.scheme == BURGERS_NEWTON;
    // (the forced on-chip path takes systems of up to 8192 rows, or of exactly 16384)
    const bool forced_fits = R0 <= cap || R0 == burgers::btcs_whole_capacity();
    if (want == 2 && (!forced_fits || is_cn || is_newton)) return BURGERS_E_UNSUPPORTED;
    if (is_newton) {            // Newton iterations of their own
      newton.push_back(i);
      if (want == 0 && R0 <= cap) {
        on_chip(newton_chip, R0, i);
        continue;
      }
      stepped.push_back(i);
      plan->newton = true;
      plan->newton_whole = want != 0;
      continue;
    }
    if (is_cn && want == 0 && R0 <= cap) {
      on_chip(cn_chip, R0, i);
      continue;
    }
    if ((want == 0 || want == 2) && fits && !is_cn) {
      whole(resident, R0, i, false);
      continue;
    }
    stepped.push_back(i);
    const bool partition = want == 3 ? R0 >= 32 : !fits;
    if (!partition) {
      // exact 8192-row systems whose first row is 16-byte aligned may take the pipelined kernel
      const int64_t first = ctx->inst_host[i].off + (p.bc == BURGERS_BC_PERIODIC ? 0 : 1);
      const bool streams = pipelined && !is_cn && R0 == burgers::btcs_wg_capacity() && (first * elem) % 16 == 0;
      whole(streams ? streamed : wg_state, R0, i, is_cn);
      continue;
    }
    if (want != 3 && longmode != 1) add_windows(i, R0, is_cn);
    int32_t R = R0;
    int64_t in_off = 0;
    for (int level = 0;; ++level) {
      if (static_cast<int>(red_sys.size()) <= level) {
        red_sys.resize(level + 1);
        wg_sys.resize(level + 1);
      }
      if (level > 0 && R <= cap) {
        wg_sys[level].push_back(SysDesc{in_off, -1, R, burgers::btcs_wg_chunks(R), i, level});
        break;
      }
      const int32_t P = (R + chunk - 1) / chunk;
      const int32_t out_rows = reduced_rows(level, P);
      const int64_t red = rows_used;
      rows_used += out_rows;
      red_sys[level].push_back(SysDesc{in_off, red, R, P, i, level, (level == 0 && is_cn) ? 1 : 0});
      in_off = red;
      R = out_rows;
    }
  }
  if (rows_used > ctx->level_capacity) return BURGERS_E_NOMEM;   // sized at create for every path
  plan->level_rows = rows_used;
  hipError_t e;
  auto upload_groups = [&](std::map<std::pair<int, int>, std::vector<SysDesc>>& groups,
                           std::vector<burgers::WgGroup>& out, bool stream) -> hipError_t {
    for (auto& kv : groups) {
      burgers::WgGroup g;
      g.shape = burgers::WidthClass{kv.first.first, kv.first.second, stream};
      g.sys = std::make_unique<DevBuf>();
      g.n = static_cast<int32_t>(kv.second.size());
      g.exact = std::all_of(kv.second.begin(), kv.second.end(),
                            [&](const SysDesc& sd) { return sd.rows == g.shape.lanes * g.shape.chunk; });
      hipError_t err = upload_on(ctx->stream, *g.sys, kv.second);
      if (err != hipSuccess) return err;
      out.push_back(std::move(g));
    }
    return hipSuccess;
  };
  plan->copy = std::make_unique<DevBuf>();
  auto ct = stream_tiles(ctx, stepped);
  plan->n_copy = static_cast<int64_t>(ct.size());
  if (!newton.empty()) {
    burgers_status nst = ensure_newton(ctx, newton);
    if (nst != BURGERS_OK) return nst;
  }
  plan->inst_half = std::make_unique<DevBuf>();
  if (!cn.empty()) {
    std::vector<burgers::InstDesc> half = ctx->inst_host;
    for (int32_t i : cn) {
      half[i].r = 0.5 * half[i].r;               // the BTCS rows of dt/2 (exact: a power of two)
      half[i].D = 0.5 * half[i].D;
    }
    if ((e = upload_on(ctx->stream, *plan->inst_half, half)) != hipSuccess) return from_hip(e);
  }
  if ((e = upload_groups(wg_state, plan->wg_state, false)) != hipSuccess ||
      (e = upload_groups(streamed, plan->wg_state, true)) != hipSuccess ||
      (e = upload_groups(resident, plan->resident, false)) != hipSuccess ||
      (e = upload_groups(cn_chip, plan->cn_chip, false)) != hipSuccess ||
      (e = upload_groups(newton_chip, plan->newton_chip, false)) != hipSuccess ||
      (e = upload_on(ctx->stream, *plan->copy, ct)) != hipSuccess)
    return from_hip(e);
  plan->win = std::make_unique<DevBuf>();
  if ((e = upload_on(ctx->stream, *plan->win, windows)) != hipSuccess) return from_hip(e);
  plan->n_win = static_cast<int64_t>(windows.size());
  if (plan->n_win > 0 &&
      (e = plan->win_flags.alloc(static_cast<size_t>(burgers::win_flags_words(ctx->count)) * sizeof(int), ctx->stream)) !=
          hipSuccess)
    return from_hip(e);
  if (only_windows && !windowed.empty() && windowed.size() == stepped.size()) {
    const int64_t words = burgers::deep_words(ctx->count);
    plan->deep = std::make_unique<DevBuf>();
    plan->deep_inst = std::make_unique<DevBuf>();
    plan->turn = std::make_unique<DevBuf>();
    if ((e = upload_on(ctx->stream, *plan->deep, deep)) != hipSuccess ||
        (e = upload_on(ctx->stream, *plan->deep_inst, windowed)) != hipSuccess ||
        (e = upload_on(ctx->stream, *plan->turn, turn)) != hipSuccess ||
        (e = plan->deep_words.alloc(static_cast<size_t>(words) * sizeof(int), ctx->stream)) != hipSuccess ||
        (e = burgers::launch_clear_ints(ctx, plan->deep_words.as<int>(), words)) != hipSuccess)
      return from_hip(e);
    plan->n_deep = static_cast<int64_t>(deep.size());
    plan->n_deep_inst = static_cast<int64_t>(windowed.size());
    plan->n_turn = static_cast<int64_t>(turn.size());
  }
  plan->levels.resize(red_sys.size());
  for (size_t l = 0; l < red_sys.size(); ++l) {
    auto& lv = plan->levels[l];
    std::vector<ChunkBlock> blocks;
    for (size_t si = 0; si < red_sys[l].size(); ++si)
      for (int64_t c = 0; c < red_sys[l][si].chunks; c += burgers::kReduceBlock)
        blocks.push_back(ChunkBlock{static_cast<int32_t>(si), static_cast<int32_t>(c)});
    lv.sys = std::make_unique<DevBuf>();
    lv.blocks = std::make_unique<DevBuf>();
    lv.wg = std::make_unique<DevBuf>();
    if ((e = upload_on(ctx->stream, *lv.sys, red_sys[l])) != hipSuccess || (e = upload_on(ctx->stream, *lv.blocks, blocks)) != hipSuccess ||
        (e = upload_on(ctx->stream, *lv.wg, wg_sys[l])) != hipSuccess)
      return from_hip(e);
    lv.n_blocks = static_cast<int32_t>(blocks.size());
    lv.n_wg = static_cast<int32_t>(wg_sys[l].size());
    lv.wg_lanes = burgers::btcs_wg_lanes(wg_sys[l]);
    lv.wg_exact = burgers::btcs_wg_exact(wg_sys[l]);
  }
  ctx->btcs[set] = std::move(plan);
  return BURGERS_OK;
}

// Rows of the partition levels the instances can need on any path (sizes the level arrays).
int64_t level_rows_needed(const burgers_ctx* ctx) {
  const int cap = burgers::btcs_wg_capacity();
  const int chunk = burgers::btcs_reduce_chunk();
  int64_t rows = 0;
  for (const auto& p : ctx->probs) {
    int64_t R = p.bc == BURGERS_BC_PERIODIC ? p.n : p.n - 2;
    if (R < 32) continue;                      // partition levels serve systems of >= 32 rows
    for (int level = 0;; ++level) {
      if (level > 0 && R <= cap) break;
      const int64_t P = (R + chunk - 1) / chunk;
      const int64_t out_rows = reduced_rows(level, static_cast<int32_t>(P));
      rows += out_rows;
      R = out_rows;
    }
  }
  return rows;
}

// The independent launch chains of a call (they advance disjoint instances), each with a rough time: the
// larger of its latency and its throughput on an otherwise idle chip, in us per step, from measurements of
// the kernels (only their order and rough size matter: run_tasks spreads the chains over streams by it).
double chain_us(int64_t steps, double latency, double nodes, double nodes_per_us) {
  return static_cast<double>(steps) * std::max(latency, nodes / nodes_per_us);
}

// nsteps explicit steps of one subset, the final state in u.
void explicit_tasks(burgers_ctx* ctx, int set, void* u, int64_t nsteps, std::vector<burgers::Task>& tasks) {
  const burgers::ExplicitPlan* pl = ctx->explicit_plans[set].get();
  void* work = ctx->work.ptr;
  const double tile = burgers::explicit_tile_nodes(ctx->dtype);
  if (pl->path == 1) {
    if (pl->n_stream == 0) return;
    tasks.push_back({chain_us(nsteps, 3.0, pl->n_stream * tile, 4e5), nsteps, [=]() -> hipError_t {
      hipError_t e = hipSuccess;
      void* bufs[2] = {u, work};
      int cur = 0;
      for (int64_t s = 0; s < nsteps; ++s) {
        if ((e = burgers::launch_explicit_stream(ctx, pl->stream->as<Tile>(), pl->n_stream, bufs[cur], bufs[cur ^ 1])) != hipSuccess)
          return e;
        cur ^= 1;
      }
      if (cur) e = burgers::launch_copy_tiles(ctx, pl->stream->as<Tile>(), pl->n_stream, work, u);
      return e;
    }});
    return;
  }
  // whole instances, in place: all steps at once, or `depth` per launch on path 3
  const int64_t whole_chunk = pl->path == 3 ? pl->depth : (int64_t{1} << 30);
  auto in_chunks = [=](auto launch) -> hipError_t {
    for (int64_t done = 0; done < nsteps;) {
      const int k = static_cast<int>(std::min(whole_chunk, nsteps - done));
      const hipError_t e = launch(k);
      if (e != hipSuccess) return e;
      done += k;
    }
    return hipSuccess;
  };
  double packed = 0;
  for (const auto& c : pl->whole_classes) {
    const double nodes = 12.0 * c.lanes * static_cast<double>(c.n_fe + 4 * c.n_rk4);   // (about 12 of 16 a lane)
    const bool own = c.lanes >= burgers::explicit_pack_lanes() || (c.lanes == 64 && !pl->pack_waves);
    if (!own) {
      packed += nodes;
      continue;
    }
    tasks.push_back({chain_us(nsteps, c.lanes == 64 ? 0.25 : 0.5, nodes, 4e6), 1, [=]() {
      return in_chunks([&](int k) {
        return burgers::launch_explicit_block(ctx, pl->whole->as<BlockTile>() + c.offset, c.n_fe, c.n_rk4, u, u, k, c.lanes);
      });
    }});
  }
  if (pl->n_packs_fe + pl->n_packs_rk4 > 0)
    tasks.push_back({chain_us(nsteps, 0.5, packed, 4e6), 1, [=]() {
      return in_chunks([&](int k) {
        return burgers::launch_explicit_packs(ctx, pl->whole->as<BlockTile>(), pl->packs->as<burgers::BlockPack>(),
                                              pl->n_packs_fe, pl->n_packs_rk4, u, k);
      });
    }});
  // windows of long instances: `depth` steps per launch, ping-pong
  if (pl->n_win > 0)
    tasks.push_back({chain_us(nsteps, 0.6, 8192.0 * static_cast<double>(pl->n_win), 4e6), nsteps / pl->depth + 1,
                     [=]() -> hipError_t {
      hipError_t e = hipSuccess;
      void* bufs[2] = {u, work};
      int cur = 0;
      for (int64_t done = 0; done < nsteps;) {
        const int k = static_cast<int>(std::min<int64_t>(pl->depth, nsteps - done));
        if ((e = burgers::launch_explicit_block(ctx, pl->win->as<BlockTile>(), pl->n_win - pl->n_win_rk4, pl->n_win_rk4,
                                                bufs[cur], bufs[cur ^ 1], k)) != hipSuccess)
          return e;
        cur ^= 1;
        done += k;
      }
      if (cur) e = burgers::launch_copy_tiles(ctx, pl->win_copy->as<Tile>(), pl->n_win_copy, work, u);
      return e;
    }});
}

// nsteps implicit steps through HBM of a plan's stepped instances, the final state in u.
hipError_t enqueue_stepped(burgers_ctx* ctx, const burgers::BtcsPlan& pl, void* u, int64_t nsteps) {
  hipError_t e = hipSuccess;
  void* bufs[2] = {u, ctx->work.ptr};
  int cur = 0;
  if (nsteps > 0 && (e = burgers::launch_btcs_window_reset(ctx, pl)) != hipSuccess) return e;
  for (int64_t s = 0; s < nsteps; ++s) {
    if ((e = burgers::launch_btcs_step(ctx, pl, bufs[cur], bufs[cur ^ 1], s)) != hipSuccess) return e;
    if (pl.newton) {
      burgers::NewtonPlan& np = *ctx->newton;
      const burgers::AdjTile* lt = np.long_tiles->as<burgers::AdjTile>();
      if ((pl.newton_whole && (e = burgers::launch_newton_init(ctx, np.tiles->as<burgers::AdjTile>(), np.n_tiles,
                                                               bufs[cur], bufs[cur ^ 1])) != hipSuccess) ||
          (e = burgers::launch_newton_init(ctx, lt, np.n_long_tiles, bufs[cur], bufs[cur ^ 1])) != hipSuccess)
        return e;
      int* flags = np.flags.as<int>();
      for (int it = 0; it < burgers::kNewtonIters; ++it) {
        const bool last = it == burgers::kNewtonIters - 1;
        for (const burgers::WgGroup& g : np.whole)
          if (pl.newton_whole && (e = burgers::launch_newton_whole(ctx, g, bufs[cur], bufs[cur ^ 1], last, flags)) != hipSuccess) return e;
        if (np.n_long_tiles == 0) continue;
        if ((e = burgers::launch_newton_assemble(ctx, lt, np.n_long_tiles, bufs[cur], bufs[cur ^ 1], np.NA.as<double>(),
                                                 np.NC.as<double>(), np.ND.as<double>(), flags)) != hipSuccess ||
            (e = burgers::launch_array_solve(ctx, np.solve, np.NA.as<double>(), np.NC.as<double>(), np.ND.as<double>(),
                                             np.NX.as<double>())) != hipSuccess ||
            (e = burgers::launch_newton_update(ctx, lt, np.n_long_tiles, bufs[cur], bufs[cur ^ 1], np.NX.as<double>(),
                                               last, flags)) != hipSuccess)
          return e;
      }
    }
    cur ^= 1;
  }
  if (cur) e = burgers::launch_copy_tiles(ctx, pl.copy->as<Tile>(), pl.n_copy, ctx->work.ptr, u);
  return e;
}

// Windows of several steps serve calls of three steps and more: they begin with a pass over the states for the
// bound that holds for the whole call, and keep 416 of 512 chunks against 224 of 256.  (2^24 rows, us per step with the
// copy of the state, by windows of one step / of several: 2 steps 79 / 107, 3 steps 83 / 78, 4 steps 66 / 63.)
constexpr int64_t kDeepLeast = 3, kDeepCall = int64_t{1} << 24;
bool takes_deep(const burgers::BtcsPlan& pl, int64_t nsteps) { return pl.n_deep > 0 && nsteps >= kDeepLeast; }

// nsteps implicit steps of one subset, the final state in u.
void btcs_tasks(burgers_ctx* ctx, int set, void* u, int64_t nsteps, std::vector<burgers::Task>& tasks) {
  const burgers::BtcsPlan* pl = ctx->btcs[set].get();
  auto on_chip = [&](const burgers::WgGroup& g, double scale, auto launch) {   // on-chip systems, in place
    const double rows = 0.75 * g.shape.lanes * g.shape.chunk * static_cast<double>(g.n);
    tasks.push_back({scale * chain_us(nsteps, g.shape.lanes <= 128 ? 1.6 : 2.5, rows, 9e5), 1, [=, &g]() -> hipError_t {
      for (int64_t done = 0; done < nsteps;) {
        const int k = static_cast<int>(std::min<int64_t>(nsteps - done, int64_t{1} << 30));
        const hipError_t e = launch(g, k);
        if (e != hipSuccess) return e;
        done += k;
      }
      return hipSuccess;
    }});
  };
  for (const burgers::WgGroup& g : pl->resident)
    on_chip(g, 1.0, [=](const burgers::WgGroup& q, int k) { return burgers::launch_btcs_resident(ctx, q, u, k); });
  for (const burgers::WgGroup& g : pl->cn_chip)
    on_chip(g, 1.5, [=](const burgers::WgGroup& q, int k) {
      return burgers::launch_cn_resident(ctx, pl->inst_half->as<InstDesc>(), q, u, k);
    });
  for (const burgers::WgGroup& g : pl->newton_chip)
    on_chip(g, 6.0, [=](const burgers::WgGroup& q, int k) {
      return burgers::launch_newton_resident(ctx, q, u, k, ctx->newton->flags.as<int>());
    });
  if (takes_deep(*pl, nsteps)) {
    const double rows = 8192.0 * static_cast<double>(pl->n_deep);
    tasks.push_back({chain_us(nsteps, 4.0, rows, 8e5), nsteps / 4, [=]() -> hipError_t {
      hipError_t e = hipSuccess;
      for (int64_t done = 0; done < nsteps && e == hipSuccess; done += kDeepCall)
        e = burgers::launch_btcs_deep(ctx, *pl, u, ctx->work.ptr, std::min(nsteps - done, kDeepCall));
      return e;
    }});
    // (mostly idle: but each of its launches waits for the other chains' workgroups to leave a CU, about 9 us)
    tasks.push_back({chain_us(nsteps, 18.0, 0.0, 1.0), 2 * nsteps, [=]() {
      return burgers::launch_btcs_beyond(ctx, *pl, u, ctx->work.ptr, nsteps);
    }});
  } else if (pl->n_copy > 0) {
    const double nodes = static_cast<double>(pl->n_copy) * burgers::explicit_tile_nodes(ctx->dtype);
    tasks.push_back({chain_us(nsteps, pl->newton ? 100.0 : 11.0, nodes, 3e5), 4 * nsteps,
                     [=]() { return enqueue_stepped(ctx, *pl, u, nsteps); }});
  }
}

// scheme -1: each instance's own scheme, explicit instances nsteps steps and BTCS ones nsteps_btcs.
hipError_t enqueue_all(burgers_ctx* ctx, int set, int scheme, void* u, int64_t nsteps, int64_t nsteps_btcs = -1) {
  if (nsteps_btcs < 0) nsteps_btcs = nsteps;
  const bool mixed = scheme < 0;
  const int64_t bsteps = mixed ? nsteps_btcs : nsteps;
  std::vector<burgers::Task> tasks;
  if (scheme == BURGERS_EXPLICIT || (mixed && !ctx->set_explicit.empty() && nsteps > 0))
    explicit_tasks(ctx, mixed ? kSetExplicit : set, u, nsteps, tasks);
  if (scheme == BURGERS_BTCS || (mixed && !ctx->set_btcs.empty() && bsteps > 0)) {
    const int bset = mixed ? kSetBtcs : set;
    const burgers::BtcsPlan& pl = *ctx->btcs[bset];
    // which instances the windows may step, and which the partition levels must: both of their chains follow
    if (takes_deep(pl, bsteps))
      if (const hipError_t e = burgers::launch_btcs_bound(ctx, pl, u, nullptr); e != hipSuccess) return e;
    btcs_tasks(ctx, bset, u, bsteps, tasks);
  }
  return burgers::run_tasks(ctx, tasks, ctx->plan.serial == 1);
}

burgers_status prepare(burgers_ctx* ctx, int set, int scheme) {
  burgers_status st;
  hipError_t e;
  const bool need_explicit = scheme == BURGERS_EXPLICIT || (scheme < 0 && !ctx->set_explicit.empty());
  const bool need_btcs = scheme == BURGERS_BTCS || (scheme < 0 && !ctx->set_btcs.empty());
  const int es = scheme < 0 ? kSetExplicit : set;
  const int bs = scheme < 0 ? kSetBtcs : set;
  if (need_explicit && (st = ensure_explicit(ctx, es)) != BURGERS_OK) return st;
  if (need_btcs && (st = ensure_btcs(ctx, bs)) != BURGERS_OK) return st;
  (void)e;
  return BURGERS_OK;
}

// Replay the launch sequence of (set, scheme, steps, u) from a captured graph, capturing it on first use.
hipError_t enqueue_graph(burgers_ctx* ctx, int set, int scheme, void* u, int64_t nsteps, int64_t nsteps_btcs) {
  const auto key = std::make_tuple(set, scheme, nsteps, nsteps_btcs, u);
  auto it = ctx->graph_cache.find(key);
  if (it == ctx->graph_cache.end()) {
    hipError_t e;
    if (!ctx->capture_stream &&
        (e = hipStreamCreateWithFlags(&ctx->capture_stream, hipStreamNonBlocking)) != hipSuccess)
      return e;
    hipStream_t user = ctx->stream;
    ctx->stream = ctx->capture_stream;
    if ((e = hipStreamBeginCapture(ctx->capture_stream, hipStreamCaptureModeThreadLocal)) != hipSuccess) {
      ctx->stream = user;
      return e;
    }
    hipError_t le = enqueue_all(ctx, set, scheme, u, nsteps, nsteps_btcs);
    hipGraph_t graph = nullptr;
    e = hipStreamEndCapture(ctx->capture_stream, &graph);
    ctx->stream = user;
    if (le != hipSuccess) { if (graph) (void)hipGraphDestroy(graph); return le; }
    if (e != hipSuccess) return e;
    hipGraphExec_t exec = nullptr;
    e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) return e;
    it = ctx->graph_cache.emplace(key, exec).first;
  }
  return hipGraphLaunch(it->second, ctx->stream);
}

// nsteps steps of `set` with `scheme` (-1: each instance's own; BTCS instances then take nsteps_btcs
// steps); the final state lands in u.
burgers_status advance(burgers_ctx* ctx, void* u, int64_t nsteps, int set, int scheme, int64_t nsteps_btcs = -1) {
  if (nsteps_btcs < 0) nsteps_btcs = nsteps;
  if (!ctx || !u || nsteps < 0) return BURGERS_E_INVALID;
  if (ctx->sticky != hipSuccess) return from_hip(ctx->sticky);
  if (nsteps == 0 && (scheme >= 0 || nsteps_btcs == 0)) return BURGERS_OK;
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return note(ctx, e);
  burgers_status st = prepare(ctx, set, scheme);
  if (st != BURGERS_OK) return st == BURGERS_E_UNSUPPORTED || st == BURGERS_E_INVALID ? st : note(ctx, hipErrorOutOfMemory);
  if (ctx->plan.use_graph == 1) e = enqueue_graph(ctx, set, scheme, u, nsteps, nsteps_btcs);
  else e = enqueue_all(ctx, set, scheme, u, nsteps, nsteps_btcs);
  if (e != hipSuccess) return note(ctx, e);
  return BURGERS_OK;
}


// Partition hierarchy for systems stored as unit-diagonal rows in binary64 arrays: root (instance, row
// offset, rows) triples; systems of up to 8192 rows are solved whole, longer ones reduced by chunk-
// partition levels whose reduced rows are appended after `rows_used` (updated).
hipError_t build_array_solve(burgers_ctx* ctx, const std::vector<std::tuple<int32_t, int64_t, int32_t>>& roots,
                             burgers::BtcsPlan& plan, int64_t& rows_used) {
  const int cap = burgers::btcs_wg_capacity();
  const int chunk = burgers::btcs_reduce_chunk();
  std::vector<std::vector<SysDesc>> red_sys(1), wg_sys(1);
  for (const auto& root : roots) {
    const int32_t i = std::get<0>(root);
    int64_t in_off = std::get<1>(root);
    int32_t R = std::get<2>(root);
    for (int level = 0;; ++level) {
      if (static_cast<int>(red_sys.size()) <= level) {
        red_sys.resize(level + 1);
        wg_sys.resize(level + 1);
      }
      if (R <= cap) {
        wg_sys[level].push_back(SysDesc{in_off, -1, R, burgers::btcs_chunks(R, 512), i, level});
        break;
      }
      const int32_t P = (R + chunk - 1) / chunk;
      const int64_t red = rows_used;
      rows_used += 2 * static_cast<int64_t>(P);
      red_sys[level].push_back(SysDesc{in_off, red, R, P, i, level});
      in_off = red;
      R = 2 * P;
    }
  }
  hipError_t e;
  plan.levels.resize(red_sys.size());
  for (size_t l = 0; l < red_sys.size(); ++l) {
    auto& lv = plan.levels[l];
    std::vector<ChunkBlock> blocks;
    for (size_t si = 0; si < red_sys[l].size(); ++si)
      for (int64_t c = 0; c < red_sys[l][si].chunks; c += burgers::kReduceBlock)
        blocks.push_back(ChunkBlock{static_cast<int32_t>(si), static_cast<int32_t>(c)});
    lv.sys = std::make_unique<DevBuf>();
    lv.blocks = std::make_unique<DevBuf>();
    lv.wg = std::make_unique<DevBuf>();
    if ((e = upload_on(ctx->stream, *lv.sys, red_sys[l])) != hipSuccess ||
        (e = upload_on(ctx->stream, *lv.blocks, blocks)) != hipSuccess ||
        (e = upload_on(ctx->stream, *lv.wg, wg_sys[l])) != hipSuccess)
      return e;
    lv.n_blocks = static_cast<int32_t>(blocks.size());
    lv.n_wg = static_cast<int32_t>(wg_sys[l].size());
    lv.wg_lanes = burgers::btcs_wg_lanes(wg_sys[l]);
    lv.wg_exact = burgers::btcs_wg_exact(wg_sys[l]);
  }
  return hipSuccess;
}

// Newton plan of the steps through HBM over the given instances (built once per context): systems of up to
// 8192 rows iterate in one fused kernel per iteration (grouped by width class; the automatic path holds them
// on chip instead), longer ones through the array path.
burgers_status ensure_newton(burgers_ctx* ctx, const std::vector<int32_t>& members) {
  if (ctx->newton) return BURGERS_OK;
  auto np = std::make_unique<burgers::NewtonPlan>();
  const int cap = burgers::btcs_wg_capacity();
  std::vector<burgers::AdjTile> tiles, long_tiles;
  std::vector<std::tuple<int32_t, int64_t, int32_t>> roots;
  std::map<int, std::vector<SysDesc>> groups;   // by lanes
  int64_t rows = 0;
  for (int32_t i : members) {
    const burgers_problem& p = ctx->probs[i];
    const int32_t n = static_cast<int32_t>(p.n);
    const int32_t R = p.bc == BURGERS_BC_PERIODIC ? n : n - 2;
    if (R <= cap) {
      for (int64_t s0 = 0; s0 < n; s0 += 256)
        tiles.push_back(burgers::AdjTile{ctx->offsets[i], 0, n, p.bc, i, static_cast<int32_t>(s0), 0, 0});
      // at most 8 rows a lane (the Newton rows need more registers than BTCS ones)
      int lanes = 128;
      while (lanes * 8 < R) lanes *= 2;
      groups[lanes].push_back(SysDesc{0, -1, R, burgers::btcs_chunks(R, lanes), i, 0});
      continue;
    }
    for (int64_t s0 = 0; s0 < n; s0 += 256)
      long_tiles.push_back(burgers::AdjTile{ctx->offsets[i], rows, n, p.bc, i, static_cast<int32_t>(s0), 0, 0});
    roots.emplace_back(i, rows, R);
    rows += R;
  }
  int64_t rows_used = rows;
  hipError_t e;
  np->tiles = std::make_unique<DevBuf>();
  np->long_tiles = std::make_unique<DevBuf>();
  if ((e = upload_on(ctx->stream, *np->tiles, tiles)) != hipSuccess ||
      (e = upload_on(ctx->stream, *np->long_tiles, long_tiles)) != hipSuccess)
    return from_hip(e);
  np->n_tiles = static_cast<int64_t>(tiles.size());
  np->n_long_tiles = static_cast<int64_t>(long_tiles.size());
  for (auto& kv : groups) {
    burgers::WgGroup g;
    g.shape = burgers::WidthClass{kv.first, 8};
    g.sys = std::make_unique<DevBuf>();
    g.n = static_cast<int32_t>(kv.second.size());
    if ((e = upload_on(ctx->stream, *g.sys, kv.second)) != hipSuccess) return from_hip(e);
    np->whole.push_back(std::move(g));
  }
  if ((e = build_array_solve(ctx, roots, np->solve, rows_used)) != hipSuccess) return from_hip(e);
  const size_t lb = static_cast<size_t>(rows_used) * sizeof(double);
  if ((e = np->NA.alloc(lb, ctx->stream)) != hipSuccess || (e = np->NC.alloc(lb, ctx->stream)) != hipSuccess ||
      (e = np->ND.alloc(lb, ctx->stream)) != hipSuccess || (e = np->NX.alloc(lb, ctx->stream)) != hipSuccess ||
      (e = np->flags.alloc(2 * sizeof(int), ctx->stream)) != hipSuccess ||
      (e = hipMemsetAsync(np->flags.ptr, 0, 2 * sizeof(int), ctx->stream)) != hipSuccess)
    return from_hip(e);
  ctx->newton = std::move(np);
  return BURGERS_OK;
}

// Launch lists and buffers of the adjoint: windows and dJ/dD slots of the explicit instances, the BTCS systems by the
// solver of their transposed ones (whole, windows and what takes those beyond the bound), and the array path's hierarchy
// over the systems of more than 16384 rows, which sit at the start of the adjoint arrays followed by their reduced rows.
burgers_status ensure_adjoint(burgers_ctx* ctx) {
  if (ctx->adjoint) return BURGERS_OK;
  auto ap = std::make_unique<burgers::AdjointPlan>();
  const int btcs_tile = burgers::adjoint_tile_nodes();
  std::vector<burgers::AdjTile> bt;
  std::vector<burgers::AdjWindow> ew;
  std::vector<int32_t> slot_begin(ctx->count + 1, 0);
  int32_t slot = 0;
  int64_t sys_rows = 0;
  std::vector<int64_t> sys_off(ctx->count, -1);
  for (int32_t i = 0; i < ctx->count; ++i) {
    const burgers_problem& p = ctx->probs[i];
    const int64_t R = p.bc == BURGERS_BC_PERIODIC ? p.n : p.n - 2;
    if (p.scheme == BURGERS_BTCS && !burgers::btcs_solved_whole(R)) {
      sys_off[i] = sys_rows;
      sys_rows += R;
    }
  }
  std::vector<std::tuple<int32_t, int64_t, int32_t>> roots;
  int64_t rows_used = sys_rows;
  std::vector<burgers::ChunkWin> deep;
  std::vector<int32_t> windowed, longs;
  std::map<std::pair<int, int>, std::vector<SysDesc>> wholes, beyond;
  for (int32_t i = 0; i < ctx->count; ++i) {
    const burgers_problem& p = ctx->probs[i];
    const int32_t n = static_cast<int32_t>(p.n);
    const int32_t R = static_cast<int32_t>(p.bc == BURGERS_BC_PERIODIC ? p.n : p.n - 2);
    slot_begin[i] = slot;
    if (p.scheme != BURGERS_BTCS) {
      // explicit: one slot per kAdjSumNodes nodes, and windows of equal shares of whole slots
      constexpr int32_t H = burgers::kAdjHalo, G = burgers::kAdjSumNodes, most = burgers::kAdjWinNodes - 2 * H;
      static_assert(most % G == 0 && H % G == 0, "windows keep whole slots");
      const int32_t shares = (n + most - 1) / most, kept = ((n + shares - 1) / shares + G - 1) / G * G;
      for (int32_t lo = 0; lo < n; lo += kept) {
        const int32_t hi = std::min(n, lo + kept);
        if (p.bc == BURGERS_BC_PERIODIC) {
          ew.push_back(burgers::AdjWindow{i, ((lo - H) % n + n) % n, (hi - lo) + 2 * H, H, hi - lo, slot + lo / G});
        } else {
          const int32_t first = std::max(0, lo - H), end = std::min(n, hi + H);
          ew.push_back(burgers::AdjWindow{i, first, end - first, lo - first, hi - lo, slot + lo / G});
        }
      }
      slot += (n + G - 1) / G;
      continue;
    }
    const bool windows = R > burgers::btcs_wg_capacity();
    if (windows) {                             // one slot per chunk of 16 rows
      burgers::btcs_deep_windows(i, R, p.bc == BURGERS_BC_PERIODIC, deep, true);
      windowed.push_back(i);
    }
    if (burgers::btcs_solved_whole(R)) {       // one slot per lane
      const burgers::WidthClass w = burgers::btcs_width_class(R, burgers::kResidentThreadsDefault);
      const int32_t P = burgers::btcs_chunks(R, w.lanes);
      (windows ? beyond : wholes)[{w.lanes, w.chunk}].push_back(SysDesc{0, -1, R, P, i, 0});
      slot += P;                               // (1024 lanes: as many as a window's chunks or more)
      continue;
    }
    const int32_t tile_slot = slot + (R + 15) / 16;
    slot = tile_slot;
    longs.push_back(i);
    for (int64_t s = 0; s < n; s += btcs_tile)
      bt.push_back(burgers::AdjTile{ctx->offsets[i], sys_off[i], n, p.bc, i, static_cast<int32_t>(s), slot++, 0});
    roots.emplace_back(i, sys_off[i], R);
  }
  slot_begin[ctx->count] = slot;
  hipError_t e;
  // windows without a Dirichlet node or part of a slot first (their launch compiles neither case)
  auto inner = [&](const burgers::AdjWindow& w) {
    const burgers_problem& p = ctx->probs[w.inst];
    return w.count % burgers::kAdjSumNodes == 0 &&
           (p.bc == BURGERS_BC_PERIODIC || (w.first > 0 && w.first + w.width < p.n));
  };
  ap->n_exp_inner = std::stable_partition(ew.begin(), ew.end(), inner) - ew.begin();
  ap->exp_wins = std::make_unique<DevBuf>();
  ap->btcs_tiles = std::make_unique<DevBuf>();
  ap->slot_begin = std::make_unique<DevBuf>();
  if ((e = upload_on(ctx->stream, *ap->exp_wins, ew)) != hipSuccess || (e = upload_on(ctx->stream, *ap->btcs_tiles, bt)) != hipSuccess ||
      (e = upload_on(ctx->stream, *ap->slot_begin, slot_begin)) != hipSuccess)
    return from_hip(e);
  ap->n_exp_wins = static_cast<int64_t>(ew.size());
  ap->n_btcs_tiles = static_cast<int64_t>(bt.size());
  ap->n_slots = slot;
  auto upload_whole = [&](std::map<std::pair<int, int>, std::vector<SysDesc>>& groups,
                          std::vector<burgers::WgGroup>& out) -> hipError_t {
    for (auto& kv : groups) {
      burgers::WgGroup g;
      g.shape = burgers::WidthClass{kv.first.first, kv.first.second};
      g.sys = std::make_unique<DevBuf>();
      g.n = static_cast<int32_t>(kv.second.size());
      const hipError_t err = upload_on(ctx->stream, *g.sys, kv.second);
      if (err != hipSuccess) return err;
      out.push_back(std::move(g));
    }
    return hipSuccess;
  };
  if ((e = upload_whole(wholes, ap->whole)) != hipSuccess || (e = upload_whole(beyond, ap->whole_beyond)) != hipSuccess)
    return from_hip(e);
  ap->long_copy = std::make_unique<DevBuf>();
  const auto lc = stream_tiles(ctx, longs);
  if ((e = upload_on(ctx->stream, *ap->long_copy, lc)) != hipSuccess) return from_hip(e);
  ap->n_long_copy = static_cast<int64_t>(lc.size());
  if (!deep.empty()) {
    burgers::BtcsPlan& w = ap->windows;
    const int64_t words = burgers::deep_words(ctx->count);
    w.transposed = true;
    w.deep = std::make_unique<DevBuf>();
    w.deep_inst = std::make_unique<DevBuf>();
    if ((e = upload_on(ctx->stream, *w.deep, deep)) != hipSuccess ||
        (e = upload_on(ctx->stream, *w.deep_inst, windowed)) != hipSuccess ||
        (e = w.deep_words.alloc(static_cast<size_t>(words) * sizeof(int), ctx->stream)) != hipSuccess ||
        (e = w.win_flags.alloc(static_cast<size_t>(burgers::win_flags_words(ctx->count)) * sizeof(int), ctx->stream)) !=
            hipSuccess ||
        (e = burgers::launch_clear_ints(ctx, w.deep_words.as<int>(), words)) != hipSuccess)
      return from_hip(e);
    w.n_deep = static_cast<int64_t>(deep.size());
    w.n_deep_inst = static_cast<int64_t>(windowed.size());
  }
  if ((e = build_array_solve(ctx, roots, ap->solve, rows_used)) != hipSuccess) return from_hip(e);
  const size_t lb = static_cast<size_t>(rows_used) * sizeof(double);
  if ((e = ap->LA.alloc(lb, ctx->stream)) != hipSuccess || (e = ap->LC.alloc(lb, ctx->stream)) != hipSuccess ||
      (e = ap->LD.alloc(lb, ctx->stream)) != hipSuccess || (e = ap->LX.alloc(lb, ctx->stream)) != hipSuccess ||
      (e = ap->gslot.alloc(static_cast<size_t>(std::max<int64_t>(slot, 1)) * sizeof(double), ctx->stream)) != hipSuccess)
    return from_hip(e);
  ctx->adjoint = std::move(ap);
  return BURGERS_OK;
}

hipError_t grow(DevBuf& b, size_t bytes, hipStream_t stream) {
  if (b.bytes >= bytes && b.ptr) return hipSuccess;
  return b.alloc(bytes, stream);
}

// One adjoint step of the BTCS instances of more than 16384 rows that are beyond their windows' bound: lam_out from
// lam_in at the forward pair (y = u^k, x = u^{k+1}).
hipError_t enqueue_adjoint_step(burgers_ctx* ctx, const double* y, const double* x, const double* lam_in,
                                double* lam_out, const int* only) {
  burgers::AdjointPlan& ap = *ctx->adjoint;
  hipError_t e;
  if ((e = burgers::launch_adj_btcs_assemble(ctx, ap.btcs_tiles->as<burgers::AdjTile>(), ap.n_btcs_tiles, y,
                                             lam_in, ap.LA.as<double>(), ap.LC.as<double>(),
                                             ap.LD.as<double>(), only)) != hipSuccess)
    return e;
  if ((e = burgers::launch_array_solve(ctx, ap.solve, ap.LA.as<double>(), ap.LC.as<double>(), ap.LD.as<double>(),
                                       ap.LX.as<double>(), only)) != hipSuccess)
    return e;
  return burgers::launch_adj_btcs_finish(ctx, ap.btcs_tiles->as<burgers::AdjTile>(), ap.n_btcs_tiles, y, x,
                                         ap.LX.as<double>(), lam_out, ap.gslot.as<double>(), only);
}

// A context for `count` problems on the current device: validated, laid out, its workspace allocated
// (or carved from the installed arena).  *out is set only on success.
burgers_status new_context(const burgers_problem* problems, int64_t count, burgers_dtype dtype, void* hip_stream,
                           burgers_ctx** out) {
  if (!problems || count < 1 || (dtype != BURGERS_F32 && dtype != BURGERS_F64))
    return BURGERS_E_INVALID;
  for (int64_t i = 0; i < count; ++i)
    if (!valid_problem(problems[i])) return BURGERS_E_INVALID;
  if (count > INT32_MAX) return BURGERS_E_INVALID;
  burgers_ctx* ctx = new (std::nothrow) burgers_ctx();
  if (!ctx) return BURGERS_E_NOMEM;
  hipError_t e = hipGetDevice(&ctx->device);
  if (e != hipSuccess) { delete ctx; return BURGERS_E_DEVICE; }
  ctx->stream = static_cast<hipStream_t>(hip_stream);
  ctx->dtype = dtype;
  ctx->word = dtype == BURGERS_F64 ? 8 : 4;
  ctx->count = count;
  ctx->probs.assign(problems, problems + count);
  ctx->offsets.resize(count + 1);
  ctx->offsets[0] = 0;
  for (int64_t i = 0; i < count; ++i) {
    const int64_t padded = (problems[i].n + BURGERS_ALIGN - 1) / BURGERS_ALIGN * BURGERS_ALIGN;
    ctx->offsets[i + 1] = ctx->offsets[i] + padded;
  }
  ctx->total = ctx->offsets[count];
  ctx->inst_host.resize(count);
  for (int64_t i = 0; i < count; ++i) {
    const burgers_problem& p = problems[i];
    ctx->inst_host[i] = burgers::inst_desc(p, ctx->offsets[i]);
    ctx->set_all.push_back(static_cast<int32_t>(i));
    (p.scheme == BURGERS_EXPLICIT || p.scheme == BURGERS_RK4 ? ctx->set_explicit : ctx->set_btcs)
        .push_back(static_cast<int32_t>(i));
  }
  burgers_status st = BURGERS_OK;
  if ((e = upload_on(ctx->stream, ctx->inst, ctx->inst_host)) != hipSuccess) st = from_hip(e);
  if (st == BURGERS_OK && (e = ctx->work.alloc(static_cast<size_t>(ctx->total) * ctx->word, ctx->stream)) != hipSuccess)
    st = from_hip(e);
  if (st == BURGERS_OK) {
    ctx->level_capacity = level_rows_needed(ctx);
    const size_t lb = static_cast<size_t>(ctx->level_capacity) * sizeof(double);   // binary64 solve
    if ((e = ctx->level_a.alloc(lb, ctx->stream)) != hipSuccess || (e = ctx->level_c.alloc(lb, ctx->stream)) != hipSuccess ||
        (e = ctx->level_d.alloc(lb, ctx->stream)) != hipSuccess || (e = ctx->level_x.alloc(lb, ctx->stream)) != hipSuccess)
      st = from_hip(e);
  }
  if (st != BURGERS_OK) {
    delete ctx;
    return st;
  }
  *out = ctx;
  return BURGERS_OK;
}

// ---- Static scratch: the workspace of burgers_run_static -------------------------------------------
// A file-scope device array, one copy per GPU the library runs on, held until the process ends.  Host
// code never passes the array's name to a kernel or a copy (on the host it is only a stand-in for the
// symbol): its device address is looked up once per device with that device current, and every use
// goes through that address.
__device__ __align__(256) unsigned char scratch[BURGERS_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
void* scratch_ptr[kMaxDevices] = {};

// Beside each device's scratch, one set of side streams for the calls on it, lent to one call at a time while it
// enqueues.
std::mutex static_sides_mutex[kMaxDevices];
burgers::SideStreams static_sides[kMaxDevices];

// Device address of the current device's scratch array.
hipError_t scratch_address(int device, void** out) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_ptr[device]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    scratch_ptr[device] = p;
  }
  *out = scratch_ptr[device];
  return hipSuccess;
}

// Installs an arena on the calling thread for the lifetime of the guard.
struct ArenaGuard {
  explicit ArenaGuard(burgers::Arena* a) { burgers::tl_arena = a; }
  ~ArenaGuard() { burgers::tl_arena = nullptr; }
};

}  // namespace

extern "C" {

int32_t burgers_abi_version(void) { return BURGERS_ABI_VERSION; }

const char* burgers_status_string(burgers_status s) {
  switch (s) {
    case BURGERS_OK: return "ok";
    case BURGERS_E_INVALID: return "invalid argument";
    case BURGERS_E_UNSUPPORTED: return "unsupported request";
    case BURGERS_E_NOMEM: return "out of device memory";
    case BURGERS_E_DEVICE: return "device error";
    case BURGERS_E_NONFINITE: return "non-finite value";
    case BURGERS_E_BUDGET: return "memory budget exceeded";
    case BURGERS_E_NOT_CONVERGED: return "Newton step not converged or Jacobian not diagonally dominant";
    case BURGERS_E_BOUND: return "truncated-window step outside its accuracy bound";
  }
  return "unknown status";
}

double burgers_cfl_dt(const burgers_problem* p, double umax, double sigma) {
  if (!p || p->n < 3 || !(p->length > 0) || !is_finite(p->length) || !(p->nu >= 0) ||
      !(sigma > 0) || !(umax >= 0) || (p->bc != BURGERS_BC_PERIODIC && p->bc != BURGERS_BC_DIRICHLET))
    return NAN;
  const double dx = grid_dx(*p);
  double lim = INFINITY;
  if (umax > 0) lim = std::min(lim, dx / umax);
  if (p->nu > 0) lim = std::min(lim, dx * dx / (2.0 * p->nu));
  return sigma * lim;
}

burgers_status burgers_ratios(const burgers_problem* p, double* r, double* D) {
  if (!p || !r || !D || !valid_problem(*p)) return BURGERS_E_INVALID;
  const double dx = grid_dx(*p);
  *r = p->dt / dx;
  *D = p->nu * p->dt / (dx * dx);
  return BURGERS_OK;
}

burgers_status burgers_create(const burgers_problem* problems, int64_t count, burgers_dtype dtype,
                              void* hip_stream, burgers_ctx** out) {
  if (!out) return BURGERS_E_INVALID;
  *out = nullptr;
  burgers_ctx* ctx = nullptr;
  burgers_status st = new_context(problems, count, dtype, hip_stream, &ctx);
  if (st == BURGERS_OK) *out = ctx;
  return st;
}

void burgers_destroy(burgers_ctx* ctx) {
  if (!ctx) return;
  (void)hipSetDevice(ctx->device);
  (void)hipStreamSynchronize(ctx->stream);
  for (auto& kv : ctx->graph_cache) (void)hipGraphExecDestroy(kv.second);
  if (ctx->capture_stream) (void)hipStreamDestroy(ctx->capture_stream);
  ctx->sides.release();
  delete ctx;
}

burgers_status burgers_offsets(const burgers_ctx* ctx, int64_t* out) {
  if (!ctx || !out) return BURGERS_E_INVALID;
  std::memcpy(out, ctx->offsets.data(), sizeof(int64_t) * ctx->offsets.size());
  return BURGERS_OK;
}

int64_t burgers_state_elems(const burgers_ctx* ctx) { return ctx ? ctx->total : -1; }

burgers_status burgers_step_explicit(burgers_ctx* ctx, void* u, int64_t nsteps) {
  return advance(ctx, u, nsteps, kSetAll, BURGERS_EXPLICIT);
}

burgers_status burgers_step_btcs(burgers_ctx* ctx, void* u, int64_t nsteps) {
  return advance(ctx, u, nsteps, kSetAll, BURGERS_BTCS);
}

burgers_status burgers_run(burgers_ctx* ctx, void* u, int64_t nsteps) {
  return advance(ctx, u, nsteps, kSetAll, -1);
}

burgers_status burgers_run_mixed(burgers_ctx* ctx, void* u, int64_t explicit_steps, int64_t btcs_steps) {
  if (btcs_steps < 0) return BURGERS_E_INVALID;
  return advance(ctx, u, explicit_steps, kSetAll, -1, btcs_steps);
}

burgers_status burgers_run_static(const burgers_problem* problems, int64_t count, burgers_dtype dtype,
                                  void* hip_stream, void* u, int64_t nsteps) {
  if (!problems || !u || nsteps < 0 || count < 1 || count > INT32_MAX ||
      (dtype != BURGERS_F32 && dtype != BURGERS_F64))
    return BURGERS_E_INVALID;
  for (int64_t i = 0; i < count; ++i)
    if (!valid_problem(problems[i])) return BURGERS_E_INVALID;
  for (int64_t i = 0; i < count; ++i)
    if (problems[i].scheme == BURGERS_NEWTON) return BURGERS_E_UNSUPPORTED;
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return BURGERS_E_DEVICE;
  void* base = nullptr;
  if ((e = scratch_address(device, &base)) != hipSuccess) return BURGERS_E_DEVICE;
  burgers::Arena arena{static_cast<char*>(base), static_cast<size_t>(BURGERS_STATIC_SCRATCH_BYTES), 0};
  burgers_status st;
  {
    ArenaGuard guard(&arena);
    burgers_ctx* ctx = nullptr;
    st = new_context(problems, count, dtype, hip_stream, &ctx);
    if (st == BURGERS_OK) {
      std::unique_lock<std::mutex> lent(static_sides_mutex[device], std::try_to_lock);
      if (lent) std::swap(ctx->sides, static_sides[device]);
      else ctx->plan.serial = 1;                   // (another thread's call has them)
      st = advance(ctx, u, nsteps, kSetAll, -1);   // plan tables carved too; eager launches
      if (st == BURGERS_OK && ctx->sticky != hipSuccess) st = from_hip(ctx->sticky);
      if (lent) std::swap(ctx->sides, static_sides[device]);
      delete ctx;                                  // host side only: carved buffers free nothing
    }
  }
  return st == BURGERS_E_NOMEM ? BURGERS_E_BUDGET : st;
}

burgers_status burgers_autotune(burgers_ctx* ctx, const void* u, int64_t explicit_steps, int64_t btcs_steps,
                                burgers_plan* best, double* best_ms) {
  if (!ctx || !u || explicit_steps < 0 || btcs_steps < 0 || explicit_steps + btcs_steps == 0)
    return BURGERS_E_INVALID;
  if (ctx->sticky != hipSuccess) return from_hip(ctx->sticky);
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return note(ctx, e);
  const bool has_exp = !ctx->set_explicit.empty() && explicit_steps > 0;
  const bool has_btcs = !ctx->set_btcs.empty() && btcs_steps > 0;
  bool long_exp = false, long_btcs = false;
  for (int32_t i : ctx->set_explicit)
    if (ctx->probs[i].n > burgers::explicit_block_capacity()) long_exp = true;
  for (int32_t i : ctx->set_btcs) {
    const burgers_problem& p = ctx->probs[i];
    if (!burgers::btcs_solved_whole(p.bc == BURGERS_BC_PERIODIC ? p.n : p.n - 2)) long_btcs = true;
  }
  // One knob at a time (coordinate descent from the current plan): the explicit path and window depth,
  // the lanes per 8192-row BTCS system, the long-system BTCS solver, concurrent launch groups, graph
  // replay.  Each candidate runs twice on a scratch copy of u (the first run builds its plans and
  // graphs) and the second run is timed.
  using Setter = void (*)(burgers_plan&, int);
  struct Knob {
    std::vector<int> values;
    Setter set;
  };
  std::vector<Knob> knobs;
  if (has_exp) {
    std::vector<int> v = {0};                                     // automatic (whole instances, windows)
    if (long_exp) v = {4, 8, 16, 32, 64, 128, 256};               // window depth (steps per HBM pass)
    v.push_back(-1);                                              // one step per HBM pass
    knobs.push_back({v, [](burgers_plan& p, int x) {
                       p.explicit_path = x < 0 ? 1 : 0;
                       p.tblock_depth = x > 0 ? x : 0;
                     }});
  }
  if (has_btcs) {
    knobs.push_back({{512, 1024}, [](burgers_plan& p, int x) { p.btcs_block = x; }});
    if (long_btcs) knobs.push_back({{0, 2, 1}, [](burgers_plan& p, int x) { p.btcs_long = x; }});
  }
  knobs.push_back({{0, 1}, [](burgers_plan& p, int x) { p.serial = x; }});
  knobs.push_back({{0, 1}, [](burgers_plan& p, int x) { p.use_graph = x; }});
  const burgers_plan base = ctx->plan;
  DevBuf scratch;
  if ((e = scratch.alloc(static_cast<size_t>(ctx->total) * ctx->word, ctx->stream)) != hipSuccess) return from_hip(e);
  hipEvent_t t0, t1;
  if ((e = hipEventCreate(&t0)) != hipSuccess) return from_hip(e);
  if ((e = hipEventCreate(&t1)) != hipSuccess) { (void)hipEventDestroy(t0); return from_hip(e); }
  const size_t bytes = static_cast<size_t>(ctx->total) * ctx->word;
  burgers_status st = BURGERS_OK;
  // time one plan; +inf when it cannot serve the batch
  auto time_plan = [&](const burgers_plan& p, double& ms_out) -> bool {
    ms_out = INFINITY;
    if ((st = burgers_set_plan(ctx, &p)) != BURGERS_OK) return false;
    float ms = 0.0f;
    for (int rep = 0; rep < 2; ++rep) {
      if ((e = hipMemcpyAsync(scratch.ptr, u, bytes, hipMemcpyDeviceToDevice, ctx->stream)) != hipSuccess) return false;
      if ((e = hipEventRecord(t0, ctx->stream)) != hipSuccess) return false;
      st = advance(ctx, scratch.ptr, explicit_steps, kSetAll, -1, btcs_steps);
      if (st == BURGERS_E_UNSUPPORTED) {
        st = BURGERS_OK;
        return true;
      }
      if (st != BURGERS_OK) return false;
      if ((e = hipEventRecord(t1, ctx->stream)) != hipSuccess || (e = hipEventSynchronize(t1)) != hipSuccess) return false;
      if ((e = hipEventElapsedTime(&ms, t0, t1)) != hipSuccess) return false;
    }
    ms_out = ms;
    return true;
  };
  burgers_plan best_p = base;
  best_p.explicit_path = 0;
  best_p.btcs_path = 0;
  double best_t = INFINITY;
  bool ok = time_plan(best_p, best_t);
  for (size_t k = 0; ok && k < knobs.size(); ++k) {
    burgers_plan knob_best = best_p;
    for (int v : knobs[k].values) {
      burgers_plan p = best_p;
      knobs[k].set(p, v);
      double t;
      if (!(ok = time_plan(p, t))) break;
      if (t < best_t) {
        best_t = t;
        knob_best = p;
      }
    }
    best_p = knob_best;
  }
  (void)hipEventDestroy(t0);
  (void)hipEventDestroy(t1);
  if (e != hipSuccess) {
    (void)burgers_set_plan(ctx, &base);
    return note(ctx, e);
  }
  if (st != BURGERS_OK || !std::isfinite(best_t)) {
    (void)burgers_set_plan(ctx, &base);
    return st != BURGERS_OK ? st : BURGERS_E_UNSUPPORTED;
  }
  (void)burgers_set_plan(ctx, &best_p);
  if (best) *best = best_p;
  if (best_ms) *best_ms = best_t;
  return BURGERS_OK;
}

burgers_status burgers_adjoint(burgers_ctx* ctx, const void* u0, const void* lambda_T, int64_t nsteps,
                               int64_t ckpt_every, void* grad_u0, void* grad_nu) {
  if (!ctx || !u0 || !lambda_T || !grad_u0 || !grad_nu || nsteps < 0 || ckpt_every < 1)
    return BURGERS_E_INVALID;
  if (ctx->dtype != BURGERS_F64) return BURGERS_E_UNSUPPORTED;
  for (const auto& p : ctx->probs)   // adjoint of forward Euler and BTCS only
    if (p.scheme != BURGERS_EXPLICIT && p.scheme != BURGERS_BTCS) return BURGERS_E_UNSUPPORTED;
  if (ctx->sticky != hipSuccess) return from_hip(ctx->sticky);
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return note(ctx, e);
  burgers_status st = prepare(ctx, kSetAll, -1);
  if (st != BURGERS_OK) return st;
  if (!ctx->set_btcs.empty() && (st = ensure_btcs(ctx, kSetBtcsHbm)) != BURGERS_OK) return st;
  if ((st = ensure_adjoint(ctx)) != BURGERS_OK) return st;
  burgers::AdjointPlan& ap = *ctx->adjoint;
  const size_t state_bytes = static_cast<size_t>(ctx->total) * sizeof(double);
  const int64_t K = std::min<int64_t>(ckpt_every, std::max<int64_t>(nsteps, 1));
  const int64_t ncp = (nsteps + K - 1) / K;   // checkpoints at steps 0, K, 2K, ...
  if ((e = grow(ap.ckpt, state_bytes * static_cast<size_t>(std::max<int64_t>(ncp, 1)), ctx->stream)) != hipSuccess ||
      (e = grow(ap.seg, state_bytes * static_cast<size_t>(K), ctx->stream)) != hipSuccess ||
      (ncp > 1 && (e = grow(ap.seg2, state_bytes * static_cast<size_t>(K), ctx->stream)) != hipSuccess) ||
      (e = grow(ap.lam0, state_bytes, ctx->stream)) != hipSuccess || (e = grow(ap.lam1, state_bytes, ctx->stream)) != hipSuccess)
    return from_hip(e);
  auto state = [&](DevBuf& b, int64_t k) { return static_cast<char*>(b.ptr) + static_cast<size_t>(k) * state_bytes; };
  const hipMemcpyKind d2d = hipMemcpyDeviceToDevice;
  // forward sweep, keeping checkpoints
  if (ncp > 0 && (e = hipMemcpyAsync(state(ap.ckpt, 0), u0, state_bytes, d2d, ctx->stream)) != hipSuccess)
    return note(ctx, e);
  for (int64_t c = 1; c < ncp; ++c) {
    if ((e = hipMemcpyAsync(state(ap.ckpt, c), state(ap.ckpt, c - 1), state_bytes, d2d, ctx->stream)) != hipSuccess ||
        (e = enqueue_all(ctx, kSetAll, -1, state(ap.ckpt, c), K)) != hipSuccess)
      return note(ctx, e);
  }
  // reverse sweep: recompute each segment's states one step at a time, then step the adjoint back
  // lam of the BTCS instances (per step) and of the explicit ones (per run of steps) ping-pong between the
  // same two buffers, each set in its own nodes
  double* lam = ap.lam0.as<double>();
  double* lam_next = ap.lam1.as<double>();
  double* lam_e = lam;
  double* lam_e_next = lam_next;
  if ((e = hipMemcpyAsync(lam, lambda_T, state_bytes, d2d, ctx->stream)) != hipSuccess ||
      (e = burgers::launch_fill(ctx, ap.gslot.as<double>(), ap.n_slots, 0.0)) != hipSuccess ||
      (ap.windows.n_deep > 0 && (e = burgers::launch_btcs_bound(ctx, ap.windows, u0, nullptr)) != hipSuccess))
    return note(ctx, e);
  const int* code = ap.windows.n_deep > 0 ? burgers::deep_code(ap.windows.deep_words.as<int>(), ctx->count) : nullptr;
  const int* beyond = ap.windows.n_deep > 0 ? burgers::win_flag_slot(ap.windows.win_flags.as<int>(), ctx->count, 0) : nullptr;
  // State k of segment c: the checkpoint for k = 0, else slot k - 1 of the segment's buffer.
  auto at = [&](int64_t c, DevBuf& seg, int64_t k) { return k == 0 ? state(ap.ckpt, c) : state(seg, k - 1); };
  // A segment's states are recomputed out of place.  Instances that the forward sweep keeps on chip are
  // kept on chip here too, by kernels that store the state after every step, or for the explicit ones every
  // kAdjGroup-th (one launch per segment, or per `depth` steps for the explicit windows, whose halos cover that
  // many steps): each is written once and nothing is read back.  The others step one launch at a time from state k - 1 straight into
  // state k: the streaming kernel for explicit instances, the per-step solves for BTCS ones.
  const burgers::ExplicitPlan* ep = ctx->set_explicit.empty() ? nullptr : ctx->explicit_plans[kSetExplicit].get();
  const bool exp_rec = ep && ep->path != 1;
  const burgers::BtcsPlan* bres = ctx->set_btcs.empty() ? nullptr : ctx->btcs[kSetBtcs].get();
  const bool btcs_rec = bres && bres->n_copy == 0 && !bres->resident.empty();
  const burgers::BtcsPlan* bp = ctx->set_btcs.empty() || btcs_rec ? nullptr : ctx->btcs[kSetBtcsHbm].get();
  const int64_t stride = ctx->total;
  auto recompute = [&](int64_t c, DevBuf& seg) -> hipError_t {
    const int64_t len = std::min(K, nsteps - c * K);
    hipError_t err = hipSuccess;
    for (int64_t k0 = 0; exp_rec && k0 < len && err == hipSuccess; k0 += ep->depth) {
      const int k = static_cast<int>(std::min<int64_t>(ep->depth, len - k0));
      for (const auto& wc : ep->whole_classes)
        if (err == hipSuccess)
          err = burgers::launch_explicit_record(ctx, ep->whole->as<BlockTile>() + wc.offset, wc.n_fe, at(c, seg, k0),
                                                at(c, seg, k0 + 1), stride, k, static_cast<int>(k0), wc.lanes);
      if (err == hipSuccess)
        err = burgers::launch_explicit_record(ctx, ep->win->as<BlockTile>(), ep->n_win, at(c, seg, k0),
                                              at(c, seg, k0 + 1), stride, k, static_cast<int>(k0));
    }
    if (btcs_rec)
      for (const burgers::WgGroup& g : bres->resident)
        if (err == hipSuccess)
          err = burgers::launch_btcs_record(ctx, g, at(c, seg, 0), at(c, seg, 1), stride, static_cast<int>(len));
    const bool exp_step = ep && !exp_rec;
    if (err == hipSuccess && bp) err = burgers::launch_btcs_window_reset(ctx, *bp);
    for (int64_t k = 1; (exp_step || bp) && k <= len && err == hipSuccess; ++k) {
      if (exp_step)
        err = burgers::launch_explicit_stream(ctx, ep->stream->as<Tile>(), ep->n_stream, at(c, seg, k - 1),
                                              at(c, seg, k));
      if (err == hipSuccess && bp) err = burgers::launch_btcs_step(ctx, *bp, at(c, seg, k - 1), at(c, seg, k), k - 1);
    }
    return err;
  };
  // Segment c's reverse steps run beside the recompute of segment c - 1 into the other segment buffer (which uses
  // none of the reverse steps' buffers), and beside each other by class, as chains of one set of tasks: the
  // recompute begins after the previous segment's reverse steps (which read the buffer it overwrites), and the next
  // segment's reverse steps after both.
  DevBuf* segs[2] = {&ap.seg, &ap.seg2};
  if (ncp > 0 && (e = recompute(ncp - 1, ap.seg)) != hipSuccess) return note(ctx, e);
  for (int64_t c = ncp - 1; c >= 0; --c) {
    const int64_t len = std::min(K, nsteps - c * K);
    DevBuf& cur = *segs[(ncp - 1 - c) & 1];
    const double* y0 = reinterpret_cast<const double*>(at(c, cur, 0));
    const double* y1 = reinterpret_cast<const double*>(at(c, cur, 1));
    double* gslot = ap.gslot.as<double>();
    std::vector<burgers::Task> tasks;
    // (a state's share of the time: the recompute and the reverse steps are of one order, and both long)
    const double us = static_cast<double>(len) * (2.0 + static_cast<double>(ctx->total) / 1e6);
    if (c > 0) tasks.push_back({us, 2, [&, c]() { return recompute(c - 1, *segs[(ncp - c) & 1]); }});
    // explicit instances: equal runs of up to kAdjRun reverse steps per launch, lam on chip (out of place)
    const int64_t runs = (len + burgers::kAdjRun - 1) / burgers::kAdjRun;
    const int64_t run = ((len + runs - 1) / runs + burgers::kAdjGroup - 1) / burgers::kAdjGroup * burgers::kAdjGroup;
    if (ap.n_exp_wins > 0)
      tasks.push_back({us, runs, [&]() -> hipError_t {
        for (int64_t hi = len; hi > 0;) {
          const int64_t lo = (hi - 1) / run * run;
          const hipError_t err = burgers::launch_adj_explicit(
              ctx, ap.exp_wins->as<burgers::AdjWindow>(), ap.n_exp_wins, ap.n_exp_inner, y0, y1, ctx->total,
              static_cast<int>(lo), static_cast<int>(hi), lam_e, lam_e_next, gslot);
          if (err != hipSuccess) return err;
          std::swap(lam_e, lam_e_next);
          hi = lo;
        }
        return hipSuccess;
      }});
    // BTCS instances, from lam to lam_next: the segment's steps in one launch where the system is solved whole, in
    // launches of several steps on windows, and one step at a time on the array path
    for (const burgers::WgGroup& g : ap.whole)
      tasks.push_back({us, 1, [&]() {
        return burgers::launch_adj_btcs_whole(ctx, g, ap.slot_begin->as<int32_t>(), y0, y1, ctx->total, 0,
                                              static_cast<int>(len), lam, lam_next, gslot);
      }});
    if (ap.windows.n_deep > 0)
      tasks.push_back({us, len / 3 + 1, [&]() {
        return burgers::launch_adj_btcs_deep(ctx, ap.windows, ap.slot_begin->as<int32_t>(), y0, y1, ctx->total,
                                             static_cast<int>(len), lam, lam_next, gslot);
      }});
    for (const burgers::WgGroup& g : ap.whole_beyond)   // (mostly idle)
      tasks.push_back({5.0, 1, [&]() {
        return burgers::launch_adj_btcs_whole(ctx, g, ap.slot_begin->as<int32_t>(), y0, y1, ctx->total, 0,
                                              static_cast<int>(len), lam, lam_next, gslot, code);
      }});
    if (ap.n_btcs_tiles > 0)
      tasks.push_back({us + 20.0 * static_cast<double>(len), 6 * len, [&]() -> hipError_t {
        double* in = lam;
        double* out = lam_next;
        for (int64_t k = len - 1; k >= 0; --k) {
          const hipError_t err = enqueue_adjoint_step(ctx, reinterpret_cast<const double*>(at(c, cur, k)),
                                                      reinterpret_cast<const double*>(at(c, cur, k + 1)), in, out, beyond);
          if (err != hipSuccess) return err;
          std::swap(in, out);
        }
        if (in == lam_next) return hipSuccess;
        return burgers::launch_copy_tiles(ctx, ap.long_copy->as<Tile>(), ap.n_long_copy, in, lam_next, beyond);
      }});
    if ((e = burgers::run_tasks(ctx, tasks, ctx->plan.serial == 1)) != hipSuccess) return note(ctx, e);
    if (!ctx->set_btcs.empty()) std::swap(lam, lam_next);
  }
  const bool split = lam_e != lam && !ctx->set_explicit.empty() && !ctx->set_btcs.empty();
  if ((e = ensure_copy(ctx, split ? kSetExplicit : kSetAll)) != hipSuccess ||
      (split && (e = ensure_copy(ctx, kSetBtcs)) != hipSuccess))
    return from_hip(e);
  auto& first_tiles = ctx->copy_tiles[split ? kSetExplicit : kSetAll];
  if ((e = burgers::launch_copy_tiles(ctx, first_tiles.first->as<Tile>(), first_tiles.second,
                                      ctx->set_btcs.empty() || split ? lam_e : lam, grad_u0)) != hipSuccess ||
      (split && (e = burgers::launch_copy_tiles(ctx, ctx->copy_tiles[kSetBtcs].first->as<Tile>(),
                                                ctx->copy_tiles[kSetBtcs].second, lam, grad_u0)) != hipSuccess) ||
      (e = burgers::launch_zero_dirichlet_ends(ctx, static_cast<double*>(grad_u0))) != hipSuccess ||
      (e = burgers::launch_adj_nu(ctx, ap.slot_begin->as<int32_t>(), ap.gslot.as<double>(),
                                  static_cast<double*>(grad_nu))) != hipSuccess)
    return note(ctx, e);
  return BURGERS_OK;
}

burgers_status burgers_sync(burgers_ctx* ctx) {
  if (!ctx) return BURGERS_E_INVALID;
  hipError_t e = hipSetDevice(ctx->device);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e == hipSuccess) e = hipGetLastError();
  note(ctx, e);
  if (ctx->sticky != hipSuccess) return from_hip(ctx->sticky);
  if (ctx->newton && ctx->newton->flags.ptr) {
    // checks of the Newton steps since the last report; cleared once reported
    int flags[2] = {0, 0};
    e = hipMemcpy(flags, ctx->newton->flags.ptr, sizeof(flags), hipMemcpyDeviceToHost);
    if (e == hipSuccess && (flags[0] || flags[1])) {
      e = hipMemsetAsync(ctx->newton->flags.ptr, 0, sizeof(flags), ctx->stream);
      if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
      if (e == hipSuccess) return BURGERS_E_NOT_CONVERGED;
    }
    if (e != hipSuccess) return note(ctx, e);
  }
  return BURGERS_OK;
}

burgers_status burgers_get_plan(const burgers_ctx* ctx, burgers_plan* out) {
  if (!ctx || !out) return BURGERS_E_INVALID;
  *out = ctx->plan;
  return BURGERS_OK;
}

burgers_status burgers_set_plan(burgers_ctx* ctx, const burgers_plan* plan) {
  if (!ctx || !plan) return BURGERS_E_INVALID;
  if (plan->explicit_path < 0 || plan->explicit_path > 3 || plan->btcs_path < 0 || plan->btcs_path > 3 ||
      plan->tblock_depth < 0 || plan->tblock_depth > kMaxDepth || plan->use_graph < -1 || plan->use_graph > 1 ||
      (plan->btcs_block != 0 && plan->btcs_block != 512 && plan->btcs_block != 1024) ||
      plan->btcs_long < 0 || plan->btcs_long > 2 || plan->serial < 0 || plan->serial > 1 ||
      plan->btcs_pipeline < 0 || plan->btcs_pipeline > 2)
    return BURGERS_E_INVALID;
  const bool explicit_changed = plan->explicit_path != ctx->plan.explicit_path ||
                                plan->tblock_depth != ctx->plan.tblock_depth;
  const bool btcs_changed = plan->btcs_path != ctx->plan.btcs_path || plan->btcs_block != ctx->plan.btcs_block ||
                            plan->btcs_long != ctx->plan.btcs_long || plan->btcs_pipeline != ctx->plan.btcs_pipeline;
  ctx->plan = *plan;
  if (explicit_changed) ctx->explicit_plans.clear();
  if (btcs_changed) ctx->btcs.clear();
  for (auto& kv : ctx->graph_cache) (void)hipGraphExecDestroy(kv.second);
  ctx->graph_cache.clear();
  return BURGERS_OK;
}

}  // extern "C"
