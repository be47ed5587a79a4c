"""Long BTCS systems at the edge of the windows' accuracy bound: pools accept what the bound accepts and report what it
does not."""
import math

import numpy as np
import pytest

import workloads as W
from gpu_util import TOL_F64, announce, device_run, oracle_run, rel_err

pytestmark = pytest.mark.gpu

# without viscosity theta = C / (1 + C), C = r max|u|, and the bound theta^257 <= 2^-56 is C <= 6.135
EDGE = 1.0 / (2.0 ** (56.0 / 257.0) - 1.0)


def long_problem(rows, bc, C, seed, nu=0.0, values=None, top=2.0):
    """A BTCS problem of `rows` unknowns, its interior state of largest magnitude `top`, and dt such that r top = C."""
    n = rows + (2 if bc == W.BC_DIRICHLET else 0)
    b = W.random_batch(seed, 1, n, n, bc=bc, scheme=W.BTCS, amplitude=2.0)
    p, u = b.problems[0], b.instance(0).copy()
    inner = u[1:-1] if bc == W.BC_DIRICHLET else u
    inner *= top / np.abs(inner).max()
    p.nu = nu
    if bc == W.BC_DIRICHLET:
        p.left, p.right = values if values else (0.5, -0.5)
        u[0], u[-1] = p.left, p.right
    dx = p.length / (n if bc == W.BC_PERIODIC else n - 1)
    p.dt = C * dx / top
    return p, u


def pool_run(problems, states, steps, tick, dtype="f64", slots=None, pool=None):
    """Every problem admitted at once, ticked until done and retired: the statuses and the states."""
    import torch
    import paper_2601_12204_amd as B
    td, npd = (torch.float64, np.float64) if dtype == "f64" else (torch.float32, np.float32)
    own = pool is None
    if own:
        pool = B.Pool(td, W.BTCS, slots or len(problems), max(int(p.n) for p in problems), tick)
    u0 = [torch.from_numpy(np.ascontiguousarray(u, dtype=npd)).to("cuda") for u in states]
    out = [torch.empty_like(u) for u in u0]
    at = [pool.admit(p, u.data_ptr(), k) for p, u, k in zip(problems, u0, steps)]
    assert min(at) >= 0
    while any(pool.remaining(s) > 0 for s in at):
        pool.tick()
    status = [pool.retire(s, o.data_ptr()) for s, o in zip(at, out)]
    torch.cuda.synchronize()
    if own:
        pool.close()
    return status, [o.cpu().numpy() for o in out]


@pytest.mark.parametrize("bc", [W.BC_PERIODIC, W.BC_DIRICHLET])
@pytest.mark.parametrize("rows", [16385, 16392, 16399, 16400, 30011])
def test_pool_accepts_up_to_the_bound(rows, bc):
    """Rows with 15, 8, 1, 0 and 5 chunks of 15 rows, up to the edge of the bound: accepted, the same bits as a
    context's run (whole calls, one step per launch) and the oracle's states; beyond it: reported."""
    factors = [0.9, 0.95, 0.9999]
    cases = [long_problem(rows, bc, f * EDGE, 40 + k) for k, f in enumerate(factors)]
    problems, states = [c[0] for c in cases], [c[1] for c in cases]
    steps = [11, 12, 13]
    announce(f"bound: {rows} rows, bc {bc}")
    status, got = pool_run(problems, states, steps, 5)
    assert status == [0, 0, 0]
    for p, u, k, g in zip(problems, states, steps, got):
        one = W._pack([p], [u])
        assert np.array_equal(g, device_run(one, k, "f64"))
        assert np.array_equal(g, device_run(one, k, "f64", plan=dict(btcs_path=1)))
        assert rel_err(g, oracle_run(one, k, "f64")) <= TOL_F64
    p, u = long_problem(rows, bc, 1.0001 * EDGE, 43)
    assert pool_run([p], [u], [3], 5)[0] == [-8]


def test_pool_boundary_values_beyond_the_bound():
    """Dirichlet values beyond the bound over an interior within it.  A value that the flow carries out (all u < 0 at the
    left end, no viscosity) never reaches a coefficient: accepted at every tick, the context's bits and the oracle's
    states.  One that it carries in is met after a few steps: reported, from then on."""
    rows, C = 16385, 3.0
    out_p, out_u = long_problem(rows, W.BC_DIRICHLET, C, 51, values=(-50.0, -1.0))
    out_u[1:-1] = -np.abs(out_u[1:-1]) - 0.1
    in_p, in_u = long_problem(rows, W.BC_DIRICHLET, C, 52, values=(50.0, 1.0))
    in_u[1:-1] = np.abs(in_u[1:-1]) + 0.1
    announce("bound: boundary values")
    status, got = pool_run([out_p, in_p], [out_u, in_u], [13, 13], 4)
    assert status == [0, -8]
    one = W._pack([out_p], [out_u])
    assert np.array_equal(got[0], device_run(one, 13, "f64", plan=dict(btcs_path=1)))
    assert rel_err(got[0], oracle_run(one, 13, "f64")) <= TOL_F64


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_pool_reports_failed_bounds_per_request(dtype):
    """A stiff request over several ticks is reported, a mild one beside it and the next ones of its slot (long, then
    short) are not and equal their solo runs; a long state that holds an infinity or a NaN is reported too."""
    import torch
    import paper_2601_12204_amd as B
    mild = [long_problem(r, bc, 0.5 * EDGE, 60 + r) for r, bc in
            ((16399, W.BC_PERIODIC), (20001, W.BC_DIRICHLET), (17000, W.BC_PERIODIC), (700, W.BC_PERIODIC))]
    stiff = long_problem(18000, W.BC_PERIODIC, 1000.0, 71)
    announce(f"bound: reports per request {dtype}")
    pool = B.Pool(torch.float64 if dtype == "f64" else torch.float32, W.BTCS, 2, 20010, 4)
    status, got = pool_run([mild[0][0], stiff[0]], [mild[0][1], stiff[1]], [9, 14], 4, dtype, pool=pool)
    assert status == [0, -8]
    for k, (a, b) in enumerate(((2, 1), (2, 3))):
        (pa, ua), (pb, ub) = mild[a], mild[b]
        status, got = pool_run([pa, pb], [ua, ub], [5, 11], 4, dtype, pool=pool)
        assert status == [0, 0], k
        for p, u, n, g in ((pa, ua, 5, got[0]), (pb, ub, 11, got[1])):
            assert np.array_equal(g, device_run(W._pack([p], [u]), n, dtype))
    for bad in (np.inf, np.nan):
        p, u = mild[1]
        u = u.copy()
        u[len(u) // 2] = bad
        assert pool_run([p, mild[0][0]], [u, mild[0][1]], [6, 6], 4, dtype, pool=pool)[0] == [-8, 0]
    pool.close()


def test_long_states_that_are_not_finite_leave_the_windows():
    """... and in a context they are solved by the partition levels, like with windows forbidden, and leave the other
    instances alone."""
    p, u = long_problem(16399, W.BC_PERIODIC, 0.5 * EDGE, 81)
    q, v = long_problem(20001, W.BC_DIRICHLET, 0.5 * EDGE, 82)
    announce("bound: states that are not finite")
    want = device_run(W._pack([q], [v]), 6, "f64")
    for bad in (np.inf, np.nan):
        w = u.copy()
        w[5] = bad
        both = W._pack([p, q], [w, v])
        got = device_run(both, 6, "f64")
        levels = device_run(both, 6, "f64", plan=dict(btcs_long=1))
        assert np.array_equal(got[:len(u)], levels[:len(u)], equal_nan=True)
        assert not np.all(np.isfinite(got[:len(u)]))
        assert np.array_equal(got[len(u):], want)
