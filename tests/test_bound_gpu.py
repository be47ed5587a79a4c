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
