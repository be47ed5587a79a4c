"""The BTCS adjoint on windows of several reverse steps, and on whole systems beyond the windows' bound, over several
launches a segment: against the oracle, and alike to the bit however the steps are grouped."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_util import announce
from test_adjoint_gpu import TOL, _device_adjoint_plan, _nu_bound

pytestmark = pytest.mark.gpu

# the edges of whole systems, with 15 to 0 chunks of 15 rows, and longer ones
ROWS = [8193, 8200, 9215, 12000, 16383, 16384, 16385, 20011]


def smooth_batch(C):
    """Positive smooth states (no node changes its upwind side) of largest magnitude 2, and r 2 = C."""
    problems, states = [], []
    for k, rows in enumerate(ROWS):
        for bc in (W.BC_PERIODIC, W.BC_DIRICHLET):
            n = rows + (2 if bc == W.BC_DIRICHLET else 0)
            p = W.random_batch(1, 1, n, n, bc=bc, scheme=W.BTCS).problems[0]
            dx = p.length / (n if bc == W.BC_PERIODIC else n - 1)
            u = 1.2 + 0.8 * np.sin(np.arange(n) * dx + 0.7 * k)
            p.dt = C * dx / 2.0
            p.nu = 0.02 * dx * dx / p.dt
            if bc == W.BC_DIRICHLET:
                p.left, p.right = u[0], u[-1]
            problems.append(p)
            states.append(u)
    return W._pack(problems, states)


@pytest.mark.parametrize("C", [0.2, 0.7, 1.7, 4.0, 9.0])
def test_btcs_adjoint_over_several_launches(C):
    """One to four PCR steps a solve (40, 20, 10 and 5 reverse steps a launch: 95 steps take 3, 5, 10 and 19 launches,
    segments of 48 and 47 two, three, five and ten), and, at C = 9, whole systems and the array path."""
    batch = smooth_batch(C)
    lam = np.random.default_rng(41).standard_normal(len(batch.u0))
    announce(f"BTCS adjoint windows C={C}, {batch.count} instances")
    g, gn = _device_adjoint_plan(batch, lam, 95, 95)
    for ckpt in (48, 7):
        other, othern = _device_adjoint_plan(batch, lam, 95, ckpt)
        assert np.array_equal(g, other) and np.array_equal(gn, othern), ckpt
    rg, rgn = oracle.adjoint(batch.problems, batch.u0, batch.offsets, lam, 95)
    for b in range(batch.count):
        lo, hi = batch.offsets[b], batch.offsets[b + 1]
        assert oracle.rel_max_abs(g[lo:hi], rg[lo:hi]) <= TOL, (b, batch.problems[b])
    bound = _nu_bound(batch, lam, 95, rgn)
    assert np.all(np.abs(gn - rgn) <= bound), (np.abs(gn - rgn), bound)
