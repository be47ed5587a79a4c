"""The explicit adjoint on one-wave windows that read every fourth state: at the edges of the windows' shares, of the
states' groups and of the runs of a launch, against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_util import announce, set_cfl_steps
from test_adjoint_gpu import TOL, _device_adjoint_plan, _nu_bound

pytestmark = pytest.mark.gpu

# a window keeps up to 896 nodes in runs of 16; instances shorter than a halo go around the window
SIZES = [3, 15, 16, 17, 63, 64, 65, 129, 895, 896, 897, 912, 1023, 1024, 1025, 1792, 1793, 5000]


@pytest.mark.parametrize("nsteps,ckpt", [(1, 1), (3, 4), (4, 4), (61, 61), (130, 65)])
def test_explicit_adjoint_windows(nsteps, ckpt):
    problems, states = [], []
    for k, n in enumerate(SIZES):
        for bc in (W.BC_PERIODIC, W.BC_DIRICHLET):
            b = W.random_batch(5100 + 23 * k + bc, 1, n, n, bc=bc, scheme=W.EXPLICIT, amplitude=2.0)
            problems.append(b.problems[0])
            states.append(b.instance(0))
    batch = set_cfl_steps(W._pack(problems, states))
    lam = np.random.default_rng(31).standard_normal(len(batch.u0))
    announce(f"explicit adjoint windows, {batch.count} instances, {nsteps} steps, checkpoints every {ckpt}")
    g, gn = _device_adjoint_plan(batch, lam, nsteps, ckpt)
    rg, rgn = oracle.adjoint(batch.problems, batch.u0, batch.offsets, lam, nsteps)
    for b in range(batch.count):
        lo, hi = batch.offsets[b], batch.offsets[b + 1]
        assert oracle.rel_max_abs(g[lo:hi], rg[lo:hi]) <= TOL, (b, batch.problems[b])
    bound = _nu_bound(batch, lam, nsteps, rgn)
    assert np.all(np.abs(gn - rgn) <= bound), (np.abs(gn - rgn), bound)
    one, onen = _device_adjoint_plan(batch, lam, nsteps, 1)
    assert np.array_equal(g, one) and np.array_equal(gn, onen)
