"""BTCS rows without viscosity: no coupling to the neighbour downstream, to the bit."""
import numpy as np
import pytest

import workloads as W
from gpu_util import announce
from test_adjoint_gpu import _device_adjoint_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_nothing_is_carried_against_the_flow(sign):
    """A flow of one sign and nu = 0: a loss of the nodes up to the middle (from there on, for a flow to the left) has
    a gradient of exactly zero on the others, after several steps and for every solver of the transposed systems."""
    problems, states, lams = [], [], []
    for n in (5, 64, 101, 700, 3000, 8194, 9003, 16386, 20002):
        p = W.random_batch(1, 1, n, n, bc=W.BC_DIRICHLET, scheme=W.BTCS).problems[0]
        x = np.arange(n) / (n - 1)
        u = sign * (1.2 + 0.7 * np.sin(40.0 * x + 0.3))
        dx = p.length / (n - 1)
        p.nu, p.left, p.right, p.dt = 0.0, u[0], u[-1], 1.3 * dx
        lam = np.where(x <= 0.5 if sign > 0 else x >= 0.5, 1.0 + x, 0.0)
        problems.append(p)
        states.append(u)
        lams.append(lam)
    batch = W._pack(problems, states)
    announce(f"row couplings, flow {sign:+.0f}")
    g, _ = _device_adjoint_plan(batch, np.concatenate(lams), 6, 3)
    for b in range(batch.count):
        mine, lam = g[batch.offsets[b]:batch.offsets[b + 1]], lams[b]
        assert np.all(mine[lam == 0.0] == 0.0), (problems[b].n, np.abs(mine[lam == 0.0]).max())
        assert np.all(mine[1:-1][lam[1:-1] != 0.0] != 0.0)
