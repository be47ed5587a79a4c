"""Explicit instances of up to 1024 nodes, held by one wave each, at the edges of the nodes per lane: bitwise
equal to the streaming kernel (forward Euler) and within the parity bars of the oracle, on their own and
packed beside longer instances."""
import numpy as np
import pytest

import workloads as W
from gpu_util import announce, assert_explicit_parity, device_run, oracle_run, set_cfl_steps

pytestmark = pytest.mark.gpu

SIZES = [3, 4, 5, 33, 62, 63, 64, 65, 66, 127, 128, 129, 191, 192, 193, 300, 449, 512, 513, 640, 777, 960, 961, 1000,
         1023, 1024]


def _batch(seed, sizes, scheme):
    problems, states = [], []
    for k, n in enumerate(sizes):
        for bc in (W.BC_PERIODIC, W.BC_DIRICHLET):
            b = W.random_batch(seed + 23 * k + bc, 1, n, n, bc=bc, scheme=scheme, amplitude=3.0)
            problems.append(b.problems[0])
            states.append(b.instance(0))
    return set_cfl_steps(W._pack(problems, states), scheme=W.EXPLICIT)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("beside", [[], [1025, 2049, 5000]])
@pytest.mark.parametrize("nsteps", [1, 40])
def test_euler_waves(dtype, beside, nsteps):
    batch = _batch(4100, SIZES + beside, W.EXPLICIT)
    announce(f"euler waves {dtype} beside {beside}, {nsteps} steps")
    got = device_run(batch, nsteps, dtype, how="run")
    assert np.array_equal(got, device_run(batch, nsteps, dtype, how="run", plan=dict(explicit_path=1)))
    assert_explicit_parity(batch, got, oracle_run(batch, nsteps, dtype), dtype)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("beside", [[], [1025, 2049, 5000]])
def test_rk4_waves(dtype, beside):
    batch = _batch(4300, SIZES + beside, W.RK4)
    announce(f"rk4 waves {dtype} beside {beside}, 21 steps")
    got = device_run(batch, 21, dtype, how="run")
    assert_explicit_parity(batch, got, oracle_run(batch, 21, dtype), dtype)
