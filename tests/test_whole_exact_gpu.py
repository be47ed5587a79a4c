"""Whole BTCS and Crank-Nicolson systems one step per launch: groups whose systems all fill their lanes, and such systems
beside ragged ones."""
import numpy as np
import pytest

import workloads as W
from gpu_util import announce, check_batch, device_run, set_cfl_steps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("rows", [[8192], [16384], [8192, 5000], [16384, 8193], [4096, 8192, 16384]])
def test_full_groups(dtype, rows):
    """Per-step solves bitwise those on chip, and the oracle's."""
    problems, states = [], []
    for k, R in enumerate(rows):
        for bc in (W.BC_PERIODIC, W.BC_DIRICHLET):
            n = R + (2 if bc == W.BC_DIRICHLET else 0)
            b = W.random_batch(6100 + 7 * k + bc, 1, n, n, bc=bc, scheme=W.BTCS, amplitude=2.0)
            problems.append(b.problems[0])
            states.append(b.instance(0))
    batch = set_cfl_steps(W._pack(problems, states))
    announce(f"whole systems per step {rows} {dtype}")
    got = device_run(batch, 6, dtype, plan=dict(btcs_path=1))
    assert np.array_equal(got, device_run(batch, 6, dtype))
    check_batch(batch, got, 6, dtype)
    for p in batch.problems:
        p.scheme = W.CN
    check_batch(batch, device_run(batch, 6, dtype, plan=dict(btcs_path=1)), 6, dtype)
