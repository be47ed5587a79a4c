"""Long BTCS systems on truncated windows of several steps per launch: against the oracle, and alike to the bit
however a call's steps are spread over launches and calls."""
import numpy as np
import pytest

import workloads as W
from gpu_util import announce, check_batch, device_run, set_cfl_steps

pytestmark = pytest.mark.gpu

# rows around one window's and several windows' share, with 0, 1 and 15 chunks of 15 rows
ROWS = [16385, 16399, 16400, 3 * 6144, 6144 * 4 + 1, 40001, 65536]


def long_batch(seed, rows, factor):
    problems, states = [], []
    for k, R in enumerate(rows):
        for bc in (W.BC_PERIODIC, W.BC_DIRICHLET):
            n = R + (2 if bc == W.BC_DIRICHLET else 0)
            b = W.random_batch(seed + 13 * k + bc, 1, n, n, bc=bc, scheme=W.BTCS, amplitude=3.0)
            problems.append(b.problems[0])
            states.append(b.instance(0))
    return set_cfl_steps(W._pack(problems, states), scheme=W.BTCS, btcs_factor=factor)


def split_run(batch, parts, dtype):
    import torch
    import paper_2601_12204_amd as B
    s = B.Solver(batch.problems, dtype=torch.float64 if dtype == "f64" else torch.float32)
    u = s.pack_flat(batch.u0, batch.offsets)
    for k in parts:
        s.run(u, k)
    s.sync()
    out = s.unpack_flat(u)
    s.close()
    return out


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("factor", [0.1, 1.0, 10.0, 30.0])
def test_windows_of_several_steps(dtype, factor):
    """Time steps whose solves take one to four PCR steps (32, 16, 8 and 4 steps a launch): the oracle, one step per
    launch, and calls split at steps that are no multiple of a launch's."""
    batch = long_batch(4100, ROWS, factor)
    n = 37
    announce(f"long windows {dtype} x{factor}, {batch.count} systems, {n} steps")
    got = device_run(batch, n, dtype, how="run")
    assert np.array_equal(got, device_run(batch, n, dtype, how="run", plan=dict(btcs_path=1)))
    assert np.array_equal(got, split_run(batch, [4, 3, 19, 11], dtype))
    assert np.array_equal(got, device_run(batch, n, dtype, how="run", plan=dict(serial=1, use_graph=1)))
    check_batch(batch, got, n, dtype)


@pytest.mark.parametrize("steps", [8, 9])
def test_windows_beside_systems_beyond_their_bound(steps):
    """Systems of one call within the windows' bound and, at 10^3 times the CFL step, beyond it: the latter bitwise
    the partition levels' solve, after even and odd step counts."""
    mild, stiff = long_batch(4300, ROWS[:4], 10.0), long_batch(4500, ROWS[1:4], 1000.0)
    both = W._pack(mild.problems + stiff.problems,
                   [mild.instance(k) for k in range(mild.count)] + [stiff.instance(k) for k in range(stiff.count)])
    announce(f"long windows beside stiff systems, {steps} steps")
    got = device_run(both, steps, "f64", how="run")
    cut = int(mild.offsets[-1])
    assert np.array_equal(got[:cut], device_run(mild, steps, "f64", how="run"))
    assert np.array_equal(got[cut:], device_run(stiff, steps, "f64", how="run", plan=dict(btcs_long=1)))
    check_batch(both, got, steps, "f64")
