"""Long BTCS systems at the windows' bound: the same bits however a call's steps are split, whichever entry point takes
them, while states come within the bound step by step."""
import numpy as np
import pytest

import workloads as W
from gpu_util import TOL_F64, announce, device_run, oracle_run, per_instance_rel
from test_bound_gpu import EDGE, long_problem
from test_windows_gpu import split_run
from test_zz_no_alloc import _dense, _static_run

pytestmark = pytest.mark.gpu

SPLITS = [[1] * 12, [2] * 6, [3, 9], [3, 3, 3, 3], [7, 1, 4], [2, 10]]


def decaying(rows, bc, over, width, seed):
    """A spike of `width` nodes over a low state, `over` times the edge of the bound: within it once it has decayed."""
    p, u = long_problem(rows, bc, over * EDGE, seed)
    inner = u[1:-1] if bc == W.BC_DIRICHLET else u
    inner *= 0.1
    at = len(inner) // 3
    inner[at:at + width] = 2.0
    return p, u


def assert_alike(batch, n, dtype, splits=SPLITS):
    want = device_run(batch, n, dtype)
    for plan in (dict(btcs_path=1), dict(serial=1, use_graph=1), dict(btcs_long=2)):
        assert np.array_equal(want, device_run(batch, n, dtype, plan=plan)), plan
    for parts in splits:
        assert np.array_equal(want, split_run(batch, parts, dtype)), parts
    return want


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_states_that_come_within_the_bound(dtype):
    """Instances beyond the bound at the start, within it after no step of the call, one, or several; some beside them
    within it all along."""
    cases = []
    for k, (over, width) in enumerate([(1.02, 1), (1.02, 60), (1.3, 25), (4.0, 3), (4.0, 200), (40.0, 4000), (0.5, 9)]):
        for bc in (W.BC_PERIODIC, W.BC_DIRICHLET):
            cases.append(decaying((16385, 16400, 30011)[k % 3], bc, over, width, 200 + 2 * k + bc))
    batch = W._pack([c[0] for c in cases], [c[1] for c in cases])
    announce(f"split: {batch.count} decaying states {dtype}")
    want = assert_alike(batch, 12, dtype)
    if dtype == "f64":   # (the windows' error is below the rounding of a binary32 state)
        # the levels alone differ where the windows took over, and only by the windows' error
        levels = device_run(batch, 12, dtype, plan=dict(btcs_long=1))
        same = [np.array_equal(want[a:b], levels[a:b]) for a, b in zip(batch.offsets[:-1], batch.offsets[1:])]
        assert any(same) and not all(same)
        assert per_instance_rel(batch, want, oracle_run(batch, 12, "f64")).max() <= TOL_F64
    # graphs replayed between calls of the context's own, the flags decided anew each time
    assert np.array_equal(device_run(batch, 4, dtype, reps=3), want)
    assert np.array_equal(device_run(batch, 4, dtype, plan=dict(use_graph=1), reps=3), want)
    u, off = _static_run(batch, dtype, 12)
    assert np.array_equal(want, _dense(u, off, batch.problems))
    # beside a long Crank-Nicolson system every step is a launch of its own
    cn, v = long_problem(17000, W.BC_PERIODIC, 1.0, 299)
    cn.scheme = W.CN
    both = W._pack(batch.problems + [cn], [c[1] for c in cases] + [v])
    assert np.array_equal(want, device_run(both, 12, dtype)[:len(want)])


def test_boundary_values_beyond_the_bound():
    """Dirichlet values beyond the bound over a small interior, carried in by the flow and out, beside a mild system."""
    a, u = long_problem(16399, W.BC_DIRICHLET, 3.0, 301, values=(50.0, 1.0))
    u[1:-1] = np.abs(u[1:-1]) + 0.1
    b, v = long_problem(16399, W.BC_DIRICHLET, 3.0, 302, values=(-50.0, -1.0))
    v[1:-1] = -np.abs(v[1:-1]) - 0.1
    c, w = long_problem(20000, W.BC_PERIODIC, 3.0, 303)
    batch = W._pack([a, b, c], [u, v, w])
    announce("split: boundary values beyond the bound")
    want = assert_alike(batch, 12, "f64")
    assert per_instance_rel(batch, want, oracle_run(batch, 12, "f64")).max() <= TOL_F64


def test_three_level_systems_that_come_within_the_bound():
    """Systems whose reduced rows are reduced again (more than 2^24 rows)."""
    p, u = decaying((1 << 24) + 5000, W.BC_PERIODIC, 1.3, 25, 311)
    batch = W._pack([p], [u])
    announce("split: more than 2^24 rows")
    want = device_run(batch, 5, "f64")
    for parts in ([1] * 5, [3, 2]):
        assert np.array_equal(want, split_run(batch, parts, "f64")), parts
