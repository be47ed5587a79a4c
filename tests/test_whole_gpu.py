"""Implicit systems solved whole by one workgroup, at the edges of the lane and slot classes, against the
oracle (the parity bars of gpu_util)."""
import numpy as np
import pytest

import workloads as W
from gpu_util import announce, check_batch, device_run, set_cfl_steps

pytestmark = pytest.mark.gpu


def edge_batch(seed, rows, scheme):
    """One problem per row count and boundary type (a Dirichlet system has two nodes more than rows)."""
    problems, states = [], []
    for k, R in enumerate(rows):
        for bc in (W.BC_PERIODIC, W.BC_DIRICHLET):
            n = R + (2 if bc == W.BC_DIRICHLET else 0)
            if n < 3:
                continue
            b = W.random_batch(seed + 19 * k + bc, 1, n, n, bc=bc, scheme=scheme, amplitude=3.0)
            problems.append(b.problems[0])
            states.append(b.instance(0))
    return set_cfl_steps(W._pack(problems, states), scheme=scheme)


# row counts on both sides of every change of lanes, chunks or slots: 64 lanes of 2 to 8 slots with 1 to 64
# chunks, then 128, 256, 512 and 1024 lanes with one chunk short by a row, all but one, and none
ROWS = [1, 2, 3, 5, 6, 7, 63, 64, 65, 96, 97, 127, 128, 129, 192, 320, 449, 511, 512, 513, 640, 1024, 1025, 2047,
        2048, 2049, 3585, 4095, 4096, 4097, 4608, 4609, 7681, 8191, 8193, 9216, 9217, 12345, 15361, 16383]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_btcs_slot_classes(dtype):
    """On chip and per step, bitwise alike, and against the oracle."""
    batch = edge_batch(3100, ROWS, W.BTCS)
    announce(f"btcs slot classes {dtype}, {batch.count} systems, 13 steps")
    chip = device_run(batch, 13, dtype, how="run")
    step = device_run(batch, 13, dtype, how="run", plan=dict(btcs_path=1))
    assert np.array_equal(chip, step)
    check_batch(batch, chip, 13, dtype)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_cn_slot_classes(dtype):
    """Crank-Nicolson systems of up to 8192 rows are held on chip, longer ones take the per-step solvers."""
    batch = edge_batch(3300, ROWS + [8192], W.CN)
    announce(f"cn slot classes {dtype}, {batch.count} systems, 9 steps")
    got = device_run(batch, 9, dtype, how="run")
    check_batch(batch, got, 9, dtype)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_newton_slot_classes(dtype):
    """Newton systems of up to 8192 rows are held on chip (at the CFL step every row stays dominant and the
    increments converge, so the checks report nothing)."""
    batch = edge_batch(3500, [r for r in ROWS if 63 <= r <= 8192] + [8192, 9000], W.NEWTON)
    announce(f"newton slot classes {dtype}, {batch.count} systems, 5 steps")
    got = device_run(batch, 5, dtype, how="run")
    check_batch(batch, got, 5, dtype)


def test_newton_checks_alike_on_chip_and_per_step():
    """The dominance and increment checks report the same on chip and through HBM (groups of 64 unknowns),
    from in range to far beyond it, on row counts whose lanes' chunks straddle the groups."""
    import paper_2601_12204_amd as B
    seen = set()
    for k, (n, factor) in enumerate([(70, 1.0), (70, 12.0), (200, 1.0), (200, 30.0), (777, 1.0), (777, 40.0),
                                     (1500, 25.0), (5000, 1.0), (5000, 60.0)]):
        for bc in (W.BC_PERIODIC, W.BC_DIRICHLET):
            batch = W.random_batch(3700 + 2 * k + bc, 1, n, n, bc=bc, scheme=W.NEWTON, amplitude=3.0, nu_lo=1e-3,
                                   nu_hi=2e-3)
            set_cfl_steps(batch, btcs_factor=factor, explicit_factor=factor)
            reports = []
            for plan in (None, dict(btcs_path=1)):
                announce(f"newton checks n={n} bc={bc} x{factor} plan={plan}")
                try:
                    device_run(batch, 1, "f64", how="run", plan=plan)
                    reports.append(0)
                except B.BurgersError as err:
                    reports.append(err.status)
            assert reports[0] == reports[1], (n, bc, factor, reports)
            seen.add(reports[0])
    assert seen == {0, -7}
