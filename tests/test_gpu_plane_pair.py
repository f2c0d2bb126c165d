"""Steps as two fused plane passes, at every grid that has both, against the four
per-axis passes; and the forward x2 pass where a block's lines run over the end of a
y2 row, against the oracle.

Tolerances: complex128, the same factors in another order over 3 steps, 1e-13 as for the
three-pass plan; complex64, at most 11 roundings of 2^-24 a step in either plan, added up
linearly over 3 steps: 2 * 33 * 2^-24 < 5e-6.
"""
import itertools

import numpy as np
import pytest

from workloads.presets import build
from tests.gpu_util import announce, oracle_run, rel_l2

pytestmark = pytest.mark.gpu

PAIRS = [(x, y) for x, y in itertools.product((8, 12, 16, 24, 32, 48, 64), repeat=2)
         if x * y <= 1024 and not (x == 64 and y == 12)]


def workload(nx, ny, steps):
    return build("pair", nx, ny, 12.5 * nx, 9.375 * ny, b_tesla=5.0, dt_fs=2.0, steps=steps, sigma_x=20.0,
                 seed=nx * 7 + ny)


@pytest.mark.parametrize("nx,ny", PAIRS)
def test_two_passes_equal_four(nx, ny):
    from paper_1903_02581_amd import Propagator
    w = workload(nx, ny, 3)
    for precision, mode, tol in (("fp64", "table", 1e-13), ("fp64", "direct", 1e-13), ("mixed", "table", 5e-6),
                                 ("mixed", "direct", 5e-6)):
        announce(f"pair vs per-axis {nx}x{ny} {precision} {mode}")
        out = []
        for plan in (0, 1):
            p = Propagator.from_workload(w, precision=precision, coulomb_mode=mode)
            p.set_pass_plan(plan)
            p.step(w.steps)
            out.append(p.store_state())
            if plan == 0:  # the same launches again give the same bits
                p.init_state(w.psi_a, w.psi_b, w.sym)
                p.step(w.steps)
                assert np.array_equal(p.store_state(), out[0])
            p.close()
        assert rel_l2(out[0], out[1]) <= tol


def test_recorded_complex64_run_keeps_its_passes():
    """A recorded complex64 run and its reverse sweep round in the same places as before."""
    from paper_1903_02581_amd import Propagator
    w = workload(32, 32, 4)
    announce("recorded complex64 run 32x32")
    p = Propagator.from_workload(w, precision="mixed")
    p.grad_begin(2, 4)
    p.step(4)
    recorded = p.store_state()
    p.grad_end()
    p.init_state(w.psi_a, w.psi_b, w.sym)
    p.pass_timing(True)  # the three-pass plan, pass by pass; checkpoints close the state every 2 steps
    p.step(2)
    p.step(2)
    assert np.array_equal(p.store_state(), recorded)
    p.close()


@pytest.mark.parametrize("nx,ny", [(96, 24), (128, 6), (48, 24), (64, 12), (256, 12), (96, 6), (24, 4)])
def test_x2_blocks_over_row_ends(nx, ny):
    w = workload(nx, ny, 2)
    announce(f"x2 blocks {nx}x{ny}")
    from paper_1903_02581_amd import Propagator
    ref, _ = oracle_run(w, 2)
    for precision, tol in (("fp64", 1e-10), ("mixed", 5e-6)):
        p = Propagator.from_workload(w, precision=precision)
        p.step(2)
        assert rel_l2(p.store_state(), ref) <= tol
        p.close()
