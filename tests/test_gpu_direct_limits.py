"""The per-point potential factor where its angle leaves the number range: what the table form
answers.  A softening length whose square underflows makes V12 infinite at r1 = r2, and a
potential whose angle overflows has no phase: the state turns non-finite and the watchdog says so
(status -6).  A softening length whose square overflows makes V12 vanish: the run is the one
without the two-body term.  On the fused small-grid steps and on the line passes.

Tolerance of the last: the same factors in FP64 over 3 steps, 1e-13; 5e-6 in complex64 (some ten
roundings of 2^-24 a step in either run).
"""
import numpy as np
import pytest

from tests.gpu_util import announce, rel_l2

pytestmark = pytest.mark.gpu

SIZES = [(16, 16, 0), (16, 16, 1), (48, 48, 0), (96, 8, 0)]


def run(nx, ny, plan, precision, mode, v, dt_fs=1.0, **kw):
    from paper_1903_02581_amd import Propagator
    announce(f"angle limits {nx}x{ny} plan {plan} {precision} {mode} {kw}")
    g = np.random.default_rng(nx + ny)
    a, b = (g.normal(size=(nx, ny)) + 1j * g.normal(size=(nx, ny)) for _ in range(2))
    p = Propagator(nx, ny, 10.0 * nx, 8.0 * ny, dt_fs=dt_fs, b_tesla=5.0, precision=precision, coulomb_mode=mode, **kw)
    try:
        p.set_pass_plan(plan)
        p.set_potential(v)
        p.init_state(a, b, -1)
        p.step(3)
        return p.store_state(), p.observables(np.full((nx, ny), 0.5))["status"]
    finally:
        p.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nx,ny,plan", SIZES)
def test_infinite_angles_are_reported(nx, ny, plan, precision):
    v = np.zeros((nx, ny))
    for mode in ("table", "direct"):
        assert run(nx, ny, plan, precision, mode, v, soft_nm=1e-200)[1] == -6, mode
    v[1, 2] = 1e308
    for mode in ("table", "direct"):
        assert run(nx, ny, plan, precision, mode, v, dt_fs=2e4, coulomb_c=0.0)[1] == -6, mode


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-13), ("mixed", 5e-6)])
@pytest.mark.parametrize("nx,ny,plan", SIZES)
def test_softening_past_the_number_range(nx, ny, plan, precision, tol):
    v = np.random.default_rng(1).uniform(-2.0, 5.0, (nx, ny))
    ref, status = run(nx, ny, plan, precision, "table", v, coulomb_c=0.0)
    assert status == 0
    for mode in ("table", "direct"):
        got, status = run(nx, ny, plan, precision, mode, v, soft_nm=1e200)
        assert status == 0 and rel_l2(got, ref) <= tol, mode
