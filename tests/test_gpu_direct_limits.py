"""The per-point potential factor where its angle leaves the number range: what the table form
answers.  A softening length whose square underflows makes V12 infinite at r1 = r2, and a
potential whose angle overflows has no phase: the state turns non-finite and the watchdog says so
(status -6).  On the fused small-grid steps and on the line passes.
"""
import numpy as np
import pytest

from tests.gpu_util import announce

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
