"""The plane pass held in registers (complex128, 64- and 128-point lines) against the four
per-axis passes, and repeated bit for bit (its waves share LDS: a missing barrier would show).

Tolerance as for the other fused plans: the same factors in another order over 3 steps, 1e-13."""
import pytest

from workloads.presets import build
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(128, 64), (64, 128), (128, 128)])
def test_register_plane_equals_per_axis(nx, ny):
    import torch
    from paper_1903_02581_amd import Propagator
    w = build("regs", nx, ny, 12.5 * nx, 9.375 * ny, b_tesla=5.0, dt_fs=2.0, steps=3, sigma_x=20.0, seed=nx + ny)
    announce(f"register plane vs per-axis {nx}x{ny}")
    p = Propagator.from_workload(w)
    p.step(w.steps)
    first = p.psi.clone()
    for _ in range(3):
        p.init_state(w.psi_a, w.psi_b, w.sym)
        p.step(w.steps)
        assert torch.equal(p.psi, first)
    p.set_pass_plan(1)
    p.init_state(w.psi_a, w.psi_b, w.sym)
    p.step(w.steps)
    assert float((p.psi - first).norm()) <= 1e-13 * float(first.norm())
    # the per-point form and a recorded run take their own passes; a recorded one the same bits
    p.set_pass_plan(0)
    p.init_state(w.psi_a, w.psi_b, w.sym)
    p.grad_begin(3, 3)
    p.step(w.steps)
    assert torch.equal(p.psi, first)
    p.grad_end()
    p.close()
    q = Propagator.from_workload(w, coulomb_mode="direct")
    q.step(w.steps)
    assert float((q.psi - first).norm()) <= 1e-13 * float(first.norm())
    q.close()
