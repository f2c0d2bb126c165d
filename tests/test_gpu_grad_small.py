"""Gradients on the grids whose nx ny is not a whole number of the finishing kernel's groups of
16 entries (4 and 6 by 6 and 12 points), and the neighbours that are, against the oracle's
stored-state adjoint; every entry of dL/dV is compared, the last ones on their own too.

Tolerance: as for every other size, 1e-10 of the largest entry (a few steps of FP64 transforms).
"""
import numpy as np
import pytest

import oracle as O
from workloads.presets import build
from tests.gpu_util import announce, grid_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("nx,ny", [(4, 6), (6, 4), (6, 6), (6, 12), (12, 6), (4, 4), (6, 8), (4, 12)])
def test_every_entry_of_the_gradient(nx, ny, noalloc):
    from paper_1903_02581_amd import Propagator
    steps = 5
    w = build("g", nx, ny, 25.0 * nx, 25.0 * ny, b_tesla=5.0, dt_fs=5.0, steps=steps, sigma_x=20.0, seed=1, sx=30.0)
    g = np.random.default_rng(nx * 100 + ny)
    # orbitals and region weights that reach every point, so that no entry vanishes
    a, b = (g.normal(size=(nx, ny)) + 1j * g.normal(size=(nx, ny)) for _ in range(2))
    v, top = g.uniform(-3.0, 3.0, (nx, ny)), g.uniform(0.0, 1.0, (nx, ny))
    announce(f"every entry of dL/dV {nx}x{ny} noalloc={noalloc}")
    psi0 = O.init_state(a, b, -1)
    ref_l, ref_v, ref_b = O.loss_and_grad_stored(psi0, grid_of(w), v, w.dt_fs, steps, top)
    p = Propagator.from_workload(w)
    try:
        p.set_potential(v)
        p.init_state(a, b, -1)
        p.grad_begin(2, steps)
        p.step(steps)
        loss, dv, db = p.grad_backward(top, noalloc=noalloc)
    finally:
        p.close()
    size = np.max(np.abs(ref_v))
    assert np.all(np.abs(ref_v) > 1e-6 * size)
    assert abs(loss - ref_l) <= 1e-12
    assert np.max(np.abs(dv - ref_v)) <= 1e-10 * size
    assert np.all(dv.reshape(-1)[-8:] != 0.0)
    assert abs(db - ref_b) <= 1e-10 * max(abs(ref_b), size)
