"""The start of a run where its kernels split their work: the transverse reduction that goes
on in the 64-row form after the first ny - 64 columns, and the initial norm over tiles of r2
that each take half of the tiles as r1 (an even and an odd number of tiles, in both tile
sizes; with sym = 0, all of them).

Tolerances: edge packets as for every size; a thread of the norm adds at most a few hundred
positive terms in turn and the blocks' sums are trees, so its relative error, and the
state's, stays below 500 eps.
"""
import numpy as np
import pytest

from tests.gpu_util import announce
from tests.test_gpu_edge import _check_workload, build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(8, 64), (8, 128), (64, 128)])
def test_packets_where_the_reduction_changes_form(nx, ny):
    announce(f"edge packets {nx}x{ny}")
    _check_workload(build("edge", nx, ny, 25.0 * nx, 4.0 * ny, b_tesla=5.0, dt_fs=1.0, steps=1, sigma_x=12.0, seed=3))


@pytest.mark.parametrize("nx,ny", [(8, 64), (12, 64), (64, 64), (64, 96)])
@pytest.mark.parametrize("sym", [-1, 0, 1])
def test_norm_over_half_the_tiles(nx, ny, sym):
    from paper_1903_02581_amd import Propagator
    announce(f"initial norm {nx}x{ny} sym {sym}")
    g = np.random.default_rng(nx + ny)
    a, b = (g.normal(size=(nx, ny)) + 1j * g.normal(size=(nx, ny)) for _ in range(2))
    p = Propagator(nx, ny, 10.0 * nx, 8.0 * ny, dt_fs=1.0, b_tesla=5.0)
    try:
        p.init_state(a, b, sym)
        # ||a b + sym b a||^2 = 2 (|a|^2 |b|^2 + sym |<a, b>|^2); |a b + sym b a| on one row
        na, nb, ab = np.sum(np.abs(a) ** 2), np.sum(np.abs(b) ** 2), np.abs(np.vdot(a, b)) ** 2
        norm = np.sqrt(na * nb if sym == 0 else 2.0 * (na * nb + sym * ab))
        got = p.psi.cpu().numpy().reshape(nx * ny, -1)
        for r in (0, 7, nx * ny - 1):
            ref = (a.flat[r] * b + (sym * b.flat[r] * a if sym else 0.0)).reshape(-1) / norm
            assert np.max(np.abs(got[r] - ref)) <= 500 * np.finfo(float).eps * np.max(np.abs(ref))
    finally:
        p.close()
