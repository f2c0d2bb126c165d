"""Forward x2 passes on grids whose y2 rows hold 2 or 4 lines to a power of two: blocks of a
wavefront, of more where the grid has lines enough, and of all the lines there are, against
the oracle.  Tolerances as for the other plans: 1e-10 in complex128, 5e-6 in complex64."""
import pytest

from workloads.presets import build
from tests.gpu_util import announce, oracle_run, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(4, 4), (8, 4), (6, 6), (16, 6), (32, 4), (48, 6), (96, 4), (96, 6), (128, 4),
                                   (256, 4), (64, 12)])
def test_x2_block_widths(nx, ny):
    from paper_1903_02581_amd import Propagator
    w = build("x2", nx, ny, 12.5 * nx, 9.375 * ny, b_tesla=5.0, dt_fs=2.0, steps=2, sigma_x=20.0, seed=nx * 7 + ny)
    announce(f"x2 block widths {nx}x{ny}")
    ref, _ = oracle_run(w, 2)
    for precision, tol in (("fp64", 1e-10), ("mixed", 5e-6)):
        p = Propagator.from_workload(w, precision=precision)
        try:
            p.set_pass_plan(1)
            p.step(2)
            assert rel_l2(p.store_state(), ref) <= tol, precision
        finally:
            p.close()
