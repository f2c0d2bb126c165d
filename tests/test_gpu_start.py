"""The start of a run where its kernels split their work: the transverse reduction that goes
on in the 64-row form after the first ny - 64 columns.  Tolerance as for every size.
"""
import pytest

from tests.gpu_util import announce
from tests.test_gpu_edge import _check_workload, build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(8, 64), (8, 128), (64, 128)])
def test_packets_where_the_reduction_changes_form(nx, ny):
    announce(f"edge packets {nx}x{ny}")
    _check_workload(build("edge", nx, ny, 25.0 * nx, 4.0 * ny, b_tesla=5.0, dt_fs=1.0, steps=1, sigma_x=12.0, seed=3))
