"""The pair kernels where their grid changes form: rows that fill four accesses per thread to just
below and above two thirds, and rows grouped in twos, threes and fours with a shorter last
group.  Checks and tolerances of the pair kernels' other sizes."""
import pytest

from tests.test_gpu_pair_kernels import test_init_and_observables as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nx,ny", [(32, 24), (24, 48), (48, 32), (96, 24), (32, 96), (12, 128)])
def test_forms_of_the_pair_grid(nx, ny, precision):
    check(nx, ny, precision)
