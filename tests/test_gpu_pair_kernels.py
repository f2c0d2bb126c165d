"""The reductions and the initial state over all pairs (r1, r2) at the edges of their
chunks: fewer pairs than one access per thread, exactly one chunk, a partial last chunk,
several chunks, both storages.

Tolerance: a thread adds at most a few hundred positive terms in turn and the blocks'
sums are trees, so the relative error stays below 500 eps = 1.1e-13.
"""
import numpy as np
import pytest

from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

TOL = 500 * np.finfo(float).eps
SIZES = [(4, 4), (6, 8), (16, 16), (32, 32), (48, 24), (64, 32), (48, 48), (8, 256), (24, 128)]


def orbitals(nx, ny, seed):
    g = np.random.default_rng(seed)
    return [g.normal(size=(nx, ny)) + 1j * g.normal(size=(nx, ny)) for _ in range(2)], g.uniform(0.0, 1.0, (nx, ny))


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_init_and_observables(nx, ny, precision):
    from paper_1903_02581_amd import Propagator
    announce(f"pair kernels {nx}x{ny} {precision}")
    (a, b), w = orbitals(nx, ny, nx * 1000 + ny)
    p = Propagator(nx, ny, 10.0 * nx, 8.0 * ny, dt_fs=1.0, b_tesla=5.0, precision=precision)
    for sym in (-1, 0, 1):
        p.init_state(a, b, sym)
        ref = np.outer(a, b) + (sym * np.outer(b, a) if sym else 0.0)
        ref /= np.sqrt(np.sum(np.abs(ref) ** 2))
        got = p.psi.cpu().numpy().reshape(ref.shape)
        # the pair product, the norm and, in complex64, one rounding to storage
        eps = TOL if precision == "fp64" else np.finfo(np.float32).eps
        assert np.max(np.abs(got - ref)) <= eps * np.max(np.abs(ref))
        d = np.abs(got.astype(np.complex128)) ** 2
        w1, w2 = w.reshape(-1, 1), w.reshape(1, -1)
        o = p.observables(w)
        for key, m in (("norm", 1.0), ("p_tt", w1 * w2), ("p_tb", w1 * (1 - w2)), ("p_bt", (1 - w1) * w2),
                       ("p_bb", (1 - w1) * (1 - w2))):
            assert abs(o[key] - np.sum(m * d)) <= TOL * np.sum(m * d), key
    with pytest.raises(Exception):
        p.init_state(a, a, -1)


@pytest.mark.parametrize("nx,ny", [(8, 12), (32, 32), (64, 48)])
def test_reverse_sweep_loss_and_finish(nx, ny):
    """A recording of no steps: the loss is the weighted sum, and there is no gradient."""
    from paper_1903_02581_amd import Propagator
    announce(f"empty recording {nx}x{ny}")
    (a, b), w = orbitals(nx, ny, 7)
    p = Propagator(nx, ny, 10.0 * nx, 8.0 * ny, dt_fs=1.0, b_tesla=5.0)
    p.set_potential(np.zeros((nx, ny)))
    p.init_state(a, b, 0)
    p.grad_begin(1, 0)
    loss, dv, db = p.grad_backward(w, (0.3, -0.2, 0.7, 1.1))
    d = np.abs(p.psi.cpu().numpy().reshape(nx * ny, -1)) ** 2
    w1, w2 = w.reshape(-1, 1), w.reshape(1, -1)
    terms = (0.3 * w1 * w2 - 0.2 * w1 * (1 - w2) + 0.7 * (1 - w1) * w2 + 1.1 * (1 - w1) * (1 - w2)) * d
    assert abs(loss - np.sum(terms)) <= TOL * np.sum(np.abs(terms))
    assert not np.any(dv) and db == 0.0
