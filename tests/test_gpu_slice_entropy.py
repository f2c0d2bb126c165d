"""hom4d_entanglement at the edges of its register blocks, against numpy's singular values.

Tolerance: the computed eigenvalues are those of rho + E, ||E||_F <= 10 m eps (||rho||_F <= 1;
10 for the products and the m reflectors' constant), so sum |d lambda| <= sqrt(m) ||E||_F
(Hoffman-Wielandt), and |d(lambda ln lambda)| <= (1 + |ln eps|) |d lambda| < 38 |d lambda|.
"""
import numpy as np
import pytest

from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

NX, NY = 256, 4


def entropy(phi):
    sv = np.linalg.svd(phi / np.linalg.norm(phi), compute_uv=False)
    lam = sv ** 2 / np.sum(sv ** 2)
    lam = lam[lam > 0.0]
    return float(-np.sum(lam * np.log(lam)))


def tol(m):
    return 38.0 * np.sqrt(m) * 10.0 * m * np.finfo(float).eps


@pytest.fixture(scope="module")
def prop():
    from paper_1903_02581_amd import Propagator
    return Propagator(NX, NY, 100.0, 40.0, dt_fs=1.0, b_tesla=5.0)


def fill(p, phi, jy1, jy2):
    import torch
    psi = torch.zeros((NX, NY, NX, NY), dtype=torch.complex128)
    psi[:, jy1, :, jy2] = torch.from_numpy(phi)
    p.psi.copy_(psi.reshape(-1))


@pytest.mark.parametrize("n1,n2", [(1, 1), (1, 9), (2, 2), (3, 2), (31, 33), (32, 32), (33, 32), (48, 200), (64, 63),
                                   (64, 64), (65, 66), (96, 128), (128, 127), (128, 128), (129, 128), (129, 131),
                                   (160, 256), (256, 256), (256, 5)])
def test_sizes(prop, n1, n2):
    announce(f"slice entropy {n1}x{n2}")
    g = np.random.default_rng(n1 * 1000 + n2)
    full = g.normal(size=(NX, NX)) + 1j * g.normal(size=(NX, NX))
    # a smooth decaying spectrum, as of interacting electrons
    u, s, vh = np.linalg.svd(full)
    full = (u * np.exp(-0.3 * np.arange(NX))) @ vh + 1e-3 * full / np.linalg.norm(full)
    fill(prop, full, 1, 2)
    ix1, ix2 = g.permutation(NX)[:n1], g.permutation(NX)[:n2]
    got = prop.entanglement(ix1, 1, ix2, 2)
    ref = entropy(full[np.ix_(ix1, ix2)])
    assert abs(got - ref) <= tol(min(n1, n2)), (got, ref)
    assert got == prop.entanglement(ix1, 1, ix2, 2)


@pytest.mark.parametrize("n", [24, 64, 100, 192])
@pytest.mark.parametrize("kind", ["product", "two terms", "zeros", "tiny", "repeated"])
def test_special_slices(prop, n, kind):
    announce(f"slice entropy {kind} {n}")
    g = np.random.default_rng(n)
    a, b = (g.normal(size=NX) + 1j * g.normal(size=NX) for _ in range(2))
    phi = np.outer(a, b)
    ix = np.arange(n)
    if kind == "two terms":  # equal weights on disjoint supports: ln 2
        half = np.arange(NX) < n // 2
        a[n:] = b[n:] = 0.0
        phi = sum(np.outer(a * h, b * h) / (np.linalg.norm(a * h) * np.linalg.norm(b * h)) for h in (half, ~half))
    elif kind == "zeros":  # most of the slice exactly zero
        phi = np.zeros((NX, NX), complex)
        phi[3:9, 5:15] = g.normal(size=(6, 10))
    elif kind == "tiny":  # squares near the end of the number range
        phi = 1e-150 * (g.normal(size=(NX, NX)) + 1j * g.normal(size=(NX, NX)))
    elif kind == "repeated":  # the same grid rows several times
        phi = g.normal(size=(NX, NX)) + 1j * g.normal(size=(NX, NX))
        ix = np.arange(n) % 7
    fill(prop, phi, 0, 3)
    got = prop.entanglement(ix, 0, ix, 3)
    ref = entropy(phi[np.ix_(ix, ix)] * (1e150 if kind == "tiny" else 1.0))
    assert abs(got - ref) <= tol(n), (got, ref)


def test_no_slice(prop):
    from paper_1903_02581_amd import Hom4dError
    for bad in (0.0, np.nan, np.inf):
        announce(f"slice of {bad}")
        fill(prop, np.full((NX, NX), bad, complex), 0, 0)
        with pytest.raises(Hom4dError) as e:
            prop.entanglement(np.arange(40), 0, np.arange(40), 0)
        assert e.value.status == -6
