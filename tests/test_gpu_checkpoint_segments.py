"""A recorded run over several checkpoints in one call leaves each segment's state in its
checkpoint and starts the next one and the reverse sweep from there, without copies; the same
run in a call per segment copies.  State, loss and gradients are the same bits either way, on
each step plan (two, three and four passes, the plane in registers) and both storages, and the
sweep leaves the initial state.
"""
import numpy as np
import pytest

from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,precision", [(16, 16, "fp64"), (24, 12, "mixed"), (48, 48, "fp64"), (64, 48, "mixed"),
                                             (64, 64, "fp64"), (96, 16, "fp64"), (128, 8, "mixed"), (8, 256, "mixed"),
                                             (256, 8, "mixed"), (128, 64, "fp64")])
def test_segments_in_one_call(nx, ny, precision):
    import torch
    from paper_1903_02581_amd import Propagator
    announce(f"checkpoint segments {nx}x{ny} {precision}")
    g = np.random.default_rng(nx + 1000 * ny)
    a, b = (g.normal(size=(nx, ny)) + 1j * g.normal(size=(nx, ny)) for _ in range(2))
    v, w = g.uniform(-2.0, 5.0, (nx, ny)), g.uniform(0.0, 1.0, (nx, ny))
    p = Propagator(nx, ny, 10.0 * nx, 8.0 * ny, dt_fs=1.0, b_tesla=5.0, precision=precision)
    try:
        p.set_potential(v)
        p.init_state(a, b, -1)
        first = p.psi.clone()
        out = []
        for calls in ((5,), (2, 2, 1), (1, 3, 1), (4, 1)):
            p.psi.copy_(first)
            p.grad_begin(2, 5)
            for n in calls:
                p.step(n)
            psi = p.psi.clone()
            loss, dv, db = p.grad_backward(w)
            assert torch.equal(p.psi, first), calls
            out.append((psi, loss, dv, db))
        ref = out[1]
        assert torch.equal(out[0][0], ref[0]) and torch.equal(out[3][0], ref[0])
        for got in (out[0], out[3]):
            assert got[1] == ref[1] and np.array_equal(got[2], ref[2]) and got[3] == ref[3]
        # a call that ends inside a segment closes the state there, which only rounds elsewhere
        bar = 1e-12 if precision == "fp64" else 2e-5
        d = torch.linalg.vector_norm((out[2][0] - ref[0]).to(torch.complex128)).item()
        assert d <= bar * torch.linalg.vector_norm(ref[0].to(torch.complex128)).item()
    finally:
        p.close()


@pytest.mark.parametrize("nx,ny,precision", [(16, 16, "fp64"), (24, 12, "mixed"), (96, 16, "fp64")])
def test_pool_off_the_passes_alignment(nx, ny, precision):
    """Such a pool is served by copies, with the same results."""
    import torch
    from ctypes import c_void_p
    from paper_1903_02581_amd import Propagator
    announce(f"checkpoint pool off 16 bytes {nx}x{ny} {precision}")
    g = np.random.default_rng(nx + 1000 * ny)
    a, b = (g.normal(size=(nx, ny)) + 1j * g.normal(size=(nx, ny)) for _ in range(2))
    w = g.uniform(0.0, 1.0, (nx, ny))
    p = Propagator(nx, ny, 10.0 * nx, 8.0 * ny, dt_fs=1.0, b_tesla=5.0, precision=precision)
    try:
        p.set_potential(g.uniform(-2.0, 5.0, (nx, ny)))
        pool = torch.empty(3 * p.state_bytes + 8, dtype=torch.uint8, device=p.device)
        out = []
        for off in (0, 8):
            p.init_state(a, b, -1)
            first = p.psi.clone()
            p._check(p.lib.hom4d_grad_begin(p.h, 2, c_void_p(pool.data_ptr() + off), 3 * p.state_bytes), "grad_begin")
            p.step(5)
            psi = p.psi.clone()
            out.append((psi, p.grad_backward(w)))
            assert torch.equal(p.psi, first)
        assert torch.equal(out[0][0], out[1][0])
        (l0, v0, b0), (l1, v1, b1) = out[0][1], out[1][1]
        assert l0 == l1 and np.array_equal(v0, v1) and b0 == b1
    finally:
        p.close()
