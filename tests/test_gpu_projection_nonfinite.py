"""Projection of several right-hand sides with infinite entries: the infinite coefficients are infinite and
not NaN, NaN stays with its own right-hand side, and the finite ones are the oracle's (1e-13 of the largest;
FP32 storage 1e-6)."""
import numpy as np
import pytest

from tests.test_gpu_parity import ovl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store,dt,tol", [("f64", torch.complex128, 1e-13), ("f32", torch.complex64, 1e-6)])
def test_projection_nonfinite(ovl, store, dt, tol):  # noqa: F811
    gen = torch.Generator().manual_seed(7)
    shape = (4, 3, 4, 4, 4, 4)
    # real vectors of disjoint support are orthogonal exactly; an entry of one meets no other's product
    phi = torch.zeros((2,) + shape, dtype=torch.complex128)
    phi[0, :, :, :2], phi[1, :, :, 2:] = 1.0, 1.0
    psi = torch.randn((4,) + shape, dtype=torch.complex128, generator=gen).to(dt)
    want = (phi.flatten(1).conj() @ psi.to(torch.complex128).flatten(1).T).T.numpy() / np.sqrt(4 * 3 * 128)
    psi.view(torch.float32 if store == "f32" else torch.float64).view(4, 4, 3, 4, 4, 4, 4, 2)[1, 0, 0, 0, 0, 0, 0, 0] = np.inf
    psi[2, 3, 2, 3, 3, 3, 3] = complex(np.nan, np.nan)
    d = ovl.Deflation(phi.cuda().to(dt), np.array([0.1, 0.2]), store)
    c = ovl.defl_project(d, psi.cuda()).cpu().numpy()
    assert c[1, 0].real == np.inf
    assert np.isnan(c[2, 1])
    fine = np.ones((4, 2), dtype=bool)
    fine[1], fine[2] = False, False
    assert np.abs(c - want)[fine].max() < tol * np.abs(want).max()
