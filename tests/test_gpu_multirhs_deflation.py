"""Deflation projection and correction of several right-hand sides against the FP64 oracle: partial
and several matrix-core tiles in both directions (16 vectors x 8 right-hand sides), more basis vectors
than one staging of coefficients (64), ragged right-hand-side passes (1, 4, 16), a volume that leaves
ragged chunks, and the gamma5 of the adjoint operator.

Tolerances: a sum of n terms rounded to unit roundoff u in any order is within n u sum|terms|; for
n = 12 V = 4320 random terms the typical error is sqrt(n) u relative to the largest projection, 1e-13
(FP64) and 1e-5 (FP32 sums of 16 products with FP64 running sums: 1e-6) hold with a wide margin."""
import numpy as np
import pytest

import latgen
from oracle import chebyshev as och
from oracle import deflation as odefl
from oracle import overlap as oov
from tests.test_gpu_parity import dev, host, max_rel, ovl, random_basis  # noqa: F401
from tests.conftest import rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DIMS = (5, 3, 4, 6)


@pytest.mark.parametrize("store", ["f64", "f32"])
@pytest.mark.parametrize("n_ev,nrhs", [(1, 2), (16, 8), (17, 9), (24, 12), (33, 17), (66, 5)])
def test_project_and_correct(ovl, store, n_ev, nrhs):  # noqa: F811
    phi, lam = random_basis(DIMS, n_ev, 61)
    psi = latgen.gaussian_spinor(DIMS, 62, nrhs=nrhs)
    f32 = store == "f32"
    cdt = torch.complex64 if f32 else torch.complex128
    tol = 1e-6 if f32 else 1e-13
    phi_r = latgen.round_to_f32(phi) if f32 else phi
    psi_r = latgen.round_to_f32(psi) if f32 else psi
    d = ovl.Deflation(dev(phi), lam, store)
    c = host(ovl.defl_project(d, dev(psi, cdt)))
    ref = np.stack([odefl.project(phi_r, psi_r[r]) for r in range(nrhs)])
    assert max_rel(c, ref) < tol
    w = np.linspace(-1.0, 2.0, n_ev)
    out = dev(psi, cdt)
    ovl.defl_correct(d, out, dev(ref), w)
    out = host(out)
    for r in range(nrhs):
        assert max_rel(out[r], odefl.correct(phi_r, psi_r[r], ref[r], w)) < tol


@pytest.mark.parametrize("nrhs", [2, 9])
def test_adjoint_projection_several_sources_fp64(ovl, nrhs):  # noqa: F811
    dims = (4, 4, 2, 4)
    u = latgen.smeared_field(dims, 34)
    psi = latgen.gaussian_spinor(dims, 63, nrhs=nrhs)
    phi, lam = random_basis(dims, 18, 64)
    alpha = och.coeffs_sign_interp(21, 0.08)
    g = ovl.GaugeField(dev(u), "f64")
    p = ovl.Polynomial(alpha, 6.5)
    d = ovl.Deflation(dev(phi), lam, "f64")
    o = host(ovl.overlap_apply(g, p, dev(psi), 0.05, defl=d, dagger=True))
    for r in range(nrhs):
        ref = oov.overlap_dagger_apply(u, psi[r], 0.05, alpha, 6.5, phi, lam)
        assert rel_err(o[r], ref) < 1e-12
