"""The correction kernel on both sides of the lines between its forms: 4 or 16 right-hand sides per thread
(few or many workgroups) and one or two FP32 components per thread (large lattices), with a last workgroup
that is not full, against the FP64 oracle.

Tolerances: a sum of m + 1 terms rounded once each is within (m + 1) u of the sum of its terms' sizes;
with m <= 3 and the largest result as the scale, 1e-14 (FP64) and 2e-6 (FP32) hold with a wide margin."""
import numpy as np
import pytest

import latgen
from oracle import deflation as odefl
from tests.test_gpu_parity import dev, host, max_rel, ovl, random_basis  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store", ["f64", "f32"])
@pytest.mark.parametrize("dims,n_ev,nrhs", [
    ((1, 1, 1, 1), 1, 16),        # one site: 12 components
    ((15, 17, 9, 7), 3, 5),       # 753 workgroups: 4 a thread, the last pass with 1
    ((15, 17, 9, 7), 2, 17),      # twice 753: 16 a thread, the last pass with 1
    ((15, 17, 9, 8), 3, 16),      # 861 workgroups: 16 a thread
    ((17, 19, 15, 18), 2, 4),     # 4088 workgroups: one component a thread
    ((18, 19, 15, 18), 2, 1),     # 4329 workgroups: two FP32 components a thread
    ((18, 19, 15, 18), 2, 3),
])
def test_correction_forms(ovl, store, dims, n_ev, nrhs):  # noqa: F811
    phi, lam = random_basis(dims, n_ev, 71)
    psi = latgen.gaussian_spinor(dims, 72, nrhs=nrhs)
    rng = np.random.default_rng(73)
    c = rng.standard_normal((nrhs, n_ev)) + 1j * rng.standard_normal((nrhs, n_ev))
    w = np.linspace(-1.0, 2.0, n_ev)
    f32 = store == "f32"
    if f32:
        phi, psi = latgen.round_to_f32(phi), latgen.round_to_f32(psi)
    d = ovl.Deflation(dev(phi), lam, store)
    out = dev(psi, torch.complex64 if f32 else torch.complex128)
    ovl.defl_correct(d, out, dev(c), w)
    out = host(out)
    for r in range(nrhs):
        assert max_rel(out[r], odefl.correct(phi, psi[r], c[r], w)) < (2e-6 if f32 else 1e-14)
