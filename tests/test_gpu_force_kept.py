"""The force without a checkpoint stride (all forward Chebyshev vectors kept): one launch of pairs, several
launches with ragged ends, and a ring of Clenshaw vectors that wraps, against the FP64 oracle and against
the checkpointed sweep of the same call.  The two sweeps add the same products in another grouping (FP64
sums): 1e-13 (FP64) and 1e-7 (one FP32 rounding of the result) relative."""
import numpy as np
import pytest

import latgen
from oracle import chebyshev as och
from oracle import force as oforce
from tests.conftest import rel_err
from tests.test_gpu_parity import LMAX, dev, host, ovl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store,cdt,tol,same", [("f64", torch.complex128, 1e-12, 1e-13),
                                                ("f32", torch.complex64, 1e-6, 1e-7)])
@pytest.mark.parametrize("degree", [1, 3, 63, 65, 131, 199])
def test_force_all_vectors_kept(ovl, store, cdt, tol, same, degree):  # noqa: F811
    dims = (4, 2, 3, 4)
    u = latgen.smeared_field(dims, 10220, steps=1)
    chi, psi = latgen.gaussian_spinor(dims, 20220), latgen.gaussian_spinor(dims, 20221)
    alpha = och.coeffs_sign_interp(degree, 0.1)
    g, p = ovl.GaugeField(dev(u), store), ovl.Polynomial(alpha, LMAX)
    kept = host(ovl.sign_force(g, p, dev(chi, cdt), dev(psi, cdt)))
    swept = host(ovl.sign_force(g, p, dev(chi, cdt), dev(psi, cdt), ckpt_stride=7))
    if store == "f32":
        u, chi, psi = (latgen.round_to_f32(a) for a in (u, chi, psi))
    assert rel_err(kept, oforce.sign_force(u, chi, psi, alpha, LMAX)) < tol
    assert rel_err(kept, swept) < same
