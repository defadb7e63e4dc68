"""Work space and link memory kept between calls: two streams whose calls overlap use different blocks,
handles made from returned blocks start clean, and a loop that makes and drops handles of changing sizes
stays within bounds."""
import numpy as np
import pytest

import latgen
from oracle import wilson as ow
from oracle import chebyshev as och
from tests.test_gpu_parity import LMAX, dev, host, max_rel, ovl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_overlapping_streams(ovl):  # noqa: F811
    """Forces (more than 16 MB of work space each) on two streams, four calls on each without a wait."""
    dims = (8, 8, 8, 8)
    u = latgen.random_su3_field(dims, 10230)
    p = ovl.Polynomial(och.coeffs_sign_interp(31, 0.1), LMAX)
    g = ovl.GaugeField(dev(u), "f64")
    vecs = [dev(latgen.gaussian_spinor(dims, 20230 + i)) for i in range(9)]
    want = [ovl.sign_force(g, p, vecs[i], vecs[i + 1]).clone() for i in range(8)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = [torch.empty_like(want[0]) for _ in range(8)]
    for i in range(8):
        with torch.cuda.stream(streams[i % 2]):
            ovl.sign_force(g, p, vecs[i], vecs[i + 1], out=got[i])
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def test_handles_from_returned_blocks(ovl):  # noqa: F811
    dims = (4, 4, 4, 6)
    psi = latgen.gaussian_spinor(dims, 20240)
    for i in range(4):
        u = latgen.random_su3_field(dims, 10240 + i, noise=0.5)
        g = ovl.GaugeField(dev(u), "f64")
        assert g.flags(clear=False) == 0
        assert max_rel(host(ovl.kernel_apply(g, dev(psi))), ow.kop(u, psi)) < 1e-13
        bad = psi.copy()
        bad[0, 0, 0, 0, 0, 0] = np.nan
        ovl.sign_apply(g, ovl.Polynomial(och.coeffs_sign_interp(5, 0.3), LMAX), dev(bad))
        assert g.flags(clear=False) != 0     # raised, left set, handle dropped
        del g


def test_handle_loop_is_bounded(ovl):  # noqa: F811
    u = torch.zeros((4, 3, 3, 8, 8, 8, 16), dtype=torch.complex128, device="cuda")
    for a in range(3):
        u[:, a, a] = 1
    free = []
    for i in range(60):
        t = 4 + i % 5
        g = ovl.GaugeField(u[:, :, :, :t].contiguous(), "f64")
        ovl.stout_smear(u[:, :, :, :t].contiguous())
        del g
        free.append(torch.cuda.mem_get_info()[0])
    assert free[-1] >= free[9] - (64 << 20)
