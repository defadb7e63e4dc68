"""memory_release gives what the library keeps back to the device, and calls after it give the results they
gave before."""
import pytest

import latgen
from oracle import chebyshev as och
from tests.test_gpu_parity import LMAX, dev, ovl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_memory_release(ovl):  # noqa: F811
    dims = (8, 8, 8, 8)
    u = dev(latgen.random_su3_field(dims, 10430))
    g, p = ovl.GaugeField(u, "f64"), ovl.Polynomial(och.coeffs_sign_interp(63, 0.1), LMAX)
    a, b = dev(latgen.gaussian_spinor(dims, 20430)), dev(latgen.gaussian_spinor(dims, 20431))
    ovl.memory_release()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    want = ovl.sign_force(g, p, a, b)    # 129 vectors of 0.8 MB
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] < before - (90 << 20)
    ovl.memory_release()
    assert torch.cuda.mem_get_info()[0] > before - (24 << 20)    # the result, in a segment of torch's
    assert torch.equal(ovl.sign_force(g, p, a, b), want)
