"""The default workgroup order of 16-bit links follows the size of a t slice's links, input and output:
memory order within 2.6 MB, tiles beyond, on either side of the line in the lattice and in the right-hand
sides; tiles give the bits of memory order."""
import pytest

from tests.test_gpu_march import CDT
from tests.test_gpu_march_faces import field, use
from tests.test_gpu_parity import ovl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# a slice is (144 + 192 n) bytes a site, n of up to 16 right-hand sides together, else 4
@pytest.mark.parametrize("dims,nrhs,order", [
    ((20, 20, 20, 8), 1, 0),     # 2.56 MB
    ((32, 16, 16, 8), 1, 1),     # 2.63
    ((16, 16, 16, 8), 2, 0),     # 2.06
    ((16, 16, 16, 8), 3, 1),     # 2.81
    ((8, 8, 8, 8), 16, 0),       # 1.57
    ((12, 12, 12, 4), 8, 1),     # 2.77
    ((12, 12, 12, 2), 17, 0)])   # 1.50 of 4 together
def test_default(ovl, tmp_path, dims, nrhs, order):  # noqa: F811
    g = ovl.GaugeField(field(dims, 43), "bf16")
    gen = torch.Generator(device="cuda").manual_seed(44)
    x = torch.randn(nrhs, 4, 3, *reversed(dims), dtype=CDT["bf16"], device="cuda", generator=gen)
    assert ovl.batch_launch_config((g, x))[1] == order
    got = ovl.kernel_apply(g, x)
    use(ovl, tmp_path, "bf16", 0, 1 - order, (dims, nrhs))
    assert torch.equal(got, ovl.kernel_apply(g, x))
