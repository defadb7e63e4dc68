"""Where the t-marching form is the default (tests: a t extent that does not pay, chunks of unequal length
below and above their bound, a launch that ends in a nearly empty round, large lattices, 16-bit links);
chunks of unequal length give the bits of the other forms."""
import pytest

from tests.test_gpu_march import CDT
from tests.test_gpu_march_faces import field, use
from tests.test_gpu_parity import ovl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# (dims, right-hand sides, order by default)
@pytest.mark.parametrize("store,dims,nrhs,order", [
    ("f64", (16, 16, 16, 2), 60, 1), ("f32", (16, 16, 16, 1), 240, 1), ("bf16", (16, 16, 16, 2), 121, 3),
    ("f64", (16, 16, 16, 5), 29, 3), ("f64", (16, 16, 16, 17), 8, 1), ("f64", (16, 16, 16, 17), 11, 3),
    ("f32", (16, 16, 16, 33), 11, 1), ("f32", (16, 16, 16, 33), 15, 3), ("f64", (16, 4, 4, 8), 400, 1),
    ("f64", (16, 4, 4, 8), 355, 3), ("f64", (16, 16, 16, 32), 2, 1), ("f64", (16, 16, 16, 32), 3, 3),
    ("f32", (16, 16, 16, 64), 3, 3), ("f32", (8, 8, 8, 16), 130, 1)])
def test_default(ovl, tmp_path, store, dims, nrhs, order):  # noqa: F811
    g = ovl.GaugeField(field(dims, 41), store)
    gen = torch.Generator(device="cuda").manual_seed(42)
    x = torch.randn(nrhs, 4, 3, *reversed(dims), dtype=CDT[store], device="cuda", generator=gen)
    assert ovl.batch_launch_config((g, x))[1] == order
    w = x.flip(0).contiguous()
    got = ovl.kernel_axpby(g, x, 0.7, src=w, a=0.2, w=w, b=-1.0, out=torch.empty_like(x))
    for other in (1, 3):
        use(ovl, tmp_path, store, 0, other, (dims, nrhs))
        assert torch.equal(got, ovl.kernel_axpby(g, x, 0.7, src=w, a=0.2, w=w, b=-1.0, out=torch.empty_like(x)))
