"""The default workgroup order of 16-bit links: memory order below 120 MB of vectors and links, tiles from
there on; both add the same terms in the same order, so the result of either is bitwise that of the order
forced through a tuning-cache entry."""
import pytest

from tests.test_gpu_parity import ovl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store,nrhs,order", [("bf16", 1, 0), ("bf16", 2, 0), ("bf16", 3, 1), ("f32", 1, 1)])
def test_default_order(ovl, tmp_path, store, nrhs, order):  # noqa: F811
    dims = (16, 16, 16, 32)
    torch.manual_seed(3)
    u = torch.linalg.qr(torch.randn((4, 32, 16, 16, 16, 3, 3), dtype=torch.complex128, device="cuda"))[0]
    g = ovl.GaugeField(u.permute(0, 5, 6, 1, 2, 3, 4).contiguous(), store)
    x = torch.randn((nrhs, 4, 3, 32, 16, 16, 16), dtype=torch.complex64, device="cuda")
    p = ovl.Polynomial(ovl.cheb_sign_coeffs(5, 0.1), 6.6)
    assert ovl.batch_launch_config((g, x)) == (64, order, 1, 1)
    got = ovl.sign_apply(g, p, x)
    cache = tmp_path / "order.txt"
    cache.write_text("B %d 0 1 16 16 16 32 %d 64 %d 1 1 0\n" % (1 if store == "f32" else 2, nrhs, 1 - order))
    assert ovl.autotune_load(str(cache)) == 1
    assert ovl.batch_launch_config((g, x)) == (64, 1 - order, 1, 1)
    assert torch.equal(got, ovl.sign_apply(g, p, x))
