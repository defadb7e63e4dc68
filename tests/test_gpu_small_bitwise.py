"""The small-problem form of the plain steps gives the bits of the general form: 16 right-hand sides take it,
17 take the general kernel of the same shape, whose first 16 results are compared."""
import pytest

import latgen
from tests.test_gpu_march import CDT, PREC
from tests.test_gpu_parity import dev, ovl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(5, 3, 7, 3), (4, 4, 4, 4), (3, 1, 1, 5)])
@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("spb", [8, 16])
@pytest.mark.parametrize("two_row", [False, True])
def test_small_bits(ovl, tmp_path, store, dims, spb, two_row):  # noqa: F811
    cache = tmp_path / "small.txt"
    cache.write_text("".join("B %d %d 1 %d %d %d %d %d %d 0 1 1 0\n" % (PREC[store], two_row, *dims, n, spb)
                             for n in (16, 17)))
    assert ovl.autotune_load(str(cache)) == 2
    g = ovl.GaugeField(dev(latgen.random_su3_field(dims, 10440, noise=0.5)), store)
    if two_row:
        g.reconstruct()
    x, src, w = (dev(latgen.gaussian_spinor(dims, 20440 + i, nrhs=17), CDT[store]) for i in range(3))
    got = []
    for n in (16, 17):
        assert ovl.batch_launch_config((g, x[:n]))[0] == spb
        y = w[:n].clone()
        ovl.kernel_axpby(g, x[:n], 0.7, src=src[:n], a=-0.3, w=y, b=1.1, out=y)
        got.append((y[:16], ovl.kernel_apply(g, x[:n])[:16], ovl.wilson_apply(g, x[:n], m_w=1.5, dagger=True)[:16]))
    for a, b in zip(*got):
        assert torch.equal(a, b)
