"""The small-problem form of the plain steps (8 and 16 sites per workgroup of one problem), each forced
through a tuning-cache entry, against the FP64 oracle: ragged and odd extents, extent 1, a last workgroup
that is partly empty, 16 right-hand sides (the last of one group) and 17 (the general form), operands in
place, two-row links.  Tolerances are those of the other launch forms (1e-13 FP64; 1e-6 FP32 and 16-bit
links against the oracle on the same rounded inputs)."""
import pytest

import latgen
from oracle import wilson as ow
from tests.conftest import complete_third_row
from tests.test_gpu_march import CDT, PREC, seen
from tests.test_gpu_parity import dev, host, max_rel, ovl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [((4, 4, 4, 4), 1), ((5, 3, 7, 3), 2), ((1, 2, 3, 1), 1), ((3, 1, 1, 5), 16), ((2, 3, 2, 3), 17),
         ((11, 7, 9, 13), 3)]


@pytest.mark.parametrize("dims,nrhs", CASES)
@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("spb", [8, 16])
@pytest.mark.parametrize("two_row", [False, True])
def test_small_steps(ovl, tmp_path, store, dims, nrhs, spb, two_row):  # noqa: F811
    cache = tmp_path / "small.txt"
    cache.write_text("B %d %d 1 %d %d %d %d %d %d 0 1 1 0\n" % (PREC[store], two_row, *dims, nrhs, spb))
    assert ovl.autotune_load(str(cache)) == 1
    u = latgen.random_su3_field(dims, 10310, noise=0.5)
    psi, src, w = (latgen.gaussian_spinor(dims, 20310 + i, nrhs=nrhs) for i in range(3))
    g = ovl.GaugeField(dev(u), store)
    if two_row:
        g.reconstruct()
    x = dev(psi, CDT[store])
    assert ovl.batch_launch_config((g, x))[0] == spb
    u_r = seen(u, store)
    if two_row:
        u_r = complete_third_row(u_r)
    psi_r, src_r, w_r = (a if store == "f64" else latgen.round_to_f32(a) for a in (psi, src, w))
    tol = 1e-13 if store == "f64" else 1e-6
    k = host(ovl.kernel_apply(g, x))
    dag = host(ovl.wilson_apply(g, x, m_w=1.5, dagger=True))
    on_w, on_src = dev(w, CDT[store]), dev(src, CDT[store])
    ovl.kernel_axpby(g, x, 0.7, src=on_src, a=-0.3, w=on_w, b=1.1, out=on_w)
    ovl.kernel_axpby(g, x, 0.7, src=on_src, a=-0.3, out=on_src)
    on_w, on_src = host(on_w), host(on_src)
    for r in range(nrhs):
        ref = ow.kop(u_r, psi_r[r])
        assert max_rel(k[r], ref) < tol
        assert max_rel(dag[r], ow.gamma5(ow.dw_minus_mass(u_r, ow.gamma5(psi_r[r]), 1.5))) < tol
        assert max_rel(on_w[r], 0.7 * ref - 0.3 * src_r[r] + 1.1 * w_r[r]) < tol
        assert max_rel(on_src[r], 0.7 * ref - 0.3 * src_r[r]) < tol
