"""The t-marching form on tiles with more face sites than sites, against the FP64 oracle and, bit for bit,
against the 64-site form of the same problem; and a batch that takes the form by default with such a
lattice among its items, bit for bit against the items run alone.  Tolerances are those of the other
launch forms (1e-13 FP64; 1e-6 FP32 and 16-bit links against the oracle on the same rounded inputs)."""
import numpy as np
import pytest

import latgen
from oracle import chebyshev as och
from oracle import force as oforce
from oracle import wilson as ow
from tests.conftest import complete_third_row, rel_err
from tests.test_gpu_march import CDT, PREC, seen
from tests.test_gpu_parity import LMAX, dev, host, max_rel, ovl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def use(ovl, tmp_path, store, r12, order, *problems):  # noqa: F811
    cache = tmp_path / "form.txt"
    items = " ".join(" ".join(map(str, d)) + f" {n}" for d, n in problems)
    cache.write_text(f"B {PREC[store]} {r12} {len(problems)} {items} 64 {order} 1 1 0\n")
    assert ovl.autotune_load(str(cache)) == 1


# (dims, nrhs) with tile sites / face sites: 64/128, 64/128 (z faces), 64/128 (y faces), 192/240, 128/256,
# 64/256; t extents 1 and 2 and ragged chunks among them
FACES = [((16, 10, 10, 4), 2), ((8, 5, 8, 3), 1), ((8, 8, 5, 9), 1), ((12, 14, 16, 2), 1),
         ((32, 8, 8, 3), 3), ((64, 5, 5, 1), 1)]
# and tiles with no more faces than sites
PLAIN = [((16, 8, 8, 6), 2), ((8, 8, 4, 4), 40)]


@pytest.mark.parametrize("dims,nrhs", FACES + PLAIN)
@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("two_row", [False, True])
def test_march_faces(ovl, tmp_path, store, dims, nrhs, two_row):  # noqa: F811
    u = latgen.random_su3_field(dims, 10410, noise=0.5)
    psi, src, w = (latgen.gaussian_spinor(dims, 20410 + i, nrhs=nrhs) for i in range(3))
    g = ovl.GaugeField(dev(u), store)
    if two_row:
        g.reconstruct()
    x = dev(psi, CDT[store])
    out = {}
    for order in (1, 3):
        use(ovl, tmp_path, store, int(two_row), order, (dims, nrhs))
        assert ovl.batch_launch_config((g, x)) == (64, order, 1, 1)
        y = dev(w, CDT[store])
        ovl.kernel_axpby(g, x, 0.7, src=dev(src, CDT[store]), a=-0.3, w=y, b=1.1, out=y)
        out[order] = (ovl.kernel_apply(g, x), ovl.wilson_apply(g, x, m_w=1.5, dagger=True), y)
    for a, b in zip(out[1], out[3]):
        assert torch.equal(a, b)
    u_r = seen(u, store)
    if two_row:
        u_r = complete_third_row(u_r)
    psi_r, src_r, w_r = (a if store == "f64" else latgen.round_to_f32(a) for a in (psi, src, w))
    tol = 1e-13 if store == "f64" else 1e-6
    k, dag, y = map(host, out[3])
    for r in range(min(nrhs, 3)):
        ref = ow.kop(u_r, psi_r[r])
        assert max_rel(k[r], ref) < tol
        assert max_rel(dag[r], ow.gamma5(ow.dw_minus_mass(u_r, ow.gamma5(psi_r[r]), 1.5))) < tol
        assert max_rel(y[r], 0.7 * ref - 0.3 * src_r[r] + 1.1 * w_r[r]) < tol


@pytest.mark.parametrize("store", ["f64", "f32"])
def test_march_faces_force_twins(ovl, tmp_path, store):  # noqa: F811
    dims = (8, 5, 8, 6)
    for n in (1, 2):
        use(ovl, tmp_path, store, 0, 3, (dims, n))
    u = latgen.smeared_field(dims, 10414, steps=1)
    chi, psi = latgen.gaussian_spinor(dims, 20414), latgen.gaussian_spinor(dims, 20415)
    alpha = och.coeffs_sign_interp(17, 0.1)
    got = host(ovl.sign_force(ovl.GaugeField(dev(u), store), ovl.Polynomial(alpha, LMAX),
                              dev(chi, CDT[store]), dev(psi, CDT[store]), ckpt_stride=5))
    if store == "f32":
        u, chi, psi = (latgen.round_to_f32(a) for a in (u, chi, psi))
    ref = oforce.sign_force(u, chi, psi, alpha, LMAX)
    assert (max_rel(got, ref) < 1e-12) if store == "f64" else (rel_err(got, ref) < 1e-6)


def field(dims, seed):
    """Special unitary links made on the GPU: two orthonormal rows and the conjugate of their cross product."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    a, b = torch.randn(2, 4, dims[0] * dims[1] * dims[2] * dims[3], 3, dtype=torch.complex128, device="cuda",
                       generator=gen)
    a = a / a.norm(dim=-1, keepdim=True)
    b = b - a * (a.conj() * b).sum(-1, keepdim=True)
    b = b / b.norm(dim=-1, keepdim=True)
    c = torch.stack([a[..., 1] * b[..., 2] - a[..., 2] * b[..., 1], a[..., 2] * b[..., 0] - a[..., 0] * b[..., 2],
                     a[..., 0] * b[..., 1] - a[..., 1] * b[..., 0]], dim=-1).conj()
    return torch.stack([a, b, c], dim=-2).permute(0, 2, 3, 1).reshape(4, 3, 3, *reversed(dims)).contiguous()


@pytest.mark.parametrize("store,other", [("f64", (12, 14, 16, 4)), ("f32", (16, 10, 10, 6)),
                                         ("bf16", (32, 16, 8, 3))])
def test_march_by_default_in_a_batch(ovl, store, other):  # noqa: F811
    """Most sites in 256-site tiles and a working set beyond the last-level cache: the form is the default
    of the whole batch, a lattice with more face sites than tile sites among it."""
    p = ovl.Polynomial(och.coeffs_sign_interp(11, 0.1), LMAX)
    gen = torch.Generator(device="cuda").manual_seed(7)
    probs = []
    for i, (dims, n) in enumerate([((16, 16, 16, 32), 4 if store == "f64" else 8), (other, 2)]):
        x = torch.randn(n, 4, 3, *reversed(dims), dtype=CDT[store], device="cuda", generator=gen)
        probs.append((ovl.GaugeField(field(dims, 30 + i), store), x))
    assert ovl.batch_launch_config(probs) == (64, 3, 1, 1)
    for (g, x), y in zip(probs, ovl.batch_sign_apply(p, probs)):
        assert torch.equal(y, ovl.sign_apply(g, p, x))
