"""The t-marching form of the plain steps (order 3), forced through a tuning-cache entry on small
lattices, against the FP64 oracle: tiles with faces in y and z, in one of them, and none (the tile
wraps), tiles of fewer than 256 sites, chunks of t that end ragged, extent-1 and extent-2 t, right-hand
sides in several groups, gamma5 on the input, the operands of the fused step, two-row links, batches of
different tiles and the force's twin steps.  Tolerances are those of the other launch forms (1e-13 /
1e-12 FP64, 1e-6 FP32 and 16-bit links against the oracle on the same rounded inputs)."""
import numpy as np
import pytest

import latgen
from oracle import chebyshev as och
from oracle import force as oforce
from oracle import overlap as oov
from oracle import wilson as ow
from tests.conftest import complete_third_row, rel_err
from tests.test_gpu_parity import LMAX, dev, host, max_rel, ovl, random_basis  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PREC = {"f64": 0, "f32": 1, "bf16": 2}
CDT = {"f64": torch.complex128, "f32": torch.complex64, "bf16": torch.complex64}


def force_form(ovl, tmp_path, store, r12, *problems):  # noqa: F811
    cache = tmp_path / "march.txt"
    items = " ".join(" ".join(map(str, d)) + f" {n}" for d, n in problems)
    cache.write_text(f"B {PREC[store]} {r12} {len(problems)} {items} 64 3 1 1 0\n")
    assert ovl.autotune_load(str(cache)) == 1


def seen(a, store):
    return {"f64": lambda x: x, "f32": latgen.round_to_f32, "bf16": latgen.round_to_bf16}[store](a)


# (dims, nrhs): 16 x 4 x 4 and 8 x 8 x 4 tiles with faces, 12 x 4 x 4 (192 sites), tiles that wrap in y
# or in both, t extents 1, 2 and ragged chunks (5, 6, 9), 40 right-hand sides of one tile (two groups)
CASES = [((16, 8, 8, 6), 2), ((8, 16, 8, 5), 1), ((12, 8, 8, 3), 1), ((16, 4, 8, 9), 3),
         ((8, 8, 4, 4), 40), ((4, 4, 4, 1), 2), ((64, 2, 2, 2), 1)]


@pytest.mark.parametrize("dims,nrhs", CASES)
@pytest.mark.parametrize("store", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("two_row", [False, True])
def test_march_kernel(ovl, tmp_path, store, dims, nrhs, two_row):  # noqa: F811
    force_form(ovl, tmp_path, store, int(two_row), (dims, nrhs))
    u = latgen.random_su3_field(dims, 10210, noise=0.5)
    psi, src, w = (latgen.gaussian_spinor(dims, 20210 + i, nrhs=nrhs) for i in range(3))
    g = ovl.GaugeField(dev(u), store)
    if two_row:
        g.reconstruct()
    x = dev(psi, CDT[store])
    assert ovl.batch_launch_config((g, x)) == (64, 3, 1, 1)
    u_r = seen(u, store)
    if two_row:
        u_r = complete_third_row(u_r)
    psi_r, src_r, w_r = (a if store == "f64" else latgen.round_to_f32(a) for a in (psi, src, w))
    tol = 1e-13 if store == "f64" else 1e-6
    k = host(ovl.kernel_apply(g, x))
    dag = host(ovl.wilson_apply(g, x, m_w=1.5, dagger=True))
    out = dev(w, CDT[store])
    ovl.kernel_axpby(g, x, 0.7, src=dev(src, CDT[store]), a=-0.3, w=out, b=1.1, out=out)
    out = host(out)
    for r in range(nrhs):
        ref = ow.kop(u_r, psi_r[r])
        assert max_rel(k[r], ref) < tol
        ref_dag = ow.gamma5(ow.dw_minus_mass(u_r, ow.gamma5(psi_r[r]), 1.5))
        assert max_rel(dag[r], ref_dag) < tol
        assert max_rel(out[r], 0.7 * ref - 0.3 * src_r[r] + 1.1 * w_r[r]) < tol


@pytest.mark.parametrize("store", ["f64", "f32"])
def test_march_overlap_and_batch(ovl, tmp_path, store):  # noqa: F811
    """D and D^+ with deflated modes (the final step runs in tiles), and a batch of two lattices whose
    tiles differ."""
    dims, nrhs, tol = (16, 8, 4, 6), 2, 1e-12 if store == "f64" else 1e-6
    force_form(ovl, tmp_path, store, 0, (dims, nrhs))
    u = latgen.smeared_field(dims, 10211, steps=1)
    psi = latgen.gaussian_spinor(dims, 20211, nrhs=nrhs)
    phi, lam = random_basis(dims, 3, 20212)
    alpha = och.coeffs_sign_interp(11, 0.1)
    g = ovl.GaugeField(dev(u), store)
    p = ovl.Polynomial(alpha, LMAX)
    d = ovl.Deflation(dev(phi), lam, store)
    x = dev(psi, CDT[store])
    s, o = host(ovl.sign_apply(g, p, x, defl=d)), host(ovl.overlap_apply(g, p, x, 0.05, defl=d, dagger=True))
    for r in range(nrhs):
        assert rel_err(s[r], och.sign_apply(u, psi[r], alpha, LMAX, phi, lam)) < tol
        assert rel_err(o[r], oov.overlap_dagger_apply(u, psi[r], 0.05, alpha, LMAX, phi, lam)) < tol
    dims2 = (12, 4, 8, 5)
    force_form(ovl, tmp_path, store, 0, (dims, nrhs), (dims2, 1))
    u2, psi2 = latgen.smeared_field(dims2, 10213, steps=1), latgen.gaussian_spinor(dims2, 20213)
    probs = [(g, x), (ovl.GaugeField(dev(u2), store), dev(psi2, CDT[store]))]
    assert ovl.batch_launch_config(probs) == (64, 3, 1, 1)
    a, b = ovl.batch_sign_apply(p, probs)
    for r in range(nrhs):
        assert rel_err(host(a)[r], och.poly_apply(u, psi[r], alpha, LMAX)) < tol
    assert rel_err(host(b), och.poly_apply(u2, psi2, alpha, LMAX)) < tol
    assert g.flags() == 0


@pytest.mark.parametrize("store", ["f64", "f32"])
def test_march_force_twins(ovl, tmp_path, store):  # noqa: F811
    dims = (8, 8, 4, 6)
    for n in (1, 2):
        force_form(ovl, tmp_path, store, 0, (dims, n))
    u = latgen.smeared_field(dims, 10214, steps=1)
    chi, psi = latgen.gaussian_spinor(dims, 20214), latgen.gaussian_spinor(dims, 20215)
    alpha = och.coeffs_sign_interp(17, 0.1)
    g = ovl.GaugeField(dev(u), store)
    got = host(ovl.sign_force(g, ovl.Polynomial(alpha, LMAX), dev(chi, CDT[store]), dev(psi, CDT[store]),
                              ckpt_stride=5))
    if store == "f32":
        u, chi, psi = (latgen.round_to_f32(a) for a in (u, chi, psi))
    ref = oforce.sign_force(u, chi, psi, alpha, LMAX)
    assert (max_rel(got, ref) < 1e-12) if store == "f64" else (rel_err(got, ref) < 1e-6)


def test_march_falls_back(ovl, tmp_path):  # noqa: F811
    """No tile fits (odd cross-section): the entry is ignored."""
    dims = (5, 3, 4, 6)
    force_form(ovl, tmp_path, "f64", 0, (dims, 1))
    u, psi = latgen.random_su3_field(dims, 10216), latgen.gaussian_spinor(dims, 20216)
    g = ovl.GaugeField(dev(u), "f64")
    assert ovl.launch_config(g, 1)[1] != 3
    assert max_rel(host(ovl.kernel_apply(g, dev(psi))), ow.kop(u, psi)) < 1e-13
