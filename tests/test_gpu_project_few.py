"""Projections of several right-hand sides on a few modes in FP64: both sides of the lines between the
matrix-core kernel and the kernel with carried sums (lattice size; 1, 2, 4 or 6 modes), and the modes per
workgroup of the latter, with sites that do not fill the last workgroup, against long-double sums over the
basis as it is stored; non-finite entries stay where they are.

Tolerance: 12 V products summed in blocks; the error of a coefficient is within 200 u of the norm of its
products, the square root of their sum of squares, for the chains and trees of either kernel (u = 2^-53)."""
import numpy as np
import pytest

from tests.test_gpu_parity import ovl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# small and large lattice by (modes, right-hand sides): 2 and 12 sides of one mode, the others
SITES = {(1, 2): ((13, 12, 20, 21), (13, 12, 21, 21)), (1, 12): ((13, 12, 7, 9), (13, 12, 7, 11))}
MORE = ((13, 12, 16, 19), (13, 12, 17, 19))


def problem(ovl, dims, n_ev, nrhs):  # noqa: F811
    gen = torch.Generator(device="cuda").manual_seed(81)
    rand = lambda n: torch.randn(n, 4, 3, *reversed(dims), dtype=torch.complex128, device="cuda", generator=gen)  # noqa: E731
    d = ovl.Deflation(rand(n_ev), np.linspace(-0.5, 0.5, n_ev), "f64")
    phi = []  # the basis as stored: a unit coefficient added to zero
    for i in range(n_ev):
        c = torch.zeros((1, n_ev), dtype=torch.complex128, device="cuda")
        c[0, i] = 1
        phi.append(ovl.defl_correct(d, torch.zeros_like(rand(1)), c, np.ones(n_ev))[0].cpu().numpy().ravel())
    return d, np.array(phi), rand(nrhs)


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("n_ev,nrhs", [(1, 2), (1, 12), (2, 6), (2, 7), (3, 4), (4, 4), (4, 5), (5, 2), (6, 2), (6, 3)])
def test_few_modes(ovl, large, n_ev, nrhs):  # noqa: F811
    dims = SITES.get((n_ev, nrhs), MORE)[large]
    d, phi, x = problem(ovl, dims, n_ev, nrhs)
    got = ovl.defl_project(d, x).cpu().numpy()
    xs = x.cpu().numpy().reshape(nrhs, -1)
    for r in range(nrhs):
        for i in range(n_ev):
            t = np.conj(phi[i]).astype(np.clongdouble) * xs[r]
            assert abs(got[r, i] - np.sum(t)) < 200 * 2.0 ** -53 * float(np.sqrt(np.sum(np.abs(t) ** 2)))


@pytest.mark.parametrize("n_ev", [1, 3, 6])
def test_nonfinite_entries(ovl, n_ev):  # noqa: F811
    dims = SITES.get((n_ev, 2), MORE)[1]
    d, _, x = problem(ovl, dims, n_ev, 2)
    want = ovl.defl_project(d, x)
    y = torch.cat([x[:1], x[:1]])
    y[1, 3, 2, dims[3] - 1, dims[2] - 1, dims[1] - 1, dims[0] - 1] = complex(np.inf, 0.0)  # the last site
    c = ovl.defl_project(d, y)
    assert torch.equal(c[0], want[0])
    assert torch.isinf(torch.view_as_real(c[1])).all()  # both parts of phi^* are nonzero there
    y[1, 0, 0, 0, 0, 0, 0] = complex(np.nan, 0.0)
    c = ovl.defl_project(d, y)
    assert torch.equal(c[0], want[0])
    assert torch.isnan(torch.view_as_real(c[1])).all()
