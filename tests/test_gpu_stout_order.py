"""Stout smearing and its chain rule on lattices whose (y, z) extents take the t-streaming tile order of
the path kernels (one tile, several tiles, a slice of two workgroups), and the derivative of the
exponential where it is scaled and squared, against the FP64 oracle (1e-13 links, 1e-12 derivatives as in
the memory-order cases)."""
import numpy as np
import pytest

import latgen
from oracle import stout as ostout
from tests.conftest import rel_err
from tests.test_gpu_stout import dev, gauss, host, ovl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(16, 4, 4, 3), (8, 8, 8, 2), (16, 8, 4, 1), (12, 8, 16, 2)])
@pytest.mark.parametrize("eps,steps", [(-0.25, 2), (1.0, 1)])
def test_tile_order(ovl, dims, eps, steps):  # noqa: F811
    u = latgen.random_su3_field(dims, 10610, noise=0.5)
    g = gauss(u.shape, 10611)
    assert rel_err(host(ovl.stout_smear(dev(u), 0.1, eps, steps)), ostout.smear(u, 0.1, eps, steps)) < 1e-13
    got = host(ovl.stout_backward(dev(u), dev(g), 0.1, eps, steps))
    assert rel_err(got, ostout.smear_backward(u, 0.1, eps, steps, g)) < 1e-12


@pytest.mark.parametrize("rho", [0.02, 0.7, 2.0])
def test_exponential_scaling(ovl, rho):  # noqa: F811
    """||M|| from well below 1/2 (no squaring) to several squarings, on rough links."""
    dims = (3, 2, 4, 2)
    u = latgen.random_su3_field(dims, 10612, noise=1.0)
    g = gauss(u.shape, 10613)
    assert rel_err(host(ovl.stout_smear(dev(u), rho, -0.25, 1)), ostout.smear(u, rho, -0.25, 1)) < 1e-12
    got = host(ovl.stout_backward(dev(u), dev(g), rho, -0.25, 1))
    assert rel_err(got, ostout.smear_backward(u, rho, -0.25, 1, g)) < 1e-12
