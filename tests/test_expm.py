"""The exponential of the smearing step and its derivative keep the precision of the sum of matrix powers
(a host program on the functions the kernels use, against extended precision)."""
from tests import host_program


def test_exp_precision(tmp_path):
    done = host_program.run("expm.hip", tmp_path)
    assert done.returncode == 0, done.stdout
