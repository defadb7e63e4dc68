"""Memory kept between calls, driven on the CPU through a stand-in for the HIP runtime."""
import pytest

from tests import host_program


@pytest.mark.parametrize("what", ["destroy", "create", "room", "streams"])
def test_memory(tmp_path, what):
    done = host_program.run("memory.cpp", tmp_path, what)
    assert done.returncode == 0, done.stdout
