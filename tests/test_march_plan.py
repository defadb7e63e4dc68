"""The t-marching form's tiles: every neighbour a step reads is staged, also where a tile has more face
sites than sites (a host program over the plan and staging functions that the kernel itself uses)."""
from tests import host_program


def test_every_neighbour_is_staged(tmp_path):
    done = host_program.run("march_plan.hip", tmp_path)
    assert done.returncode == 0, done.stdout[-2000:]
