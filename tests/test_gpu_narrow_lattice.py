"""A lattice one node wide with 2^27 rows, whose solid bitmap has more bits than
a launch has threads: it is created, and a moving wall in its last rows is
felt, node for node, as in a small lattice."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _wall_force(stream, ny, nz, z):
    from paper_1703_05158_amd import TILE_SHAPES, Lattice, config
    wall = np.zeros((nz, ny, 1), np.uint8)
    wall[z] = 1
    lat = Lattice(config(1, ny, nz, 0.8, 0.1, max_walls=1, stream=stream))
    lat.set_walls(wall, np.array([[0.0, 0.03, 0.01]]))
    lat.set_tile(TILE_SHAPES.index("16x8x2"))  # the shape whose launch covers so many rows
    lat.init_fields()
    lat.step(3)
    F, _ = lat.get_forces()
    fluid = lat.count_fluid()
    lat.close()
    return F[0], fluid


def test_force_on_a_wall_of_a_narrow_lattice(torch_stream):
    F, fluid = _wall_force(torch_stream, 16384, 8192, 8190)
    Fs, _ = _wall_force(torch_stream, 16, 32, 30)
    assert fluid == 16384 * 8191
    # integer sums of equal links: 1024 times those of 16 nodes along y
    np.testing.assert_array_equal(F, 1024 * Fs)
    assert abs(F[1]) > 1.0
