"""The fused step reads which nodes are solid from a bitmap with periodic
copies at the ends of its rows, kept in step with the owner map; the split
path reads the owner map itself.  Both must give the same populations bit for
bit where the bitmap's words, a row's copies and a tile's rows begin and end:
row lengths around multiples of 32 and 64, boxes thinner than a tile, every
tile shape, spheres that cross every face, and a geometry that comes from a
checkpoint."""
import numpy as np
import pytest

import lbm_workloads as W

from .test_gpu_paths import _compare

pytestmark = pytest.mark.gpu


def _case(nx, ny, nz, seed, walls):
    rng = np.random.Generator(np.random.PCG64(seed))
    nb = 5
    R = rng.uniform(1.0, 0.5 * min(nx, ny, nz) - 1.2, nb)
    # two centres on the faces, so that their balls straddle every end
    X = rng.uniform(0.0, 1.0, (nb, 3)) * [nx, ny, nz]
    X[0] = [0.3, ny - 0.4, 0.2]
    X[1] = [nx - 0.45, 0.35, nz - 0.3]
    wall = vel = ref = None
    if walls:
        wall = np.zeros((nz, ny, nx), np.uint8)
        wall[:, 0, :] = 1
        wall[nz // 2, ny // 2, :] = 2
        vel, ref = np.array([[0.0, 0.0, 0.0], [0.01, 0.0, -0.02]]), np.array([[1.0, 0.0, 2.0], [0.0, 3.0, 1.0]])
    return W.Case(name="bits", nx=nx, ny=ny, nz=nz, tau0=0.7, smag_c=0.1, body_force=(1e-5, 0.0, -2e-5),
                  wall_id=wall, wall_vel=vel, wall_ref=ref, X=X, V=rng.normal(0.0, 0.2, (nb, 3)),
                  Omega=rng.normal(0.0, 0.01, (nb, 3)), R=R,
                  u_init=rng.normal(0.0, 0.01, (3, nz, ny, nx)), drift=True)


@pytest.mark.parametrize("tile", range(4))
@pytest.mark.parametrize("size", [(31, 7, 9), (32, 9, 7), (33, 8, 11), (62, 7, 8), (63, 13, 7), (64, 7, 7),
                                  (65, 9, 10), (94, 8, 7), (96, 7, 9), (7, 33, 9), (127, 7, 7)])
def test_fused_equals_split_at_word_and_tile_edges(torch_stream, size, tile):
    from paper_1703_05158_amd import Lattice
    case = _case(*size, seed=size[0] + tile, walls=size[0] % 2 == 0)
    lats = [Lattice.from_case(case, stream=torch_stream, path=p) for p in ("fused", "split")]
    lats[0].set_tile(tile)
    for n in range(1, 7):
        if n == 4:  # the geometry of a checkpoint, into another handle
            state = lats[0].get_state()
            lats[0].close()
            lats[0] = Lattice.from_case(case, stream=torch_stream)
            lats[0].set_tile(tile)
            lats[0].set_state(state)
        for lat in lats:
            lat.set_bodies(*case.bodies_at(n))
            lat.step(1)
    _compare(lats)
