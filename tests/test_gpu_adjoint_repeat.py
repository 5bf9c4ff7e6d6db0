"""The drag gradient is the same, bit for bit, every time it is taken from the
same state: dJ/dV too, which is summed over the several wavefronts of each
sphere's links."""
import numpy as np
import pytest

import lbm_workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_spheres,radius,mode", [
    ((48, 40, 44), 30, (2.0, 4.0), "bouzidi"),
    ((48, 40, 44), 30, (0.6, 4.0), "halfway"),
    ((64, 60, 62), 1, (22.0, 22.0), "bouzidi"),  # more than 64 wavefronts of links per sphere
    ((20, 18, 16), 0, (2.0, 2.0), "bouzidi"),
])
def test_same_gradient_every_time(torch_stream, n, n_spheres, radius, mode):
    from paper_1703_05158_amd import Lattice
    case = W.case_box(n=n, n_spheres=n_spheres, radius=radius, tau0=0.6, smag_c=0.1, v_sigma=0.01,
                      body_force=(5e-6, 0.0, 0.0), gap=0.5, seed=11)
    lat = Lattice.from_case(case, bb_mode=mode, stream=torch_stream)
    state = lat.get_state()
    J, gF, gV = lat.drag_gradient(7, 3)
    for _ in range(5):
        lat.set_state(state)
        J2, gF2, gV2 = lat.drag_gradient(7, 3)
        assert J2 == J
        np.testing.assert_array_equal(gF2, gF)
        np.testing.assert_array_equal(gV2, gV)
    lat.close()
