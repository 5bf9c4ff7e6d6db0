"""Host sphere tables are read by the GPU from a staging buffer of two halves:
tables handed over faster than the GPU takes them, several between two steps (the
last one counts), and forces read on the host, give what device tables give, bit
for bit."""
import numpy as np
import pytest

import lbm_workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_spheres,path", [(1, "fused"), (40, "fused"), (40, "split")])
def test_host_tables_equal_device_tables(torch_stream, n_spheres, path):
    import torch
    from paper_1703_05158_amd import Lattice
    case = W.case_box(n=(48, 40, 44), n_spheres=n_spheres, radius=(2.0, 4.0), v_sigma=0.02, w_sigma=0.002, gap=0.5,
                      seed=n_spheres, drift=True)
    host, dev = (Lattice.from_case(case, stream=torch_stream, path=path) for _ in range(2))
    tables = [np.concatenate([a.reshape(n_spheres, -1) for a in case.bodies_at(k)], 1) for k in range(41)]
    on_gpu = [torch.from_numpy(t).cuda() for t in tables]
    for k in range(1, 41):
        for j in range(1 + k % 4):  # tables that are replaced before the step
            host.set_bodies(*case.bodies_at((k + 7 * (k % 4 - j)) % 41))
        dev.set_bodies_device(n_spheres, on_gpu[k])
        host.step(1)
        dev.step(1)
        if k % 10 == 0:
            for a, b in zip(host.get_forces(), dev.get_forces()):
                np.testing.assert_array_equal(a, b)
            for a, b in zip(host.get_forces(), dev.get_forces()):  # read twice: from the handle's copy
                np.testing.assert_array_equal(a, b)
    np.testing.assert_array_equal(host.get_populations(), dev.get_populations())
    host.close()
    dev.close()
