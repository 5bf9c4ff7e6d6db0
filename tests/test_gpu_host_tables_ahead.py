"""A host that hands tables over ahead of the GPU waits for the table whose
staging half it takes, not for what was queued after it."""
import time

import numpy as np
import pytest

import lbm_workloads as W

pytestmark = pytest.mark.gpu


def test_only_the_table_is_waited_for(torch_stream):
    import torch
    from paper_1703_05158_amd import Lattice
    case = W.case_box(n=(128, 128, 128), n_spheres=20, radius=(3.0, 5.0), v_sigma=0.01, gap=0.5, seed=9, drift=True)
    lat, ref = (Lattice.from_case(case, stream=torch_stream) for _ in range(2))
    bodies = [case.bodies_at(k) for k in range(4)]

    def clock(f):
        t = time.perf_counter()
        f()
        return time.perf_counter() - t

    def steps(x, n):
        x.step(n)
        torch.cuda.synchronize()

    for x in (lat, ref):
        x.set_bodies(*bodies[0])
        steps(x, 50)
    long = clock(lambda: steps(lat, 1200))
    ref.step(1200)
    torch.cuda.synchronize()
    # the third table takes the half of the first, which the GPU reads after
    # the first steps; 1200 more are queued behind it
    lat.step(600)
    lat.set_bodies(*bodies[1])
    lat.step(1)
    lat.set_bodies(*bodies[2])
    lat.step(1200)
    lat.set_bodies(*bodies[3])
    left = clock(torch.cuda.synchronize)
    lat.step(1)
    assert left > 0.4 * long, (left, long)
    # and the tables were those of their steps
    ref.step(600)
    for k, n in ((1, 1), (2, 1200), (3, 1)):
        torch.cuda.synchronize()
        ref.set_bodies(*bodies[k])
        ref.step(n)
    np.testing.assert_array_equal(lat.get_populations(), ref.get_populations())
    lat.close()
    ref.close()
