"""The gradient's listed links where two spheres face each other across gaps of
one and two nodes, whose links share adjoint slots, and the device memory that a
handle keeps from one gradient to the next."""
import dataclasses

import numpy as np
import pytest

import lbm_workloads as W

pytestmark = pytest.mark.gpu


def _case(gap, axis, seed=3):
    """Two spheres of radius 3 whose surfaces are `gap` apart along an axis, and
    a third across the periodic corner."""
    n = (26, 24, 25)
    case = W.case_box(n=n, n_spheres=3, radius=(3.0, 3.0), tau0=0.6, smag_c=0.1, body_force=(5e-6, 0.0, 0.0),
                      u_sigma=0.0, gap=2.0, seed=seed)
    X = np.array([[8.03, 9.07, 10.02], [8.03, 9.07, 10.02], [0.4, 23.7, 0.3]])
    X[1, axis] += 6.0 + gap
    rng = np.random.Generator(np.random.PCG64(seed))
    return dataclasses.replace(case, X=X, V=rng.normal(0.0, 0.01, size=(3, 3)))


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(b))


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("gap", [0.2, 1.05, 2.1])
def test_facing_spheres_against_the_fp64_reference(torch_stream, gap, axis):
    """The bar of the gradient tests, 1e-3 in norm.  J itself nearly cancels
    between two spheres that push each other apart, so no relative bar holds for
    it: it is the sum of the forces that the call leaves behind, exactly."""
    import oracle
    from oracle.adjoint import DragProblem
    from paper_1703_05158_amd import Lattice
    case, steps = _case(gap, axis), 12
    o = oracle.Oracle.from_case(case)
    _, gFr, gVr = DragProblem(o).gradient(o.populations(), case.body_force, case.V, steps)
    lat = Lattice.from_case(case, stream=torch_stream)
    state = lat.get_state()
    J, gF, gV = lat.drag_gradient(steps, 5)
    assert J == sum(lat.get_forces()[0][:, 0])
    assert _rel(gF, gFr) < 1e-3
    assert _rel(gV, gVr) < 1e-3
    # the sums' order is fixed: the same gradient from the same state (dJ/dV adds
    # FP64 wavefront sums in any order: 1e-12)
    lat.set_state(state)
    J2, gF2, gV2 = lat.drag_gradient(steps, 5)
    assert J2 == J
    np.testing.assert_array_equal(gF2, gF)
    assert _rel(gV2, gV) < 1e-12
    lat.close()


def test_kept_memory(torch_stream):
    """Gradients of different lengths in turn use what the handle kept, and give
    what a fresh handle gives; the memory is counted while it is held."""
    from paper_1703_05158_amd import Lattice
    case = _case(2.1, 0)
    lat = Lattice.from_case(case, stream=torch_stream)
    state, held = lat.get_state(), lat.info()["device_bytes"]
    fresh = {}
    for steps, ckpt in ((3, 1), (9, 4), (20, 20)):
        one = Lattice.from_case(case, stream=torch_stream)
        fresh[steps, ckpt] = one.drag_gradient(steps, ckpt)
        one.close()
    for steps, ckpt in ((9, 4), (3, 1), (20, 20), (9, 4)):
        lat.set_state(state)
        J, gF, gV = lat.drag_gradient(steps, ckpt)
        assert J == fresh[steps, ckpt][0]
        np.testing.assert_array_equal(gF, fresh[steps, ckpt][1])
        assert _rel(gV, fresh[steps, ckpt][2]) < 1e-12
    assert lat.info()["device_bytes"] > held
    lat.close()
