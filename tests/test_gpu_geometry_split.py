"""The wavefronts that share a sphere of the geometry update: balls of fewer than
64, fewer than 192 and more columns, and wider than half the box, by one, two
and four wavefronts (the number of spheres decides), at rest and moving, among
overlaps; the owner map must equal the oracle's after every update."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# radii: at most 4 (9x9 columns), 6.5 (13x13) and more; boxes of which the
# largest balls cover more than half an axis
@pytest.mark.parametrize("n,nb,r,v", [
    ((41, 38, 43), 5, (0.6, 17.9), 0.3),
    ((41, 38, 43), 9, (9.6, 13.0), 2.0),
    ((23, 50, 17), 12, (0.6, 7.4), 0.0),
    ((64, 30, 33), 1100, (0.6, 4.0), 0.4),
    ((72, 66, 18), 4200, (0.6, 3.0), 0.3),
])
def test_owner_map(torch_stream, n, nb, r, v):
    import oracle
    from paper_1703_05158_amd import Lattice, config
    rng = np.random.Generator(np.random.PCG64(nb))
    box = np.array(n, float)
    R = rng.uniform(*r, nb)
    X = rng.uniform(0.0, 1.0, (nb, 3)) * box
    V = rng.uniform(-v, v, (nb, 3))
    Z = np.zeros((nb, 3))
    lat = Lattice(config(*n, 0.8, 0.1, max_bodies=nb, stream=torch_stream))
    o = oracle.Oracle(*n, 0.8, 0.1)
    lat.set_bodies(X, Z, Z, R)
    lat.init_fields()
    for k in range(1, 9):
        X = np.mod(X + V, box)
        X[X >= box] = 0.0
        if k == 5:  # every sphere elsewhere: more nodes than a list holds
            X = rng.uniform(0.0, 1.0, (nb, 3)) * box
        lat.set_bodies(X, Z, Z, R)
        lat.step(1)
        o.set_bodies(X, Z, Z, R)
        np.testing.assert_array_equal(lat.get_owner().reshape(-1), o.own, err_msg=f"update {k}")
    lat.close()


def test_refills_of_many_nodes(torch_stream):
    """Spheres that jump leave whole balls, whose nodes are refilled a lane each:
    populations against the oracle's, to the storage's rounding of a value near
    its weight."""
    import oracle
    from paper_1703_05158_amd import Lattice, config
    from ._pair import pop_rel_err
    rng = np.random.Generator(np.random.PCG64(2))
    n, R = (30, 28, 26), np.array([7.0, 4.0, 1.2, 2.5])
    lat = Lattice(config(*n, 0.8, 0.1, max_bodies=4, stream=torch_stream))
    o = oracle.Oracle(*n, 0.8, 0.1)
    for k in range(3):
        X = np.array([[8.0, 9.0, 7.5], [22.3, 20.1, 19.7], [20.0, 6.0, 20.0], [6.0, 22.0, 21.0]])
        X = np.mod(X + k * np.array([13.0, 11.0, 9.0]), n)
        V, Om = rng.normal(0.0, 0.01, (2, 4, 3))
        for s in (lat, o):
            s.set_bodies(X, V, Om, R)
        if k == 0:
            lat.init_fields()
            o.init_fields()
        lat.step(1)
        o.step(1)
    assert pop_rel_err(o, lat) < 1e-5
    lat.close()


def test_cost_of_overlaps(torch_stream):
    """Twelve spheres of radius 20 to 28 in 160^3, most of them overlapping: an
    update took 3.5 times the step kernel's time, with one wavefront per sphere
    that listed every node of a marked ball 15 times (8 times before there were
    marks).  The bar of 7 leaves a factor of two to either side."""
    import lbm_workloads as W
    from paper_1703_05158_amd import Lattice
    case = W.case_box(n=(160, 160, 160), n_spheres=12, radius=(20.0, 28.0), v_sigma=0.05, w_sigma=0.001, gap=0.5,
                      drift=True)
    lat = Lattice.from_case(case, stream=torch_stream)
    ratio = []
    for rep in range(3):
        for k in range(5):
            lat.set_bodies(*case.bodies_at(1000 + 10 * rep + k))
            lat.step(1)
            if k == 0:
                lat.profile(1)
        ms, steps = lat.profile_read_parts()
        assert steps == 4
        ratio.append(list(ms.values())[0] / list(ms.values())[2])
    lat.close()
    assert min(ratio) < 7.0, ratio
