"""Device memory that handles keep from a drag gradient: given back, from every
handle that keeps some, when an allocation would fail otherwise, and counted."""
import threading

import pytest

import lbm_workloads as W

pytestmark = pytest.mark.gpu

GIB = 1 << 30


def _case(n=(96, 96, 96)):
    return W.case_box(n=n, n_spheres=8, radius=(4.0, 4.0), tau0=0.6, smag_c=0.1, gap=2.0, seed=6)


def _keeps(torch_stream, case, steps):
    """A handle that keeps the memory of a gradient of `steps` checkpoints."""
    from paper_1703_05158_amd import Lattice
    lat = Lattice.from_case(case, stream=torch_stream)
    own, state = lat.info()["device_bytes"], lat.get_state()
    grad = lat.drag_gradient(steps, 1)
    assert lat.info()["device_bytes"] > own + steps * 19 * 4 * 96 ** 3
    return lat, own, state, grad


def test_given_back_when_an_allocation_would_fail(torch_stream):
    import torch
    from paper_1703_05158_amd import Lattice
    case = _case()
    kept = [_keeps(torch_stream, case, 20) for _ in range(2)]  # 1.4 GiB each
    torch.cuda.empty_cache()
    # all but 1.5 GiB of what is left, so that a lattice of 2.2 GiB fits only
    # in what the two keep
    free = torch.cuda.mem_get_info()[0]
    fill = torch.empty(free - 3 * GIB // 2, dtype=torch.uint8, device="cuda")
    try:
        # a third thread counts meanwhile: the owners' figures are whole
        seen, stop = [], threading.Event()

        def watch():
            while not stop.is_set():
                seen.append(kept[0][0].info()["device_bytes"])

        t = threading.Thread(target=watch)
        before = kept[0][0].info()["device_bytes"]
        t.start()
        big = Lattice.from_case(_case((256, 256, 232)), stream=torch_stream)
        stop.set()
        t.join()
        assert set(seen) <= {before, kept[0][1]}
        assert [lat.info()["device_bytes"] for lat, *_ in kept] == [own for _, own, _, _ in kept]
        big.close()
    finally:
        del fill
        torch.cuda.empty_cache()
    for lat, _, state, (J, gF, gV) in kept:  # and a gradient allocates again
        lat.set_state(state)
        J2, gF2, gV2 = lat.drag_gradient(20, 1)
        assert J2 == J and (gF2 == gF).all() and (gV2 == gV).all()
        lat.close()


def test_released_to_other_allocators(torch_stream):
    import torch
    lat, own, state, (J, gF, gV) = _keeps(torch_stream, _case(), 20)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    lat.release_memory()
    lat.release_memory()  # nothing left: no error
    assert lat.info()["device_bytes"] == own
    assert torch.cuda.mem_get_info()[0] >= free + GIB
    lat.set_state(state)
    J2, gF2, gV2 = lat.drag_gradient(20, 1)
    assert J2 == J and (gF2 == gF).all() and (gV2 == gV).all()
    lat.close()
