"""A change of the launch form that runs out of device memory on the way: the
lattice refuses to step while its lists cannot be built, and steps as it should
once they can."""
import numpy as np
import pytest
import torch

from paper_1307_4703_amd import Lattice
from paper_1307_4703_amd import _abi as A
from paper_1307_4703_amd import workloads as W
from tests.parity_util import log, seeded_init

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("launch", [False, True])
@pytest.mark.parametrize("allowed", [0, 1, 2])
def test_failed_lists_lose_no_step(allowed, launch, monkeypatch):
    """The allocations of gg_set_two_step (or gg_set_launch) fail after the
    first `allowed`; a lattice in graph replays and plain launches."""
    keep = {}
    left = [10 ** 9]

    def alloc(nbytes, _ctx):
        if left[0] <= 0:
            return None
        left[0] -= 1
        t = torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device="cuda")
        keep[t.data_ptr()] = t
        return t.data_ptr()

    def release(ptr, _ctx):
        keep.pop(ptr)

    al = A.gg_alloc(A.GG_ALLOC_FN(alloc), A.GG_RELEASE_FN(release), None)
    monkeypatch.setattr("paper_1307_4703_amd.lattice._torch_allocator", lambda _s: al)
    wl = W.gradient_generator(nx=900, ny=452, half_period=9, storage="f32")
    init = seeded_init(wl, 3)
    ref = Lattice.from_workload(wl, init=False)
    lat = Lattice.from_workload(wl, init=False, device_allocator="torch")
    for x in (ref, lat):
        x.set_launch(64, 4, 16)
        x.set_two_step(5, 6)
        x.init(**init)
        x.step(32)
    log(f"lists fail after {allowed} allocations")
    left[0] = allowed
    with pytest.raises(A.GGError):
        if launch:
            lat.set_launch(32, 8, 16)
        else:
            lat.set_two_step(5, 14)
    left[0] = 0
    with pytest.raises(A.GGError):
        lat.step(8)
    assert lat.info()["t"] == 32
    left[0] = 10 ** 9
    for x in (ref, lat):
        x.step(16)
        x.step(9)
    for a, b in zip(ref.populations(), lat.populations()):
        assert np.array_equal(a, b)
    assert ref.info()["t"] == lat.info()["t"]
    for x in (ref, lat):
        x.close()
    assert not keep
