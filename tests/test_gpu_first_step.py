"""The first step of a lattice with pressure segments or the paper's walls: the
tile lists that the lattice was created with serve it as they are, and a change
of the segments' kind is followed by the form of the passes."""
import numpy as np
import pytest
import torch

from paper_1307_4703_amd import Lattice
from paper_1307_4703_amd import _abi as A
from paper_1307_4703_amd import workloads as W
from tests.parity_util import log, seeded_init

pytestmark = pytest.mark.gpu


def _workload(pressure):
    wl = W.gradient_generator(nx=300, ny=150, half_period=9, storage="f32")
    if pressure:
        wl.segments = [W.Segment(s.id, "pressure", s.normal, rho=1.001, c_in=s.c_in, fix_c=True)
                       for s in wl.segments]
    return wl


@pytest.mark.parametrize("walls", [False, True])
def test_first_step_rebuilds_no_list(walls, monkeypatch):
    """Allocations between the creation and the end of the first steps: the
    list of nodes beside pressure segments and, with the paper's walls, three
    lists of their own."""
    counts = {"alloc": 0, "free": 0}
    keep = {}

    def alloc(nbytes, _ctx):
        t = torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device="cuda")
        keep[t.data_ptr()] = t
        counts["alloc"] += 1
        return t.data_ptr()

    def release(ptr, _ctx):
        keep.pop(ptr)
        counts["free"] += 1

    al = A.gg_alloc(A.GG_ALLOC_FN(alloc), A.GG_RELEASE_FN(release), None)
    monkeypatch.setattr("paper_1307_4703_amd.lattice._torch_allocator", lambda _s: al)
    wl = _workload(True)
    lat = Lattice.from_workload(wl, init=False, device_allocator="torch")
    if walls:
        lat.set_wall_scheme("equilibrium")
    lat.init(**seeded_init(wl, 3))
    before = dict(counts)
    log(f"first step, walls {walls}")
    lat.step(8)
    lat.sync()
    assert counts["alloc"] - before["alloc"] == (4 if walls else 1)
    assert counts["free"] == before["free"]
    lat.close()
    assert not keep


@pytest.mark.parametrize("first", [True, False])
def test_form_follows_the_segments(first):
    """Pressure segments replaced by inlets and outlets, and back: the boundary
    tiles' kernel apart with the former only, the state as in single steps."""
    out = []
    for fuse in (1, 3):
        lat = Lattice.from_workload(_workload(first), init=False)
        lat.set_two_step(fuse, 6)
        lat.init(**seeded_init(_workload(first), 3))
        for pressure in (first, not first, first):
            for s in _workload(pressure).segments:
                lat.set_segment(s.id, s.kind, s.normal, s.u_max, s.c_in, s.rho, s.fix_c)
            lat.step(12)
            if fuse == 3:
                assert (lat.step_profile(0)["pass_side_tiles"] > 0) == pressure
        out.append(lat.populations())
        lat.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
