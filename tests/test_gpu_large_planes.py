"""Lattices whose fourteen planes span more than 4 GiB: the passes that store a
node's links through 32-bit offsets from the first plane take their other way.
Compared with single steps on the device."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1307_4703_amd import Lattice
from paper_1307_4703_amd import _abi as A
from paper_1307_4703_amd import workloads as W
from tests.parity_util import log

pytestmark = pytest.mark.gpu


def _mask(nx, ny):
    mask = np.zeros((ny, nx), np.uint8)
    mask[0, :] = mask[-1, :] = 1
    mask[:, 0] = mask[:, -1] = 1
    mask[100:-1:97, 31:-31:53] = 1
    mask[1:ny // 2, 0] = 2
    mask[ny // 2:-1, -1] = 3
    return mask


def _state(lat, f, g):
    A.call("gg_read_populations", lat.handle, ctypes.c_void_p(f.data_ptr()),
           ctypes.c_void_p(g.data_ptr()), A.GG_DEVICE)


@pytest.mark.parametrize("storage, nx, ny", [("f64", 6300, 6310), ("f32", 8800, 8810)])
def test_passes_equal_single_steps(storage, nx, ny):
    mask = _mask(nx, ny)
    segs = [W.Segment(2, "inlet", (-1, 0), u_max=0.02, c_in=1.0), W.Segment(3, "outlet", (1, 0))]
    wl = W.Workload("large", mask, tau_f=0.8, D=0.03, segments=segs, storage=storage)
    assert 14 * nx * ny * (8 if storage == "f64" else 4) > 1 << 32
    lat = Lattice.from_workload(wl, init=False)
    yy, xx = np.mgrid[0:ny, 0:nx].astype(np.float32)
    wave = np.cos(xx * 0.07) * np.cos(yy * 0.05)
    init = {"ux": 0.02 * wave, "uy": -0.015 * wave, "C": 0.5 + 0.4 * wave}
    shape = (ny, nx)
    ref = [torch.empty((k, *shape), dtype=torch.float64, device="cuda") for k in (9, 5)]
    got = [torch.empty_like(a) for a in ref]
    for what, steps in (("coupled", 24), ("compound", 24)):
        log(f"{what} steps of a {nx}x{ny} lattice, {storage}")
        for form, out in ((0, ref), (1, got)):
            lat.set_two_step(3, 6)
            lat.init(**init)
            if what == "compound":
                lat.set_velocity_field(0)
                lat.set_cde_launch(14 if form else 0)
                lat.cde_step(steps)
            else:
                lat.set_two_step(5 if form else 1, 6)
                lat.step(steps)
            _state(lat, *out)
        for a, b in zip(ref, got):
            assert bool((a.view(torch.int64) == b.view(torch.int64)).all()), what
    lat.close()
