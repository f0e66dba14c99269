"""Compound-only passes of eight, four and two steps (a wavefront per strip of
50 columns): bitwise the single steps' compound where strips end, on periodic
axes as short as the passes allow, with the schedule and the field changing
inside a pass, and at strips that meet more than two segments."""
from dataclasses import replace

import numpy as np
import pytest

from paper_1307_4703_amd import workloads as W
from tests.parity_util import log
from tests.test_gpu_cde import _cde_pair, _fields, _same_compound

pytestmark = pytest.mark.gpu


def _run(wl, storage, runs, layout="paired", chunk=0, R=None, n_fields=1):
    one, two = _cde_pair(wl, storage, 5, 14, chunk=chunk, R=R)
    two.set_layout(layout)
    fields = _fields(wl.mask.shape, 9)
    for lat in (one, two):
        for k in range(n_fields):
            lat.set_velocity_field(k, *fields[k])
        if n_fields == 2:
            lat.set_phase_fields([0, 1])
    log(f"compound walk, {wl.nx}x{wl.ny} {storage} {layout}")
    for n in runs:
        one.cde_step(n)
        two.cde_step(n)
    _same_compound(one, two, sum(runs))
    for lat in (one, two):
        lat.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx, ny", [(50, 8), (49, 7), (51, 40), (101, 33), (8, 9), (7, 8),
                                    (4, 30), (3, 5), (2, 2), (1, 6)])
def test_strip_edges_and_short_periodic_axes(storage, nx, ny):
    """Random masks, periodic along both axes (passes of 8, 4 or 2 steps, or
    single steps, by the shorter axis); runs that use all of them."""
    mask = W.random_mask(nx, ny, seed=3, periodic=(True, True))
    mask[ny // 2, nx // 2] = 0
    wl = W.Workload("random", mask, tau_f=0.7, D=0.03, periodic=(True, True), storage=storage)
    _run(wl, storage, (28, 16, 2))


@pytest.mark.parametrize("layout", ["paired", "planes"])
@pytest.mark.parametrize("source, n_fields", [(False, 1), (False, 2), (True, 1)])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_changes_inside_a_pass(storage, source, n_fields, layout):
    """Valves that switch every 3 and 5 steps, with one field or one per
    phase, and a source: graph replays of eight-step passes and shorter runs."""
    wl = W.gradient_generator(nx=230, ny=116, half_period=5, storage=storage)
    wl.schedule[0] = replace(wl.schedule[0], duration=3)
    R = None
    if source:
        R = np.zeros(wl.mask.shape)
        R[20:40, 60:150] = 1e-3
    _run(wl, storage, (64, 30), layout, chunk=32, R=R, n_fields=n_fields)


@pytest.mark.parametrize("nx, ny", [(64, 40), (112, 19)])
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_many_segments_in_a_strip(storage, nx, ny):
    """Five segments along two edges that meet, two cells apart, more than a
    strip's lanes keep sums for; the fluxes are the single steps'."""
    mask = np.zeros((ny, nx), np.uint8)
    mask[0, :] = mask[-1, :] = 1
    mask[:, 0] = mask[:, -1] = 1
    segs = []
    for k, (a, b) in enumerate([(2, 5), (7, 9), (11, 12)]):
        mask[a:b, 0] = 2 + k
        segs.append(W.Segment(2 + k, "inlet" if k != 1 else "outlet", (-1, 0),
                              u_max=0.0, c_in=0.5 + k))
    mask[0, 1:4] = 5
    mask[0, 8:20] = 6
    segs += [W.Segment(5, "outlet", (0, -1)), W.Segment(6, "inlet", (0, -1), u_max=0.0, c_in=2.0)]
    wl = W.Workload("segments", mask, tau_f=0.8, D=0.04, segments=segs, storage=storage)
    _run(wl, storage, (48, 12))
