"""Pipelined passes (fuse 5) of four and eight steps: bitwise the single
steps' state where strips end: widths around a strip's 58 and 50 columns,
heights around its rows, runs that end in shorter passes, links and segments
across strip edges, periodic wraps, both population layouts, batches."""
import numpy as np
import pytest

from paper_1307_4703_amd import Batch
from paper_1307_4703_amd import workloads as W
from tests.parity_util import log, make_lattice, seeded_init

pytestmark = pytest.mark.gpu


def _same(a, b, what):
    fa, ga = a.populations()
    fb, gb = b.populations()
    assert a.info()["t"] == b.info()["t"]
    assert np.array_equal(fa, fb) and np.array_equal(ga, gb), what


def _run(wl, storage, runs, steps_per_pass, layout="paired", chunk=0):
    init = seeded_init(wl, 7)
    one = make_lattice(wl, storage, init, chunk=chunk)
    one.set_two_step(1)
    two = make_lattice(wl, storage, init, chunk=chunk)
    two.set_layout(layout)
    two.set_two_step(5, 6)
    assert two.step_profile(0)["steps_per_pass"] == steps_per_pass
    log(f"pipelined pass of {steps_per_pass}, {wl.nx}x{wl.ny} {storage} {layout}")
    for n in runs:
        one.step(n)
        two.step(n)
    _same(one, two, (wl.nx, wl.ny, storage))
    for lat in (one, two):
        lat.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx, ny", [(57, 9), (58, 8), (59, 17), (65, 4), (117, 33), (9, 120)])
def test_four_step_strip_edges(storage, nx, ny):
    """All fluid, periodic along x, walls at the rows' ends; runs of 8k + 4
    and odd steps."""
    wl = W.all_fluid_channel(nx, ny, storage=storage)
    _run(wl, storage, (12, 1, 16), 4)


@pytest.mark.parametrize("layout", ["paired", "planes"])
@pytest.mark.parametrize("nx, ny", [(131, 70), (60, 19)])
def test_four_step_segments_on_every_side(nx, ny, layout):
    """Inlets and outlets on vertical and horizontal edges, meeting at a
    corner, with valves that close in turn."""
    mask = np.zeros((ny, nx), np.uint8)
    mask[0, :] = mask[-1, :] = 1
    mask[:, 0] = mask[:, -1] = 1
    mask[1:9, 0] = 2
    mask[ny - 9:ny - 1, -1] = 3
    mask[0, 1:12] = 4
    mask[-1, nx - 14:nx - 2] = 5
    segs = [W.Segment(2, "inlet", (-1, 0), u_max=0.03, c_in=1.0), W.Segment(3, "outlet", (1, 0)),
            W.Segment(4, "inlet", (0, -1), u_max=0.02, c_in=0.2), W.Segment(5, "outlet", (0, 1))]
    sched = [W.Phase(3, frozenset({2, 3})), W.Phase(5, frozenset({2, 4, 5}), ((2, 0.4),))]
    wl = W.Workload("sides", mask, tau_f=0.8, D=0.02, segments=segs, schedule=sched)
    for storage in ("f64", "f32", "f16"):
        _run(wl, storage, (24, 3, 21), 4, layout)


@pytest.mark.parametrize("periodic", [(True, True), (False, False)])
def test_eight_step_obstacles(periodic):
    """Beyond two million fluid nodes FP32 passes take eight steps; runs of
    16k + 12 end in passes of four and two."""
    mask = W.random_mask(1777, 1433, seed=3, periodic=periodic)
    wl = W.Workload("obstacles", mask, tau_f=0.7, D=0.03, periodic=periodic)
    assert wl.n_fluid > 2_000_000
    _run(wl, "f32", (28, 16), 8)


@pytest.mark.parametrize("layout", ["paired", "planes"])
def test_eight_step_segments(layout):
    """The straight channel's vertical inlet and outlet in eight-step passes,
    from graph replays, boundary strips beside the others."""
    wl = W.straight_channel(2301, 901, storage="f32", poiseuille_init=False)
    _run(wl, "f32", (32, 12), 8, layout, chunk=16)


def test_eight_step_batch():
    """Two uneven members whose fluid nodes together call for eight steps."""
    wls = [W.all_fluid_channel(1500, 999), W.gradient_generator(nx=2048, ny=1024, half_period=9)]
    wls.append(W.all_fluid_channel(901, 801))
    ones, members = [], []
    for k, wl in enumerate(wls):
        init = seeded_init(wl, k)
        ones.append(make_lattice(wl, "f32", init))
        ones[-1].set_two_step(1)
        members.append(make_lattice(wl, "f32", init))
    assert sum(w.n_fluid for w in wls) > 2_000_000
    b = Batch(members, graph_chunk=0, fuse=5)
    for n in (16, 1, 13):
        b.step(n)
    for k, (one, lat) in enumerate(zip(ones, members)):
        one.step(30)
        _same(one, lat, k)
    b.close()
