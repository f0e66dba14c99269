"""Passes of four steps over pipelined strips (lattices of more than a thousand
four-step tiles) and over those tiles (the others), and the two-step passes that
end a run: bitwise the single steps' state and the same boundary fluxes on both
sides of the lines between the forms."""
import numpy as np
import pytest

from paper_1307_4703_amd import Batch
from paper_1307_4703_amd import workloads as W
from tests.parity_util import log, make_lattice, seeded_init

pytestmark = pytest.mark.gpu


def _same(a, b, what):
    """Fluxes: FP64 sums of the same terms in another order, at most 1e6."""
    fa, ga = a.populations()
    fb, gb = b.populations()
    assert a.info()["t"] == b.info()["t"]
    assert np.array_equal(fa, fb) and np.array_equal(ga, gb), what
    da, db = a.diagnostics(), b.diagnostics()
    for k in ("seg_mass", "seg_solute"):
        for x, y in zip(da[k], db[k]):
            assert y == pytest.approx(x, rel=1e-9, abs=1e-9), (what, k)


def _run(wl, storage, runs, tiles, layout="paired", chunk=0, steps=4):
    init = seeded_init(wl, 7)
    one = make_lattice(wl, storage, init, chunk=chunk)
    one.set_two_step(1)
    two = make_lattice(wl, storage, init, chunk=chunk)
    two.set_layout(layout)
    two.set_two_step(5, 6)
    p = two.step_profile(0)
    assert p["steps_per_pass"] == steps
    log(f"passes of {steps}, {wl.nx}x{wl.ny} {storage} {layout}, {p['pass_tiles']} tiles of {p['rows']} rows")
    if tiles:
        assert p["rows"] == 6 and p["pass_tiles"] <= 1024
    for n in runs:
        one.step(n)
        two.step(n)
    _same(one, two, (wl.nx, wl.ny, storage))
    for lat in (one, two):
        lat.close()


def _sides(nx, ny):
    """Inlets and outlets on every side, two of them meeting at a corner, with
    valves that close in turn."""
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
    return W.Workload("sides", mask, tau_f=0.8, D=0.02, segments=segs, schedule=sched)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx, ny", [(1102, 331), (1103, 337), (1101, 343), (58, 6200), (9, 6300)])
def test_strip_edges(storage, nx, ny):
    """All fluid, periodic along x, walls at the rows' ends; widths around the
    strips' 58 columns, runs that end in two-step passes and single steps."""
    wl = W.all_fluid_channel(nx, ny, storage=storage)
    _run(wl, storage, (12, 1, 16), False)


@pytest.mark.parametrize("layout", ["paired", "planes"])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx, ny, tiles", [(131, 70, True), (60, 19, True), (59, 23, True),
                                           (1210, 331, False)])
def test_segments_on_every_side(nx, ny, tiles, storage, layout):
    _run(_sides(nx, ny), storage, (24, 3, 21), tiles, layout, chunk=8)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx, ny", [(57, 5), (58, 6), (59, 7), (4, 40), (117, 4), (5, 5)])
@pytest.mark.parametrize("periodic", [(True, True), (False, False)])
def test_tile_edges(storage, nx, ny, periodic):
    """Random obstacles; axes as short as the passes allow, periodic or not."""
    mask = W.random_mask(nx, ny, seed=3, periodic=periodic)
    if mask.all():
        mask[:] = 0
    wl = W.Workload("obstacles", mask, tau_f=0.7, D=0.03, periodic=periodic, storage=storage)
    _run(wl, storage, (20, 3, 8), True)


@pytest.mark.parametrize("layout", ["paired", "planes"])
@pytest.mark.parametrize("chunk", [0, 16])
def test_eight_steps_and_their_fluxes(layout, chunk):
    """Passes of eight steps, then of four and two, with segments."""
    wl = _sides(2301, 901)
    _run(wl, "f32", (32, 28, 1), False, layout, chunk, steps=8)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("size", [1, 4, 14, 16])
def test_batches(storage, size):
    """Uneven members in tiles, in strips and, FP32, in passes of eight steps;
    the boundary tiles in the one kernel and apart."""
    wls = [_sides(131 * size, 70 * size), W.gradient_generator(nx=300 + 90 * size, ny=150 + 45 * size, half_period=9),
           _sides(60 * size, 19 * size)]
    ones, members = [], []
    for k, wl in enumerate(wls):
        init = seeded_init(wl, k)
        ones.append(make_lattice(wl, storage, init))
        ones[-1].set_two_step(1)
        members.append(make_lattice(wl, storage, init))
    log(f"batch of {sum(w.n_fluid for w in wls)} nodes, {storage}")
    b = Batch(members, graph_chunk=0, fuse=5)
    for n in (16, 1, 15):
        b.step(n)
    for k, (one, lat) in enumerate(zip(ones, members)):
        one.step(32)
        _same(one, lat, k)
    b.close()
    for lat in ones + members:
        lat.close()
