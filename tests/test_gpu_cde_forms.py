"""The forms of the compound-only passes on both sides of the lines between them:
four-step tiles on lattices of up to 100000 fluid nodes, with a source and where
the field changes every few steps; the walk on larger ones; two-step tiles at the
end of runs. Bitwise the single steps' compound, the same fluxes."""
import numpy as np
import pytest

from paper_1307_4703_amd import workloads as W
from tests.parity_util import log
from tests.test_gpu_cde import _cde_pair, _fields, _same_compound

pytestmark = pytest.mark.gpu


def _run(wl, storage, runs, rows=14, layout="paired", chunk=0, R=None, n_fields=1):
    one, two = _cde_pair(wl, storage, 5, rows, chunk=chunk, R=R)
    two.set_layout(layout)
    fields = _fields(wl.mask.shape, 9)
    for lat in (one, two):
        for k in range(n_fields):
            lat.set_velocity_field(k, *fields[k])
        if n_fields == 2:
            lat.set_phase_fields([0, 1])
    log(f"compound passes, {wl.name} {wl.nx}x{wl.ny} {storage} {layout} rows {rows}")
    for n in runs:
        one.cde_step(n)
        two.cde_step(n)
    _same_compound(one, two, sum(runs))
    return one, two


def _close(*lats):
    for lat in lats:
        lat.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx, ny", [(1050, 128), (1049, 127), (1051, 126), (50, 2700), (8, 16000),
                                    (7, 18000), (4, 30000), (30000, 5)])
def test_walk_strip_edges(storage, nx, ny):
    """Random masks, periodic along both axes, passes of 8 or 4 and then of 4 and
    2 steps."""
    mask = W.random_mask(nx, ny, seed=3, periodic=(True, True))
    wl = W.Workload("random", mask, tau_f=0.7, D=0.03, periodic=(True, True), storage=storage)
    assert wl.n_fluid > 100_000
    _close(*_run(wl, storage, (28, 16, 2)))


def _segments(nx, ny, storage):
    mask = np.zeros((ny, nx), np.uint8)
    mask[0, :] = mask[-1, :] = 1
    mask[:, 0] = mask[:, -1] = 1
    segs = []
    for k, (a, b) in enumerate([(2, 5), (7, 9), (11, ny - 1)]):
        mask[a:b, 0] = 2 + k
        segs.append(W.Segment(2 + k, "inlet" if k != 1 else "outlet", (-1, 0), u_max=0.0,
                              c_in=0.5 + k))
    mask[0, 1:4], mask[0, 8:nx // 2] = 5, 6
    mask[-1, 60:90] = 7
    segs += [W.Segment(5, "outlet", (0, -1)), W.Segment(6, "inlet", (0, -1), u_max=0.0, c_in=2.0),
             W.Segment(7, "inlet", (0, 1), u_max=0.0, c_in=0.7)]
    sched = [W.Phase(13, frozenset({2, 3, 6})), W.Phase(17, frozenset({2, 4, 5, 7}), ((2, 0.4),))]
    return W.Workload("segments", mask, tau_f=0.8, D=0.04, segments=segs, schedule=sched,
                      storage=storage)


@pytest.mark.parametrize("layout", ["paired", "planes"])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx, ny, n_fields, rows", [(1052, 131, 1, 14), (1052, 131, 2, 14),
                                                    (131, 59, 2, 14), (131, 59, 1, -10),
                                                    (101, 31, 1, -6)])
def test_segments_and_schedule(storage, nx, ny, n_fields, rows, layout):
    """Valves that switch every 13 and 17 steps, a field for both or one each;
    graph replays and plain launches."""
    wl = _segments(nx, ny, storage)
    _close(*_run(wl, storage, (64, 30), rows, layout, chunk=32, n_fields=n_fields))


@pytest.mark.parametrize("layout", ["paired", "planes"])
@pytest.mark.parametrize("storage, nx, ny", [("f64", 2101, 1501), ("f32", 1052, 131), ("f32", 2101, 1001),
                                             ("f16", 2101, 1001), ("f16", 300, 150)])
def test_source(storage, nx, ny, layout):
    """A source: the walk in large FP64 lattices, tiles of four and of two steps
    elsewhere; taken away, and a field of another phase set, in between."""
    wl = _segments(nx, ny, storage)
    R = np.zeros(wl.mask.shape)
    R[20:60, 10:200] = 1e-3
    one, two = _run(wl, storage, (32, 12), 14, layout, chunk=16, R=R)
    for lat in (one, two):
        lat.set_source(None)
    one.cde_step(48)
    two.cde_step(48)
    for lat in (one, two):
        lat.set_velocity_field(1, *_fields(wl.mask.shape, 4)[1])
        lat.set_phase_fields([0, 1])
        lat.set_schedule([W.Phase(5, frozenset({2, 3, 6})), W.Phase(3, frozenset({4, 5, 7}))])
        lat.cde_step(36)
    _same_compound(one, two, 128)
    _close(one, two)
