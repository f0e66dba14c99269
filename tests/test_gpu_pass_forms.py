"""Where the two-step pass takes the boundary tiles in the one kernel: up to 512
tiles of 14 rows (3072 in FP64, and of 6 rows); the state is the single steps' on
both sides of the line."""
import numpy as np
import pytest

from paper_1307_4703_amd import workloads as W
from tests.parity_util import log, make_lattice, seeded_init

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx, ny, tiles", [(992, 448, 512), (1054, 448, 544)])
@pytest.mark.parametrize("fuse", [3, 5])
def test_fourteen_rows(storage, nx, ny, tiles, fuse):
    mask = np.zeros((ny, nx), np.uint8)
    mask[0, 1:9], mask[-1, 1:nx // 2] = 2, 3
    segs = [W.Segment(2, "inlet", (0, -1), u_max=0.02, c_in=1.0), W.Segment(3, "outlet", (0, 1))]
    wl = W.Workload("edges", mask, tau_f=0.8, D=0.03, segments=segs, periodic=(True, False),
                    storage=storage)
    init = seeded_init(wl, 3)
    one = make_lattice(wl, storage, init)
    one.set_two_step(1)
    two = make_lattice(wl, storage, init)
    two.set_two_step(3, 14)
    p = two.step_profile(0)
    log(f"14 rows, {nx}x{ny} {storage}, {p['pass_tiles']} tiles and {p['pass_side_tiles']} apart")
    assert (p["pass_side_tiles"] == 0) == (storage == "f64" or tiles <= 512)
    two.set_two_step(fuse, 14)
    for n in (4, 1, 15):
        one.step(n)
        two.step(n)
    for a, b in zip(one.populations(), two.populations()):
        assert np.array_equal(a, b)
    for lat in (one, two):
        lat.close()
