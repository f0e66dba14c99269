"""Default passes on both sides of the size up to which boundary tiles share
the one kernel with the others, and boundary fluxes summed by work-groups:
bitwise the single steps' state, the same fluxes."""
import numpy as np
import pytest

from paper_1307_4703_amd import workloads as W
from tests.parity_util import log, make_lattice, seeded_init

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx, ny, split", [(70, 9, False), (2976, 370, False), (3100, 400, True)])
@pytest.mark.parametrize("fuse", [3, 5])
def test_forms_and_fluxes(nx, ny, split, fuse):
    """Inlets and outlets over whole edges and two more that meet them at
    corners. Fluxes: FP64 sums of the same terms in another order, at most
    1e5 of them."""
    mask = np.zeros((ny, nx), np.uint8)
    mask[0, :] = mask[-1, :] = 1
    mask[:, 0] = mask[:, -1] = 1
    mask[1:-1, 0], mask[1:-1, -1] = 2, 3
    mask[0, 1:9], mask[-1, 1:nx // 2] = 4, 5
    segs = [W.Segment(2, "inlet", (-1, 0), u_max=0.02, c_in=1.0), W.Segment(3, "outlet", (1, 0)),
            W.Segment(4, "inlet", (0, -1), u_max=0.01, c_in=0.7), W.Segment(5, "outlet", (0, 1))]
    wl = W.Workload("edges", mask, tau_f=0.8, D=0.03, segments=segs, storage="f32")
    init = seeded_init(wl, 3)
    one = make_lattice(wl, "f32", init)
    one.set_two_step(1)
    two = make_lattice(wl, "f32", init)
    two.set_two_step(fuse, 6)
    if fuse == 3:
        assert (two.step_profile(0)["pass_side_tiles"] > 0) == split
    log(f"default passes {nx}x{ny}, fuse {fuse}")
    for n in (1, 11, 16):
        one.step(n)
        two.step(n)
    (fa, ga), (fb, gb) = one.populations(), two.populations()
    assert np.array_equal(fa, fb) and np.array_equal(ga, gb)
    da, db = one.diagnostics(), two.diagnostics()
    for k in ("seg_mass", "seg_solute"):
        assert any(abs(v) > 0 for v in da[k])
        for a, b in zip(da[k], db[k]):
            assert b == pytest.approx(a, rel=1e-10, abs=1e-10)
    for lat in (one, two):
        lat.close()
