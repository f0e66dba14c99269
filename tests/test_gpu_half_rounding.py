"""FP16 storage in the compound-only passes: every value between steps is the
FP32 result rounded to binary16, as a store and load of a single step rounds it
(a conversion folded into the arithmetic would round once and differ in about
one value in a million)."""
import numpy as np
import pytest

from paper_1307_4703_amd import workloads as W
from tests.parity_util import log
from tests.test_gpu_cde import _cde_pair, _fields, _same_compound

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4, 8, 48])
@pytest.mark.parametrize("layout", ["paired", "planes"])
@pytest.mark.parametrize("links", [False, True])
def test_half_steps_round_as_single_ones(links, layout, n):
    """Half a million nodes, in passes of two, four and eight steps."""
    wl = W.straight_channel(1001, 503, storage="f16", poiseuille_init=False)
    if not links:
        wl = W.Workload("fluid", np.zeros((503, 1001), np.uint8), tau_f=0.8, D=0.02,
                        periodic=(True, True), c_shift=0.5, storage="f16")
    one, two = _cde_pair(wl, "f16", 5, 14, chunk=0)
    two.set_layout(layout)
    for lat in (one, two):
        lat.set_velocity_field(0, *_fields(wl.mask.shape, 9)[0])
    log(f"half rounding, {wl.name} {layout}, {n} steps")
    one.cde_step(n)
    two.cde_step(n)
    _same_compound(one, two, n)
    for lat in (one, two):
        lat.close()
