"""Adjoint runs that take the buffers of the run before: the gradients are those
of a fresh lattice, whatever sizes the runs before asked for."""
import numpy as np
import pytest

from paper_1307_4703_amd import Lattice
from paper_1307_4703_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("before", [(12, 0), (30, 0), (12, 5), (3, 1)])
@pytest.mark.parametrize("fuse", [1, 3, 4])
def test_gradients_after_another_run(fuse, before):
    """dL/dC_in is summed by atomics: FP64 rounding of at most 1e4 terms."""
    wl = W.gradient_generator(nx=230, ny=116, half_period=9, storage="f32")
    weight, target, r_box = W.chamber_misfit_setup(wl)
    out = []
    for runs in ((), (before, (12, 0)), (before,)):
        lat = Lattice.from_workload(wl)
        lat.set_two_step(fuse, 6)
        for n, every in runs:
            lat.adjoint(n, weight, target, r_box=r_box if n != 30 else None, ckpt_every=every)
            lat.init()
        out.append(lat.adjoint(12, weight, target, r_box=r_box))
        lat.close()
    for r in out[1:]:
        assert r["loss"] == pytest.approx(out[0]["loss"], rel=1e-11)
        assert r["d_D"] == pytest.approx(out[0]["d_D"], rel=1e-11)
        assert np.allclose(r["d_R"], out[0]["d_R"], rtol=1e-11, atol=0.0)
        assert np.allclose(r["d_c_in"], out[0]["d_c_in"], rtol=1e-11, atol=0.0)
