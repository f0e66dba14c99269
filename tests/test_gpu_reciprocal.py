"""The FP32 reciprocal of the density (hardware approximation and one Newton step)
is the division's value over the range of normal results: the state equals the
replay with the division, bit for bit, for densities over four decades around 1
and near both ends of the type's range."""
import numpy as np
import pytest

from paper_1307_4703_amd import Lattice
from paper_1307_4703_amd import workloads as W
from tests.emu import emu
from tests.parity_util import log
from tests.test_gpu_bitwise_emulation import _raw_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fuse", [1, 3, 5])
@pytest.mark.parametrize("rho0", [1e-36, 1.0, 1e36])
def test_reciprocal_is_the_division(rho0, fuse):
    nx, ny = 512, 256
    mask = W.random_mask(nx, ny, 11, periodic=(True, True))
    wl = W.Workload("box", mask, tau_f=0.8, D=0.03, periodic=(True, True), storage="f32",
                    rho0=rho0)
    rng = np.random.default_rng(5)
    rho = rho0 * 10.0 ** rng.uniform(-2.0, 1.8, mask.shape)
    lat = Lattice.from_workload(wl, init=False)
    lat.set_two_step(fuse, 6)
    lat.init(rho=rho, ux=rng.uniform(-0.1, 0.1, mask.shape), uy=rng.uniform(-0.1, 0.1, mask.shape),
             C=rng.random(mask.shape))
    h, k, t = _raw_state(lat, "f32")
    e = emu.Emulator(wl, "f32")
    log(f"reciprocal, rho0 {rho0}, fuse {fuse}")
    fl = mask == 0
    for n in (2, 4, 2):
        lat.step(n)
        h, k = e.step(h, k, t, n)
        t += n
        hg, kg, tg = _raw_state(lat, "f32")
        assert tg == t
        for a, b in ((hg, h), (kg, k)):
            assert np.array_equal(a[:, fl], b[:, fl], equal_nan=True)
        assert np.isfinite(h[:, fl]).mean() > 0.5
    lat.close()
