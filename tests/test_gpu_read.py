"""Read-back where its one kernel can go wrong: row ends off its 256 cells, one
row or column, lattices without fluid, outputs left out."""
import numpy as np
import pytest
import torch

from paper_1307_4703_amd import workloads as W
from tests.parity_util import log, make_lattice, seeded_init

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx, ny", [(255, 3), (256, 5), (257, 4), (515, 9), (5, 70), (24, 12)])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_fields_are_the_populations_moments(storage, nx, ny):
    """The fields against the moments of the FP64 populations read back beside
    them (a few roundings of 1 apart), NaN and 0 off the fluid, at both
    parities; a field read alone is the same."""
    mask = W.random_mask(nx, ny, 11)
    wl = W.Workload("read", mask, tau_f=0.8, D=0.03, storage=storage)
    lat = make_lattice(wl, storage, seeded_init(wl, 2))
    log(f"read-back {nx}x{ny} {storage}")
    fluid = mask == 0
    for steps in (0, 1, 3):
        lat.step(steps)
        f, g = lat.populations()
        out = [torch.full((ny, nx), 7.0, dtype=torch.float64, device="cuda") for _ in range(4)]
        lat.read_device(*out)
        rho, ux, uy, C = [o.cpu().numpy() for o in out]
        for a in (rho, ux, uy, C):
            assert np.isnan(a[~fluid]).all()
        assert not f[:, ~fluid].any() and not g[:, ~fluid].any()
        fs, gs = f[:, fluid], g[:, fluid]
        jx = fs[1] - fs[3] + fs[5] - fs[6] + fs[8] - fs[7]
        jy = fs[2] - fs[4] + fs[5] - fs[7] + fs[6] - fs[8]
        for a, b in ((rho, fs.sum(0)), (ux, jx / fs.sum(0)), (uy, jy / fs.sum(0)), (C, gs.sum(0))):
            assert np.abs(a[fluid] - b).max(initial=0.0) < 1e-14
        alone = torch.full((ny, nx), 7.0, dtype=torch.float64, device="cuda")
        lat.read_device(None, None, None, alone)
        assert np.array_equal(alone.cpu().numpy(), C, equal_nan=True)
    lat.close()
