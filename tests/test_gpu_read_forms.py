"""Read-back of lattices that are mostly walls, on both sides of the size from
which their outputs are filled first: a field is the same read alone, with one
other and with all, and with the populations."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1307_4703_amd import _abi as A
from paper_1307_4703_amd import workloads as W
from tests.parity_util import log, make_lattice, seeded_init

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx, ny", [(4095, 2048), (4096, 2048), (8192, 2049)])
def test_outputs_agree(nx, ny):
    mask = np.ones((ny, nx), np.uint8)
    mask[1:-1, 3:nx // 4] = 0
    mask[5:-5:3, 9:nx // 4:7] = 1
    wl = W.Workload("walls", mask, tau_f=0.8, D=0.03, storage="f16")
    lat = make_lattice(wl, "f16", seeded_init(wl, 2))
    lat.step(3)
    log(f"read-back {nx}x{ny}")
    new = lambda: torch.full((ny, nx), 7.0, dtype=torch.float64, device="cuda")
    four = [new() for _ in range(4)]
    lat.read_device(*four)
    fluid = torch.from_numpy(mask == 0).cuda()
    for a in four:
        assert torch.isnan(a[~fluid]).all() and torch.isfinite(a[fluid]).all()
    one, two, three = new(), [new(), new()], [new() for _ in range(3)]
    lat.read_device(None, None, None, one)
    lat.read_device(None, two[0], two[1], None)
    lat.read_device(*three, None)
    same = lambda a, b: bool((a.view(torch.int64) == b.view(torch.int64)).all())
    assert same(one, four[3])
    assert same(two[0], four[1]) and same(two[1], four[2])
    assert all(same(a, b) for a, b in zip(three, four))
    g = torch.full((5, ny, nx), 7.0, dtype=torch.float64, device="cuda")
    A.call("gg_read_populations", lat.handle, None, ctypes.c_void_p(g.data_ptr()), A.GG_DEVICE)
    f = torch.full((9, ny, nx), 7.0, dtype=torch.float64, device="cuda")
    g2 = torch.full_like(g, 7.0)
    A.call("gg_read_populations", lat.handle, ctypes.c_void_p(f.data_ptr()),
           ctypes.c_void_p(g2.data_ptr()), A.GG_DEVICE)
    assert same(g, g2)
    assert not g[:, ~fluid].any() and not f[:, ~fluid].any()
    assert torch.allclose(g.sum(0)[fluid], four[3][fluid], rtol=0.0, atol=1e-14)
    assert torch.allclose(f.sum(0)[fluid], four[0][fluid], rtol=0.0, atol=1e-14)
    lat.close()
