"""Device memory that adjoint runs leave with their lattices: bounded over all
lattices, and given back when another allocation needs it."""
import numpy as np
import pytest
import torch

from paper_1307_4703_amd import Lattice
from paper_1307_4703_amd import _abi as A
from paper_1307_4703_amd import workloads as W
from tests.parity_util import log

pytestmark = pytest.mark.gpu

GIB = 2 ** 30


def _used():
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free


def _gradient(lat, wl, n=400):
    weight, target, r_box = W.chamber_misfit_setup(wl)
    return lat.adjoint(n, weight, target, r_box=r_box)


def test_lattices_together_keep_eight_gib():
    """Each run of 400 steps takes more than a GiB of checkpoints and tapes."""
    wl = W.gradient_generator(nx=1024, ny=512, half_period=150, storage="f32")
    lats = [Lattice.from_workload(wl) for _ in range(10)]
    base = _used()
    for k, lat in enumerate(lats):
        log(f"adjoint of lattice {k}")
        _gradient(lat, wl)
    kept = _used() - base
    assert 2 * GIB < kept < 8.25 * GIB
    for lat in lats:
        lat.close()
    assert _used() <= base


def test_kept_buffers_go_where_memory_is_short(monkeypatch):
    """An allocator that has memory only once the adjoint's buffers are back."""
    wl = W.gradient_generator(nx=1024, ny=512, half_period=150, storage="f32")
    small = W.gradient_generator(nx=300, ny=150, half_period=150, storage="f32")
    a = Lattice.from_workload(wl)
    first = _gradient(a, wl)
    a.init()
    limit = _used() - GIB // 2
    keep = {}

    def alloc(nbytes, _ctx):
        if _used() > limit:
            return None
        t = torch.empty(max(int(nbytes), 1), dtype=torch.uint8, device="cuda")
        keep[t.data_ptr()] = t
        return t.data_ptr()

    def release(ptr, _ctx):
        keep.pop(ptr)

    al = A.gg_alloc(A.GG_ALLOC_FN(alloc), A.GG_RELEASE_FN(release), None)
    monkeypatch.setattr("paper_1307_4703_amd.lattice._torch_allocator", lambda _s: al)
    b = Lattice.from_workload(small, device_allocator="torch")
    b.step(4)
    again = _gradient(a, wl)
    assert again["loss"] == pytest.approx(first["loss"], rel=1e-11)
    assert np.allclose(again["d_R"], first["d_R"], rtol=1e-11, atol=0.0)
    for lat in (a, b):
        lat.close()
