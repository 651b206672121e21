"""Workspaces of 2D grids that run several levels per launch: the scratch of
the levels is bounded, and a workspace of the size that one step per launch
needs is still accepted, for the grid and for its gradient (both then run one
step per launch, with bitwise the same results)."""
import ctypes

import pytest
import torch

from gpu_common import need_gpu
from paper_1906_10811_amd import _lib


def _bytes(shape, so, tb, storage=0, lib=None):
    d = _lib.GridDesc()
    d.ndim, d.space_order, d.time_block, d.storage = 2, so, tb, storage
    for a in range(2):
        d.shape[a], d.spacing[a] = shape[a], 10.0
    n = ctypes.c_size_t()
    _lib.check((lib or _lib.load()).fd_grid_workspace_bytes(ctypes.byref(d), ctypes.byref(n)))
    return n.value


@pytest.mark.parametrize("so", [2, 4, 6, 8, 12])
@pytest.mark.parametrize("shape", [(2481, 1281), (4081, 2081), (12000, 9000), (16000, 15000)])
def test_level_scratch_is_bounded(shape, so):
    field = 4 * shape[0] * shape[1]
    more = _bytes(shape, so, 0) - _bytes(shape, so, 1)
    assert more <= 2 * 1.1 * field + (2 << 30)


def _runs(lib, workspace_of):
    """Forward, adjoint and gradients on a grid whose workspace queries are
    answered for the time_block that workspace_of gives per query."""
    from paper_1906_10811_amd import Grid
    gen = torch.Generator(device="cuda").manual_seed(3)
    v = 1500.0 + 3000.0 * torch.rand(90, 150, generator=gen, device="cuda")
    kw = dict(space_order=4, nbl=10)
    one = Grid((150, 90), (10.0, 10.0), v, time_block=1, **kw)
    real_grid, real_grad = lib.fd_grid_workspace_bytes, lib.fd_gradient_workspace_bytes

    def grid_bytes(d, out):
        if workspace_of["grid"] == 1:
            c = _lib.GridDesc.from_buffer_copy(d._obj)
            c.time_block = 1
            d = ctypes.byref(c)
        return real_grid(d, out)

    def grad_bytes(h, nt, nrec, K, flags, out):
        return real_grad(one._h if workspace_of["gradient"] == 1 else h, nt, nrec, K, flags, out)

    lib.fd_grid_workspace_bytes, lib.fd_gradient_workspace_bytes = grid_bytes, grad_bytes
    try:
        g = Grid((150, 90), (10.0, 10.0), v, **kw)
        src, rec = [(700.0, 33.0)], [(10.0 * i, 20.0) for i in range(0, 140, 7)]
        wav = torch.randn(37, 1, generator=gen, device="cuda")
        obs = torch.randn(37, len(rec), generator=gen, device="cuda")
        dt = 0.4 * 10.0 / 4500.0
        r, s = g.forward(src, wav, rec, dt, save_state=True)
        out = [r, *s, g.adjoint(src, rec, obs, dt)]
        for every in (1, 10, 37):
            out += g.gradient(src, wav, rec, obs, dt, checkpoint_every=every, want_src_adj=True)
        torch.cuda.synchronize()
        levels = g.time_block
        g.close()
    finally:
        lib.fd_grid_workspace_bytes, lib.fd_gradient_workspace_bytes = real_grid, real_grad
    one.close()
    return out, levels


@pytest.mark.gpu
@pytest.mark.parametrize("grid,gradient", [(1, 0), (0, 1)])
def test_one_step_workspace_is_accepted(grid, gradient):
    need_gpu()
    lib = _lib.load()
    want, levels = _runs(lib, dict(grid=0, gradient=0))
    got, had = _runs(lib, dict(grid=grid, gradient=gradient))
    assert levels > 1 and had == (1 if grid else levels)
    for i, (a, b) in enumerate(zip(got, want)):
        assert torch.isfinite(b).all() and torch.equal(a, b), i


def _accepted(shape, so, storage=0):
    ok = []
    for tb in range(0, 10):
        try:
            ok.append((tb, _bytes(shape, so, tb, storage)))
        except _lib.FDError:
            pass
    return ok


@pytest.mark.parametrize("so", [2, 4, 8, 10, 16])
@pytest.mark.parametrize("storage", [0, 2])
def test_only_the_automatic_level_count_is_accepted(so, storage):
    (a, auto), (b, one), (levels, same) = _accepted((150, 90), so, storage)
    assert (a, b) == (0, 1) and 2 <= levels <= 16 // (so // 2) and same == auto > one


def test_no_level_count_where_there_are_none():
    assert [tb for tb, _ in _accepted((2481, 1281), 16)] == [0, 1]


@pytest.mark.gpu
def test_reported_level_count_describes_the_grid():
    need_gpu()
    from paper_1906_10811_amd import Grid
    v = torch.full((90, 150), 2000.0, device="cuda")
    g = Grid((150, 90), (10.0, 10.0), v, space_order=4)
    h = Grid((150, 90), (10.0, 10.0), v, space_order=4, time_block=g.time_block)
    assert h.time_block == g.time_block > 1
    g.close()
    h.close()
