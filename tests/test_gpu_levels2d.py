"""2D grids run several time levels per launch (k_step2d_tb); each level is
the one-step kernel's sequence of operations, so every result is bitwise
that of time_block = 1 (one step per launch, itself held to the oracle in
test_gpu_parity.py): forward traces and state, adjoint, gradient by both
schedules, over all orders and storages, tiles cut at every edge, more
steps than a multiple of the levels, source points in the recomputed ring,
more source points in a tile than its table holds, windowed-sinc points,
and grids beyond the many-tiles line of the level rule."""
import numpy as np
import pytest
import torch

from gpu_common import need_gpu

pytestmark = pytest.mark.gpu

# shape, damping points, steps, sources, receivers, sinc half-width, caller state
SMALL = [((67, 41), 3, 19, 2, 5, 0, True), ((130, 97), 0, 40, 1, 33, 0, False),
         ((33, 150), 10, 33, 200, 3, 0, False), ((200, 70), 5, 21, 3, 40, 3, False),
         ((32, 33), 0, 17, 1, 2, 0, True), ((3, 65), 0, 9, 1, 1, 0, True)]
LARGE = [((1700, 1100), 20, 11, 2, 40, 0, False)]


def _run(shape, nbl, nt, nsrc, nrec, sinc, state, so, storage, tb):
    from paper_1906_10811_amd import Grid
    dev = torch.device("cuda")
    rng = np.random.default_rng(so)
    gen = torch.Generator(device=dev)
    gen.manual_seed(so)
    v = 1500.0 + 3000.0 * torch.rand(tuple(reversed(shape)), generator=gen, device=dev)
    ext = np.array([(n - 1) * 10.0 for n in shape])
    src, rec = rng.uniform(0, 1, (nsrc, 2)) * ext, rng.uniform(0, 1, (nrec, 2)) * ext
    src[0], rec[0] = ext, 0.0          # on two corners of the grid
    dt = 0.4 * 10.0 / 4500.0
    g = Grid(shape, (10.0, 10.0), v, space_order=so, nbl=nbl, storage=storage, sinc_radius=sinc, time_block=tb,
             max_src=max(64, nsrc))
    wav = torch.randn(nt, nsrc, generator=gen, device=dev)
    u0 = torch.randn(g.array_shape, generator=gen, device=dev) if state else None
    r, s = g.forward(src, wav, rec, dt, u0=u0, u_prev=u0, save_state=True)
    out = [r, *s, g.adjoint(src, rec, torch.randn(nt, nrec, generator=gen, device=dev), dt)]
    if storage == "f32":
        for every in (7, nt):
            out += g.gradient(src, wav, rec, 0 * r, dt, checkpoint_every=every, want_src_adj=True)
    torch.cuda.synchronize()
    levels = g.time_block
    g.close()
    return out, levels


@pytest.mark.parametrize("so", [2, 4, 6, 8, 10, 12, 14, 16])
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_levels_are_bitwise_single_steps(so, storage):
    need_gpu()
    for case in SMALL + (LARGE if storage == "f32" else []):
        got, levels = _run(*case, so, storage, 0)
        want, one = _run(*case, so, storage, 1)
        assert one == 1 and levels * (so // 2) <= 16
        assert levels > 1 or (case in LARGE and so >= 14)
        for i, (a, b) in enumerate(zip(got, want)):
            assert torch.isfinite(b).all() and torch.equal(a, b), (case, so, storage, levels, i)


def test_server_reserves_single_step_fields():
    """Served 2D shots keep the workspace of one step per launch (the budget admits by it)."""
    import ctypes

    from paper_1906_10811_amd import Server, _lib
    kw = dict(shape=(120, 90), spacing=(10.0, 10.0), space_order=4, nbl=10, vp=np.full((90, 120), 2000.0, np.float32),
              src_xyz=[(300.0, 40.0)], wavelet=np.ones((20, 1), np.float32), rec_xyz=[(100.0, 20.0)], dt=1e-3)
    assert Server.request_bytes(**kw) == Server.request_bytes(**kw, time_block=1)
    r, _ = Server._request(**kw)
    n0, n1 = ctypes.c_size_t(), ctypes.c_size_t()
    _lib.check(_lib.load().fd_grid_workspace_bytes(ctypes.byref(r.grid), ctypes.byref(n0)))
    r.grid.time_block = 1
    _lib.check(_lib.load().fd_grid_workspace_bytes(ctypes.byref(r.grid), ctypes.byref(n1)))
    assert n0.value > n1.value
