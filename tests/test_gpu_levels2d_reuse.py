"""A 2D call of several levels per launch does not see what an earlier call
on the same grid left behind: after a run whose field went non-finite, the
next forward, adjoint and gradient equal those of a fresh grid bit for bit.
The points lie on the last grid line before a tile's edge, so that their
nodes of weight zero belong to the next tile."""
import numpy as np
import pytest

from gpu_common import need_gpu, torch

pytestmark = pytest.mark.gpu
SHAPE, H, NT = (130, 101), 10.0, 21


def _grid(so, storage, sinc):
    from paper_1906_10811_amd import Grid
    gen = torch.Generator(device="cuda").manual_seed(so)
    v = 1500.0 + 3000.0 * torch.rand(tuple(reversed(SHAPE)), generator=gen, device="cuda")
    return Grid(SHAPE, (H, H), v, space_order=so, storage=storage, sinc_radius=sinc)


def _calls(g, so, storage, at):
    gen = torch.Generator(device="cuda").manual_seed(so)
    dt = 0.4 * H / 4500.0
    src = rec = [H * np.array(at)]
    wav = torch.randn(NT, 1, generator=gen, device="cuda")
    res = torch.randn(NT, 1, generator=gen, device="cuda")
    r, s = g.forward(src, wav, rec, dt, save_state=True)
    out = [r, *s, g.adjoint(src, rec, res, dt)]
    if storage == "f32":
        for every in (8, NT):
            out += g.gradient(src, wav, rec, res, dt, checkpoint_every=every, want_src_adj=True)
    torch.cuda.synchronize()
    return out


def _poison(g):
    nan = torch.full(g.array_shape, float("nan"), device="cuda")
    pts = np.stack(np.meshgrid(np.arange(0.5, SHAPE[0] - 1, 4.0), np.arange(0.5, SHAPE[1] - 1, 4.0)), -1).reshape(-1, 2)
    r = g.forward(H * pts[:4], torch.ones(NT, 4, device="cuda"), H * pts, 0.4 * H / 4500.0, u0=nan, u_prev=nan)
    torch.cuda.synchronize()
    assert torch.isnan(r).all()


@pytest.mark.parametrize("so", [2, 4, 6, 8, 10])
@pytest.mark.parametrize("edge", ["row", "column"])
@pytest.mark.parametrize("storage,sinc", [("f32", 0), ("f16", 0), ("f32", 3)])
def test_earlier_nan_run_leaves_no_trace(so, storage, sinc, edge):
    need_gpu()
    fresh = _grid(so, storage, sinc)
    lev = fresh.time_block
    assert lev > 2
    height = 64 - so * lev            # rows a tile writes; the tables' columns are 64 points wide
    at = (40.5, height - 1) if edge == "row" else (63, 20.5)
    g = _grid(so, storage, sinc)
    _poison(g)
    for i, (a, b) in enumerate(zip(_calls(g, so, storage, at), _calls(fresh, so, storage, at))):
        assert torch.isfinite(b).all() and torch.equal(a, b), i
    g.close()
    fresh.close()
