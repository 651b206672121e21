"""Which 2D grids run several levels per launch: those on which one step per
launch measured faster do not (large grids at high order, the more so in 16
bits, and grids a few points thick), those on which the levels win do.  And
the three levels of large float32 grids at so 8 against one step per launch."""
import ctypes

import pytest
import torch

from gpu_common import need_gpu
from paper_1906_10811_amd import _lib

F32, F16, BF16 = 0, 1, 2
ONE_STEP = [((4081, 2081), 10, BF16), ((4081, 2081), 10, F16), ((2481, 1281), 12, BF16), ((2481, 1281), 12, F16),
            ((4081, 2081), 12, F32), ((4081, 2081), 12, BF16), ((7000, 5000), 12, F32), ((12000, 9000), 12, F32),
            ((7000, 5000), 8, BF16), ((7000, 5000), 6, BF16), ((400000, 5), 4, F32), ((400000, 5), 6, F32),
            ((400000, 5), 8, F32), ((400000, 5), 12, F32), ((100000, 20), 8, BF16), ((2481, 1281), 16, F32)]
LEVELS = [((101, 101), 16, BF16, 2), ((2481, 1281), 2, F32, 8), ((2481, 1281), 4, BF16, 4), ((4081, 2081), 6, BF16, 4),
          ((4081, 2081), 8, F32, 2), ((4081, 2081), 10, F32, 2), ((2481, 1281), 12, F32, 2), ((2481, 1281), 10, F16, 2),
          ((7000, 5000), 8, F32, 3), ((5600, 3000), 8, BF16, 2), ((5, 400000), 8, F32, 2), ((7000, 5000), 6, F32, 4)]


def _bytes(shape, so, storage, tb):
    d = _lib.GridDesc()
    d.ndim, d.space_order, d.time_block, d.storage = 2, so, tb, storage
    for a in range(2):
        d.shape[a], d.spacing[a] = shape[a], 10.0
    n = ctypes.c_size_t()
    rc = _lib.load().fd_grid_workspace_bytes(ctypes.byref(d), ctypes.byref(n))
    return n.value if rc == 0 else 0


@pytest.mark.parametrize("shape,so,storage", ONE_STEP)
def test_one_step_per_launch(shape, so, storage):
    assert _bytes(shape, so, storage, 0) == _bytes(shape, so, storage, 1) > 0


@pytest.mark.parametrize("shape,so,storage,levels", LEVELS)
def test_several_levels(shape, so, storage, levels):
    assert _bytes(shape, so, storage, levels) == _bytes(shape, so, storage, 0) > _bytes(shape, so, storage, 1) > 0


@pytest.mark.gpu
def test_three_levels_are_bitwise_single_steps():
    need_gpu()
    from paper_1906_10811_amd import Grid
    gen = torch.Generator(device="cuda").manual_seed(8)
    v = 1500.0 + 3000.0 * torch.rand(2701, 4003, generator=gen, device="cuda")
    wav = torch.randn(11, 2, generator=gen, device="cuda")
    obs = torch.randn(11, 40, generator=gen, device="cuda")
    src, rec = [(20000.0, 13.0), (40020.0, 27000.0)], [(1000.0 * i, 20.0) for i in range(40)]
    out = []
    for tb in (0, 1):
        g = Grid((4003, 2701), (10.0, 10.0), v, space_order=8, time_block=tb)
        assert g.time_block == (1 if tb else 3)
        r, s = g.forward(src, wav, rec, 8e-4, save_state=True)
        out.append([r, *s, g.adjoint(src, rec, obs, 8e-4),
                    *g.gradient(src, wav, rec, obs, 8e-4, checkpoint_every=5, want_src_adj=True)])
        torch.cuda.synchronize()
        g.close()
    for a, b in zip(*out):
        assert torch.isfinite(b).all() and torch.equal(a, b)
