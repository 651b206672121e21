"""2D diffusion, several levels per launch by two kernels (tiles for small
grids, strips for large ones): both keep one step's operations, so u^nt is
bitwise the same whatever time_block allows.  Grids around the tile and
strip widths, ragged in both axes, narrow ones, and ones beyond the line
between the kernels at each radius, against one step per launch; the strip
kernel's single step against the FP64 reading on a grid that takes it."""
import numpy as np
import pytest

import oracle
from gpu_common import need_gpu, rel_l2, torch

pytestmark = pytest.mark.gpu
SMALL = [(2, 3), (31, 65), (64, 64), (66, 33), (257, 130)]
# beyond 2 M, 4 M and 7 M points: strips, ragged, one and many of them
LARGE = [(2300, 911), (241, 16700), (16700, 243), (2900, 2450)]


@pytest.mark.parametrize("so", [2, 4, 6, 8, 10, 12, 14, 16])
def test_result_does_not_depend_on_time_block(so):
    need_gpu()
    from paper_1906_10811_amd import diffusion, diffusion_dt_limit
    gen = torch.Generator(device="cuda")
    gen.manual_seed(so)
    for nx, ny in SMALL + LARGE:
        u0 = torch.randn(ny, nx, generator=gen, device="cuda")
        dt = 0.9 * diffusion_dt_limit((nx, ny), (1.0, 1.5), so, 0.5)
        want = diffusion(u0, (1.0, 1.5), so, 0.5, dt, 21, time_block=1)
        for tb in (0, 2, 3, 16):
            got = diffusion(u0, (1.0, 1.5), so, 0.5, dt, 21, time_block=tb)
            assert torch.isfinite(want).all() and torch.equal(got, want), (so, nx, ny, tb)


@pytest.mark.parametrize("so", [2, 6, 8, 16])
def test_strips_against_oracle(so):
    need_gpu()
    from paper_1906_10811_amd import diffusion
    nx, ny = 2900, 2450
    g = oracle.Grid((nx, ny), (1.0, 1.5), (0.0, 0.0), so)
    dt = 0.8 * oracle.diffusion_critical_dt(g, 0.5)
    u0 = np.random.default_rng(so).standard_normal((ny, nx)).astype(np.float32)
    got = diffusion(torch.from_numpy(u0).cuda(), (1.0, 1.5), so, 0.5, dt, 5).cpu().numpy()
    e = rel_l2(got, oracle.diffusion(g, u0.astype(np.float64), 0.5, dt, 5))
    print("strips so %d: rel L2 %.3e" % (so, e))
    assert e <= 1e-5
