"""The 3D gradient's reverse sweep accumulates three levels per imaging step
where a segment and the fold allow it (kImage3).  The binomial schedule images
every level in a step of its own; the products and their order are the same,
so both gradients are bitwise equal: every radius and tile shape, ragged
edges, segments that leave one or two levels over, and a run across a fold."""
import pytest

from gpu_common import case, gpu_grid, need_gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("so", [2, 4, 6, 8, 10, 12, 14, 16])
@pytest.mark.parametrize("tile_x", [64, 32, 96])
def test_three_levels_equal_single_levels(so, tile_x):
    need_gpu()
    c = case((71, 35, 18), so, 2, 37, seed=so, nsrc=2, nrec=5)
    dev = torch.device("cuda:0")
    g = gpu_grid(c, tile_x=tile_x)
    wav = torch.from_numpy(c["wav"]).to(dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(so)
    obs = 1e-3 * torch.randn(37, len(c["rec"]), generator=gen, device=dev)
    want = g.gradient(c["src"], wav, c["rec"], obs, c["dt"], binomial_slots=3, want_src_adj=True)
    for every in (4, 5, 37):
        got = g.gradient(c["src"], wav, c["rec"], obs, c["dt"], checkpoint_every=every, want_src_adj=True)
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(zip(got, want)):
            assert torch.isfinite(b).all() and torch.equal(a, b), (so, tile_x, every, i)
    assert float(want[1].abs().max()) > 0.0
    g.close()
