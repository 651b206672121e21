"""One diffusion level per launch where it has a kernel or a launch shape of
its own (fields beyond 128 MB, radius 8, many waves at radius 1 and 2): bit
for bit the levels taken several at a time, on ragged grids."""
import pytest

from gpu_common import need_gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(6001, 5990), (34567, 1003), (4601, 4502), (2601, 2603), (2099, 2201), (1533, 1405)])
@pytest.mark.parametrize("so", [2, 4, 8, 12, 16])
def test_single_levels(shape, so):
    need_gpu()
    from paper_1906_10811_amd import diffusion, diffusion_dt_limit
    gen = torch.Generator(device="cuda")
    gen.manual_seed(so)
    u0 = torch.randn(shape[1], shape[0], generator=gen, device="cuda")
    dt = 0.9 * diffusion_dt_limit(shape, (1.0, 1.0), so, 0.5)
    want = diffusion(u0, (1.0, 1.0), so, 0.5, dt, 8)
    assert torch.equal(diffusion(u0, (1.0, 1.0), so, 0.5, dt, 8, time_block=1), want)
    assert torch.isfinite(want).all() and not torch.equal(want, u0)
