"""The velocity and p fields set up four points at a time: the extension of a
physical velocity into the absorbing layers is the edge value (numpy's pad),
at rows of every remainder, with float32 p and with its 16-bit code.  Two
grids of the same padded velocity step to the same bits; the second is given
the padded field itself."""
import numpy as np
import pytest

from gpu_common import need_gpu, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [2, 3, 4, 13, 66, 259])
@pytest.mark.parametrize("nbl", [0, 1, 6])
@pytest.mark.parametrize("param", ["f32", "q16"])
def test_extended_velocity(nx, nbl, param):
    need_gpu()
    from paper_1906_10811_amd import Grid
    for shape in ((nx, 7, 5), (nx, 9)):
        if param == "q16" and len(shape) == 2:
            continue
        rng = np.random.default_rng(nx * 10 + nbl)
        v = rng.uniform(1500.0, 4000.0, tuple(reversed(shape))).astype(np.float32)
        full = np.pad(v, nbl, mode="edge")
        u0 = torch.from_numpy(rng.standard_normal(full.shape).astype(np.float32)).cuda()
        got = []
        for vel, flag in ((v, False), (full, True)):
            g = Grid(shape, (10.0,) * len(shape), torch.from_numpy(vel).cuda(), space_order=4, nbl=nbl, param=param,
                     vp_padded=flag)
            dt = 0.5 * g.critical_dt
            _, (u, um) = g.forward([], torch.zeros(2, 0, device="cuda"), [], dt, u0=u0, u_prev=u0, save_state=True)
            torch.cuda.synchronize()
            got.append((u, um))
            g.close()
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
        assert torch.isfinite(got[0][0]).all()
