"""Every diffusion kernel and level count that large and narrow grids take,
against float64 steps in plain torch on the same input.

Tolerance: a float32 step sums 4 R + 3 terms whose weights have the absolute
sum A, so it errs by at most (4 R + 4) A 2^-24 of the field in the 2-norm, the
rounding of the weights included, and a stable step does not amplify what came
before."""
import pytest

import oracle
from gpu_common import need_gpu, torch

pytestmark = pytest.mark.gpu
H, NU = (1.0, 1.5), 0.5
CASES = [  # nx, ny, so: the kernel of 9 steps (strips: levels per launch)
    (3000, 3001, 2), (3000, 6000, 4), (4003, 4001, 6), (3000, 6000, 8),      # strips 8, 8, 4, 4
    (2300, 3001, 10), (2300, 3001, 12), (2300, 3001, 14), (6001, 5990, 16),  # strips 2
    (4601, 4502, 16),                                                        # strips 1
    (2502, 2499, 16), (6001, 5990, 12),                                      # single levels of whole tiles (12: the last)
    (8, 1000001, 2), (64, 125000, 4), (99, 80001, 6), (260, 30001, 8), (48, 170000, 10),   # narrow: tiles
    (8, 380001, 12), (500, 10001, 12), (261, 30001, 14), (241, 90001, 16)]   # narrow: single levels


def _steps64(u, r, dt, nt):
    c = torch.zeros(r + 1, dtype=torch.float64)
    w = oracle.fd_weights(2 * r)
    c[:] = torch.tensor([float(x) for x in w], dtype=torch.float64)
    k = [NU * dt / (h * h) for h in H]
    ny, nx = u.shape
    for _ in range(nt):
        p = torch.nn.functional.pad(u, (r, r, r, r))
        v = u + c[0].item() * (k[0] + k[1]) * u
        for j in range(1, r + 1):
            v += c[j].item() * k[0] * (p[r:r + ny, r + j:r + j + nx] + p[r:r + ny, r - j:r - j + nx])
            v += c[j].item() * k[1] * (p[r + j:r + j + ny, r:r + nx] + p[r - j:r - j + ny, r:r + nx])
        u = v
    a = abs(1.0 + c[0].item() * (k[0] + k[1])) + 2.0 * float(c[1:].abs().sum()) * (k[0] + k[1])
    return u, a


@pytest.mark.parametrize("nx,ny,so", CASES)
def test_kernel_against_float64(nx, ny, so):
    need_gpu()
    from paper_1906_10811_amd import diffusion, diffusion_dt_limit
    r, nt = so // 2, 9
    gen = torch.Generator(device="cuda").manual_seed(so)
    u0 = torch.randn(ny, nx, generator=gen, device="cuda")
    dt = 0.8 * diffusion_dt_limit((nx, ny), H, so, NU)
    want, a = _steps64(u0.double(), r, dt, nt)
    for time_block in (0, 1):
        got = diffusion(u0, H, so, NU, dt, nt, time_block=time_block).double()
        e = float((got - want).norm() / want.norm())
        tol = nt * (4 * r + 4) * a * 2.0 ** -24 * float(u0.norm()) / float(want.norm())
        print("%d x %d so %d time_block %d: rel L2 %.2e (bound %.2e)" % (nx, ny, so, time_block, e, tol), flush=True)
        assert e <= tol
