"""The velocity extremes found at grid creation (they set the stability limit
and the scale of the 16-bit p codes): every position class of a row, ragged
rows, one workgroup and many; non-positive and non-finite values refused."""
import numpy as np
import pytest
import torch

from paper_1906_10811_amd import FDError, Grid

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2, 2), (5, 3, 2), (67, 9, 6), (259, 40, 33), (4, 130, 130)]


@pytest.mark.parametrize("shape", SHAPES)
def test_extremes_anywhere(shape):
    arr = tuple(reversed(shape))
    n = int(np.prod(arr))
    for hi, lo in ((n - 1, 0), (0, n - 1), (shape[0] - 1, n - shape[0])):
        v = torch.full((n,), 2000.0, device="cuda")
        v[hi] = 4321.5
        v[lo] = 1234.25
        g = Grid(shape, (10.0,) * 3, v.reshape(arr), space_order=4, param="q16")
        assert g.vmax == 4321.5
        dt = 0.5 * g.critical_dt
        g.forward([], torch.zeros(1, 0, device="cuda"), [], dt)
        p0, dp = g.param_scale()
        assert p0 == float(np.float32(dt * dt * 1234.25 ** 2))
        assert dp == float(np.float32(dt * dt * (4321.5 ** 2 - 1234.25 ** 2) / 65535.0))
        g.close()


@pytest.mark.parametrize("bad", [0.0, -1.0, float("nan"), float("inf")])
@pytest.mark.parametrize("shape", SHAPES)
def test_bad_velocity_is_refused(shape, bad):
    arr = tuple(reversed(shape))
    n = int(np.prod(arr))
    for at in (0, n // 2, n - 1):
        v = torch.full((n,), 2000.0, device="cuda")
        v[at] = bad
        with pytest.raises(FDError):
            Grid(shape, (10.0,) * 3, v.reshape(arr), space_order=4)
