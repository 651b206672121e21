"""16-bit 3D fields at so 10 to 16: the kernels that read float32 p with
ordinary loads (grids whose p fits the memory-side cache), those that read it
past the cache (larger grids) and those of the mixed tile shape give bitwise
the same fields.  A wave that stays inside a box is stepped on the box and on
a grid that holds the box and is beyond the line."""
import pytest

from gpu_common import need_gpu, torch

pytestmark = pytest.mark.gpu
SMALL, LARGE, AT = (90, 101, 97), (340, 300, 340), (128, 66, 91)   # the box, the grid, where it lies
NT = 3


def _field(shape, box):
    x = torch.zeros(tuple(reversed(shape)), device="cuda")
    (nx, ny, nz), (x0, y0, z0) = SMALL, AT if shape == LARGE else (0, 0, 0)
    x[z0:z0 + nz, y0:y0 + ny, x0:x0 + nx] = box
    return x


def _box(shape, f):
    (nx, ny, nz), (x0, y0, z0) = SMALL, AT if shape == LARGE else (0, 0, 0)
    return f[z0:z0 + nz, y0:y0 + ny, x0:x0 + nx].clone()


@pytest.mark.parametrize("so", [10, 12, 14, 16])
@pytest.mark.parametrize("storage", ["f16", "bf16", "f16_diff", "bf16_diff"])
def test_box_equals_grid(so, storage):
    need_gpu()
    from paper_1906_10811_amd import Grid
    gen = torch.Generator(device="cuda").manual_seed(so)
    v = 1500.0 + 2900.0 * torch.rand(tuple(reversed(SMALL)), generator=gen, device="cuda")
    v[50, 50, 45] = 4500.0
    u = torch.zeros_like(v)
    u[30:67, 31:70, 30:60] = torch.randn(37, 39, 30, generator=gen, device="cuda")
    wav = torch.randn(NT, 1, generator=gen, device="cuda")
    out = []
    for shape, tile_x in ((SMALL, 0), (LARGE, 0), (SMALL, 96), (SMALL, 64)):
        o = [10.0 * k for k in AT] if shape == LARGE else [0.0] * 3
        vel = _field(shape, v)
        vel[vel == 0] = 1500.0
        u0 = _field(shape, u)
        g = Grid(shape, (10.0,) * 3, vel, space_order=so, storage=storage, tile_x=tile_x)
        src, rec = [[443.0 + o[0], 512.0 + o[1], 480.0 + o[2]]], [[450.0 + o[0], 501.0 + o[1], 455.0 + o[2]]]
        r, s = g.forward(src, wav, rec, 0.38 * 10.0 / 4500.0, u0=u0, u_prev=u0, save_state=True)
        torch.cuda.synchronize()
        out.append((r, _box(shape, s[0]), _box(shape, s[1])))
        g.close()
    assert float(out[0][1].abs().max()) > 0.0
    for k, got in enumerate(out[1:]):
        for i, (a, b) in enumerate(zip(got, out[0])):
            assert torch.isfinite(a).all() and torch.equal(a, b), (k, i)
