"""Dense fields in and out of the pitched layout four points at a time: rows of
every remainder, base addresses on and off 16-byte boundaries, every storage.
With no time steps the state comes back as stored: exactly the input in
float32, the input rounded once to 16 bits (scale 1 here) otherwise."""
import pytest

from gpu_common import need_gpu, torch

pytestmark = pytest.mark.gpu


def _at(t, shift):
    """The same values, contiguous, `shift` floats past an aligned address."""
    buf = torch.empty(t.numel() + 4, dtype=torch.float32, device=t.device)
    out = buf[shift:shift + t.numel()].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("nx", [2, 5, 32, 67, 259, 1024])
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16", "f16_diff", "bf16_diff"])
def test_state_round_trip(nx, storage):
    need_gpu()
    from paper_1906_10811_amd import Grid
    dev = torch.device("cuda")
    half = {"f32": torch.float32, "f16": torch.float16}.get(storage.split("_")[0], torch.bfloat16)
    for shape in ((nx, 6, 5), (nx, 9)):
        if storage.endswith("_diff") and len(shape) == 2:
            continue
        v = torch.full(tuple(reversed(shape)), 2000.0, device=dev)
        g = Grid(shape, (10.0,) * len(shape), v, space_order=4, storage=storage, amp_scale=1.0)
        gen = torch.Generator(device=dev)
        gen.manual_seed(nx)
        a = torch.randn(g.array_shape, generator=gen, device=dev)
        b = torch.randn(g.array_shape, generator=gen, device=dev)
        for shift in (0, 1, 2):
            _, (u, um) = g.forward([], torch.zeros(0, 0, device=dev), [], 1e-3, u0=_at(a, shift), u_prev=_at(b, shift),
                                   save_state=True)
            torch.cuda.synchronize()
            ra = a.to(half).float()
            assert torch.equal(u, ra)
            want = ra - (a - b).to(half).float() if storage.endswith("_diff") else b.to(half).float()
            assert torch.equal(um, want)
        g.close()


@pytest.mark.parametrize("nx", [5, 64, 66])
def test_diffusion_on_shifted_addresses(nx):
    need_gpu()
    from paper_1906_10811_amd import diffusion, diffusion_dt_limit
    u0 = torch.randn(70, nx, device="cuda")
    dt = 0.9 * diffusion_dt_limit((nx, 70), (1.0, 1.0), 4, 0.5)
    want = diffusion(u0, (1.0, 1.0), 4, 0.5, dt, 9)
    for shift in (1, 2, 3):
        out = _at(torch.zeros_like(u0), shift)
        diffusion(_at(u0, shift), (1.0, 1.0), 4, 0.5, dt, 9, out=out)
        assert torch.equal(out, want)
