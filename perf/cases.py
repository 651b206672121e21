"""The work that this library's performance is judged on.

Each case is one call (or one forward plus backward, or one batch of served
shots) through the public Python entry points, on seeded synthetic inputs.
The listed cases span the range of use: a 101 x 101 section where launches
and latency count, the thesis's diffusion sizes, the 336^3 and 592^3 padded
acoustic grids of the benchmark, odd sizes, every direction (forward,
adjoint, gradient, autograd) and the storage forms; `draw` gives others of
the same ranges.

A case holds: kind ("forward", "adjoint", "gradient", "modeling",
"diffusion" or "serve"), the physical points nx, ny, nz (ny = 0: 2D, axes x
and z), the space order so, the damping points nbl, the time steps nt, the
storage of the wavefields and of p = dt^2 v^2, the numbers of sources and
receivers, sinc (half-width of the windowed-sinc points, 0: multilinear),
state (the final wavefields are returned too), the medium ("layered" or
"random") and ckpt (gradient: steps between checkpoints).

`exact` evaluates the same definitions in float64 with plain torch.
"""
import math

import numpy as np
import torch

import paper_1906_10811_amd as fd

H = 10.0          # grid spacing, m
VMIN, VMAX = 1500.0, 4500.0
NU = 0.5          # diffusivity of the diffusion benchmark
COURANT = 0.38    # dt v_max / h, below the 3D limit of space order 16

_DEFAULTS = dict(ny=0, so=8, nbl=40, storage="f32", param="f32", nsrc=1, nrec=64, sinc=0, state=False,
                 medium="layered", ckpt=50)


def _case(name, kind, **kw):
    c = dict(name=name, kind=kind)
    c.update({k: v for k, v in _DEFAULTS.items()} if kind != "diffusion" else {})
    c.update(kw)
    return c


def listed():
    return [
        # the smallest section: a test or tutorial run, bound by launches
        _case("forward2d_101", "forward", nx=101, nz=101, so=4, nbl=0, nt=200, nrec=101),
        # one shot of a 2D survey line, a section of 24 x 12 km
        _case("forward2d_2401", "forward", nx=2401, nz=1201, so=8, nt=300, nrec=401, state=True),
        # one 2D inversion step: loss, backward to the velocity and the wavelet
        _case("modeling2d_301", "modeling", nx=301, nz=151, so=4, nbl=30, nt=400, nrec=151),
        # the smallest 3D box: smoke tests, interactive use
        _case("forward3d_48", "forward", nx=48, ny=40, nz=36, nbl=6, nt=80, nrec=24, state=True),
        # the headline model (336^3 padded), one shot; the state is kept to
        # continue the run
        _case("forward3d_256", "forward", nx=256, ny=256, nz=256, nt=200, nrec=256, state=True),
        # the largest grid (592^3 padded) in the narrowest storage
        _case("forward3d_512_bf16_q16", "forward", nx=512, ny=512, nz=512, nt=100, nrec=512, storage="bf16",
              param="q16", medium="random"),
        # odd sizes, windowed-sinc points, high order, value and difference
        # kept in half precision
        _case("forward3d_odd_f16diff", "forward", nx=187, ny=143, nz=101, so=12, nbl=21, nt=150, nsrc=3, nrec=93,
              sinc=4, storage="f16_diff", state=True),
        # back-propagation of recorded residuals (reverse-time migration), low order
        _case("adjoint3d_192", "adjoint", nx=192, ny=192, nz=192, so=4, nt=200, nrec=192),
        # one 3D inversion gradient with checkpoints
        _case("gradient3d_200", "gradient", nx=200, ny=200, nz=200, nt=200, nrec=200),
        # the thesis's diffusion benchmark at its two sizes
        _case("diffusion_2500_so2", "diffusion", nx=2500, nz=2500, so=2, nt=200),
        _case("diffusion_10000_so8", "diffusion", nx=10000, nz=10000, so=8, nt=100),
        # four shots of different grids queued at once on the shot server
        _case("serve_4", "serve", nx=128, ny=128, nz=128, nt=150, nrec=128, shots=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _steps(points, lo, hi, budget, rng):
    """Time steps between lo and hi, fewer where points x steps would exceed budget."""
    return max(8, min(rng.randint(lo, hi), int(budget / points)))


def draw(rng):
    kind = rng.choice(["forward2d", "forward2d", "modeling", "forward3d", "forward3d", "forward3d", "forward3d",
                       "adjoint", "gradient", "diffusion", "diffusion", "serve"])
    so = 2 * rng.randint(1, 8)
    c = dict(_DEFAULTS)
    if kind == "forward2d":
        nx, nz, nbl = _log(rng, 101, 4001), _log(rng, 101, 2001), rng.choice([0, 20, 40])
        pts = (nx + 2 * nbl) * (nz + 2 * nbl)
        return dict(c, kind="forward", nx=nx, nz=nz, so=so, nbl=nbl, nt=_steps(pts, 150, 400, 3e9, rng),
                    nsrc=rng.randint(1, 4), nrec=min(nx, rng.randint(16, 401)), state=rng.random() < 0.5,
                    storage=rng.choice(["f32", "f32", "f32", "bf16"]), medium=rng.choice(["layered", "random"]))
    if kind == "modeling":
        nx, nz, nbl = _log(rng, 101, 501), _log(rng, 81, 301), rng.choice([20, 30, 40])
        return dict(c, kind="modeling", nx=nx, nz=nz, so=2 * rng.randint(1, 4), nbl=nbl, nt=rng.randint(150, 400),
                    nrec=rng.randint(16, 151), ckpt=rng.choice([25, 50, 100]))
    if kind in ("forward3d", "adjoint", "gradient"):
        top = {"forward3d": 512, "adjoint": 256, "gradient": 220}[kind]
        nbl = rng.choice([10, 21, 40])
        n = [min(top, max(36, int(_log(rng, 40, top) * rng.uniform(0.7, 1.3)))) for _ in range(3)]
        pts = math.prod(a + 2 * nbl for a in n)
        c.update(nx=n[0], ny=n[1], nz=n[2], nbl=nbl, so=so, nrec=rng.randint(24, 512), nsrc=rng.randint(1, 3),
                 medium=rng.choice(["layered", "random"]))
        if kind == "gradient":
            return dict(c, kind=kind, so=min(so, 12), ckpt=rng.choice([25, 50]), nt=_steps(pts, 60, 200, 4e9, rng))
        if kind == "adjoint":
            return dict(c, kind=kind, nt=_steps(pts, 60, 200, 8e9, rng))
        return dict(c, kind="forward", nt=_steps(pts, 60, 200, 1e10, rng), state=rng.random() < 0.5,
                    sinc=rng.choice([0, 0, 0, 4]), param=rng.choice(["f32", "f32", "q16"]),
                    storage=rng.choice(["f32", "f32", "f32", "bf16", "f16", "bf16_diff", "f16_diff"]))
    if kind == "diffusion":
        nx, nz = _log(rng, 200, 10000), _log(rng, 200, 10000)
        return dict(kind=kind, nx=nx, nz=nz, so=so, nt=_steps(nx * nz, 50, 250, 1e10, rng))
    n = [rng.randint(64, 144) for _ in range(3)]
    return dict(c, kind="serve", nx=n[0], ny=n[1], nz=n[2], so=2 * rng.randint(2, 6), nt=rng.randint(80, 150),
                nrec=rng.randint(24, 128), shots=rng.randint(2, 4))


# ------------------------------------------------------------------ inputs
def _shape(c):
    return (c["nx"], c["ny"], c["nz"]) if c["ny"] else (c["nx"], c["nz"])


def _dt():
    return COURANT * H / VMAX


def _gen(seed, device):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed) % (1 << 62))
    return g


def _velocity(shape, medium, seed, device):
    """float32 velocity, slowest axis first: ten layers at random depths, or
    a smooth random field of 200 m correlation length, 1.5 to 4.5 km/s."""
    arr = tuple(reversed(shape))
    rng = np.random.default_rng(seed)
    if medium == "layered":
        nz = arr[0]
        faces = np.sort(rng.uniform(0.0, nz, 9))
        vz = VMIN + (VMAX - VMIN) * np.searchsorted(faces, np.arange(nz), side="right") / 9.0
        v = torch.from_numpy(vz.astype(np.float32)).to(device)
        return v.reshape((nz,) + (1,) * (len(arr) - 1)).expand(arr).contiguous()
    coarse = tuple(max(2, n // 20 + 2) for n in arr)
    noise = torch.randn((1, 1) + coarse, generator=_gen(seed, device), device=device)
    f = torch.nn.functional.interpolate(noise, size=arr, mode="trilinear" if len(arr) == 3 else "bilinear",
                                        align_corners=True)[0, 0]
    lo, hi = f.min(), f.max()
    return (VMIN + (VMAX - VMIN) * (f - lo) / (hi - lo)).contiguous()


def _geometry(shape, nsrc, nrec, seed):
    """Off-grid sources near the top of the middle, a receiver line along x at 20 m depth."""
    rng = np.random.default_rng(seed + 77)
    ext = [(n - 1) * H for n in shape]
    src = np.empty((nsrc, len(shape)))
    for s in range(nsrc):
        for a in range(len(shape) - 1):
            src[s, a] = ext[a] * rng.uniform(0.35, 0.65)
        src[s, -1] = rng.uniform(20.0, 60.0)
    rec = np.empty((nrec, len(shape)))
    rec[:, 0] = np.linspace(0.0, ext[0], nrec)
    if len(shape) == 3:
        rec[:, 1] = src[0, 1] + rng.uniform(-5.0, 5.0)
    rec[:, -1] = 20.0
    return src, rec


def _ricker(nt, n, seed):
    """[nt, n] Ricker wavelets about 15 Hz, float32."""
    rng = np.random.default_rng(seed + 5)
    f = 15.0 * rng.uniform(0.9, 1.1, n)
    a = (math.pi * f * (np.arange(nt)[:, None] * _dt() - 0.5 / f)) ** 2
    return ((1.0 - 2.0 * a) * np.exp(-a) * rng.uniform(0.5, 1.5, n)).astype(np.float32)


def _traces(nt, n, seed, device, amp):
    """[nt, n] smooth oscillating traces (recorded data or residuals)."""
    g = _gen(seed + 9, device)
    x = torch.randn(nt + 8, n, generator=g, device=device).cumsum(0)
    x = x[8:] - 0.125 * sum(x[i:nt + i] for i in range(8))
    return (amp * x).float().contiguous()


def _hat(c, seed, device):
    """Hat function (2 inside a random box, 1 outside) with small noise."""
    rng = np.random.default_rng(seed)
    u = 1.0 + 0.01 * torch.randn(c["nz"], c["nx"], generator=_gen(seed, device), device=device)
    x0, z0 = int(c["nx"] * rng.uniform(0.2, 0.5)), int(c["nz"] * rng.uniform(0.2, 0.5))
    u[z0:z0 + c["nz"] // 4, x0:x0 + c["nx"] // 4] += 1.0
    return u


def _shots(c, seed):
    """The served requests: grids of different shapes, all fields on the host."""
    out = []
    for i in range(c["shots"]):
        shape = (c["nx"] + 32 * (i % 2), c["ny"] + 16 * (i % 3), c["nz"] + 24 * (i // 2))
        so = (c["so"], 4, 12, 8)[i % 4]
        s = seed * 31 + i
        src, rec = _geometry(shape, c["nsrc"], c["nrec"], s)
        out.append(dict(shape=shape, so=so, seed=s, src=src, rec=rec, wav=_ricker(c["nt"], c["nsrc"], s)))
    return out


def _diffusion_dt(c):
    w = _weights(c["so"] // 2)
    return 0.8 / (2.0 * NU * sum(w[j] for j in range(1, len(w), 2)) * 2.0 / (H * H))


def prepare(case, seed):
    c = case
    dev = torch.device("cuda")
    k = c["kind"]
    if k == "diffusion":
        return dict(c=c, u0=_hat(c, seed, dev), dt=_diffusion_dt(c))
    if k == "serve":
        reqs = []
        for s in _shots(c, seed):
            vp = _velocity(s["shape"], c["medium"], s["seed"], "cpu").numpy()
            reqs.append(dict(shape=s["shape"], spacing=(H,) * 3, space_order=s["so"], nbl=c["nbl"], vp=vp,
                             src_xyz=s["src"], wavelet=s["wav"], rec_xyz=s["rec"], dt=_dt(), storage=c["storage"]))
        budget = sum(fd.Server.request_bytes(**r) for r in reqs) + (64 << 20)
        return dict(c=c, reqs=reqs, server=fd.Server(budget, max_slots=4))
    shape = _shape(c)
    src, rec = _geometry(shape, c["nsrc"], c["nrec"], seed)
    s = dict(c=c, src=src, rec=rec, dt=_dt())
    v = _velocity(shape, c["medium"], seed, dev)
    s["wav"] = torch.from_numpy(_ricker(c["nt"], c["nsrc"], seed)).to(dev)
    if k == "modeling":
        s["shape"] = shape
        s["vp"] = _edge(v, c["nbl"]).requires_grad_(True)
        s["wav"].requires_grad_(True)
        s["obs"] = _traces(c["nt"], c["nrec"], seed, dev, 3e-2)
        return s
    s["grid"] = fd.Grid(shape, (H,) * len(shape), v, space_order=c["so"], nbl=c["nbl"], storage=c["storage"],
                        param=c["param"], sinc_radius=c["sinc"], max_src=max(4, c["nsrc"]), max_rec=512)
    if k != "forward":
        s["obs"] = _traces(c["nt"], c["nrec"], seed, dev, 5e-4)
    return s


def run(state):
    s = state
    c = s["c"]
    k = c["kind"]
    if k == "diffusion":
        return fd.diffusion(s["u0"], (H, H), c["so"], NU, s["dt"], c["nt"])
    if k == "serve":
        tickets = [s["server"].submit(**r) for r in s["reqs"]]
        return [s["server"].wait(t)[0] for t in tickets]
    if k == "modeling":
        rec = fd.modeling(s["vp"], s["wav"], s["shape"], (H,) * len(s["shape"]), c["so"], c["nbl"], s["src"],
                          s["rec"], s["dt"], checkpoint_every=c["ckpt"])
        loss = 0.5 * ((rec - s["obs"]) ** 2).sum()
        gv, gw = torch.autograd.grad(loss, (s["vp"], s["wav"]))
        return rec.detach(), gv, gw
    g = s["grid"]
    if k == "forward":
        out = g.forward(s["src"], s["wav"], s["rec"], s["dt"], save_state=c["state"])
        return (out[0], *out[1]) if c["state"] else out
    if k == "adjoint":
        return g.adjoint(s["src"], s["rec"], s["obs"], s["dt"])
    misfit, grad, rec, _ = g.gradient(s["src"], s["wav"], s["rec"], s["obs"], s["dt"], checkpoint_every=c["ckpt"])
    return misfit, grad, rec


# -------------------------------------------------------------------- work
def _acoustic_work(shape, so, nbl, nt, sweeps):
    pts = math.prod(n + 2 * nbl for n in shape)
    flops = pts * nt * sweeps * (3.0 * len(shape) * (so // 2) + 12.0)
    return pts, math.prod(shape), flops


def work(case):
    """Inputs read once and outputs written once; the arithmetic of every
    step (3 operations per radius and axis, 12 for the centre and the update)."""
    c = case
    if c["kind"] == "diffusion":
        n = c["nx"] * c["nz"]
        return dict(bytes=8.0 * n, flops=n * c["nt"] * (3.0 * c["so"] + 3.0))
    tr = 4.0 * c["nt"] * (c["nrec"] + c["nsrc"])
    if c["kind"] == "serve":
        b = f = 0.0
        for s in _shots(c, 0):
            _, phys, fl = _acoustic_work(s["shape"], s["so"], c["nbl"], c["nt"], 1)
            b, f = b + 4.0 * phys + tr, f + fl
        return dict(bytes=b, flops=f)
    sweeps = 2 if c["kind"] in ("gradient", "modeling") else 1
    pts, phys, flops = _acoustic_work(_shape(c), c["so"], c["nbl"], c["nt"], sweeps)
    if c["kind"] == "forward":
        return dict(bytes=4.0 * phys + tr + (8.0 * pts if c["state"] else 0.0), flops=flops)
    if c["kind"] == "adjoint":
        return dict(bytes=4.0 * phys + tr, flops=flops)
    if c["kind"] == "gradient":
        return dict(bytes=4.0 * phys + 2.0 * tr + 8.0 * pts, flops=flops)
    return dict(bytes=8.0 * pts + 3.0 * tr, flops=flops)


# ------------------------------------------------------------------- exact
def _weights(r):
    f = math.factorial
    c = [0.0] + [2.0 * (-1) ** (j + 1) * f(r) ** 2 / (j * j * f(r - j) * f(r + j)) for j in range(1, r + 1)]
    c[0] = -2.0 * sum(c[1:])
    return c


def _edge(v, n):
    """v with n points of edge replication on every face."""
    for a in range(v.dim()):
        i = torch.arange(-n, v.shape[a] + n, device=v.device).clamp(0, v.shape[a] - 1)
        v = v.index_select(a, i)
    return v.contiguous()


class _Exact:
    """The stepper in float64: fields carry r zero cells on every face."""

    def __init__(self, shape, so, nbl, vp, dt):
        self.dev, self.dt, self.r = vp.device, dt, so // 2
        self.n = [k + 2 * nbl for k in reversed(shape)]
        self.nd = len(shape)
        self.cell = H ** self.nd
        self.shape, self.nbl = shape, nbl
        self.v2 = vp.double() ** 2
        self.w = [x / (H * H) for x in _weights(self.r)]
        smax = 3.0 * float(vp.max()) * math.log(1000.0) / (2.0 * nbl * H) if nbl else 0.0
        self.s = torch.zeros(self.n, dtype=torch.float64, device=self.dev)
        for a, k in enumerate(self.n):
            i = torch.arange(k, device=self.dev, dtype=torch.float64)
            d = torch.clamp(torch.maximum(nbl - i, i - (k - 1 - nbl)), min=0.0) / max(nbl, 1)
            self.s += (smax * dt / 2.0 * d * d).reshape([-1 if b == a else 1 for b in range(self.nd)])

    def field(self):
        return torch.zeros([k + 2 * self.r for k in self.n], dtype=torch.float64, device=self.dev)

    def inner(self, u):
        return u[tuple(slice(self.r, self.r + k) for k in self.n)]

    def points(self, xyz, sinc):
        """Flat indices into a grid-sized array and weights, [points, nodes]."""
        idx, wts = [], []
        for p in xyz:
            i = torch.zeros(1, dtype=torch.int64)
            w = torch.ones(1, dtype=torch.float64)
            for a in reversed(range(self.nd)):        # slowest grid axis first
                t, n = p[a] / H, self.shape[a]
                if sinc:
                    k = np.floor(t) - sinc + 1 + np.arange(2 * sinc)
                    d = k - t
                    b = math.pi * sinc / 2.0
                    wa = np.sinc(d) * np.i0(b * np.sqrt(np.maximum(0.0, 1.0 - (d / sinc) ** 2))) / np.i0(b)
                else:
                    k0 = min(int(np.floor(t)), n - 2)
                    k, wa = np.array([k0, k0 + 1.0]), np.array([1.0 - (t - k0), t - k0])
                k = k.astype(np.int64) + self.nbl
                full = n + 2 * self.nbl
                wa = np.where((k >= 0) & (k < full), wa, 0.0)
                k = np.clip(k, 0, full - 1)
                i = (i[:, None] * full + torch.from_numpy(k)[None, :]).reshape(-1)
                w = (w[:, None] * torch.from_numpy(wa)[None, :]).reshape(-1)
            idx.append(i)
            wts.append(w)
        return torch.stack(idx).to(self.dev), torch.stack(wts).to(self.dev)

    def step(self, u, um, inject):
        """The new level written over um; inject adds to the Laplacian's flat array."""
        lap = torch.mul(self.inner(u), self.nd * self.w[0])
        for a, k in enumerate(self.n):
            v = u
            for b, kb in enumerate(self.n):
                if b != a:
                    v = v.narrow(b, self.r, kb)
            for j in range(1, self.r + 1):
                lap.add_(v.narrow(a, self.r + j, k), alpha=self.w[j])
                lap.add_(v.narrow(a, self.r - j, k), alpha=self.w[j])
        inject(lap.view(-1))
        lap.mul_(self.v2).mul_(self.dt ** 2)
        old = self.inner(um)
        new = lap.add_(self.inner(u), alpha=2.0).sub_(old).addcmul_(self.s, old).div_(1.0 + self.s)
        old.copy_(new)

    def sample(self, u, pts):
        return (self.inner(u).reshape(-1)[pts[0]] * pts[1]).sum(1) if self.nd < 3 else self._sample3(u, pts)

    def _sample3(self, u, pts):
        n = self.n
        z, y, x = pts[0] // (n[1] * n[2]), pts[0] // n[2] % n[1], pts[0] % n[2]
        return (u[z + self.r, y + self.r, x + self.r] * pts[1]).sum(1)

    def forward(self, wav, src, rec, brackets=None):
        u, um = self.field(), self.field()
        out = []
        for n in range(wav.shape[0]):
            q = (src[1] * (wav[n] / self.cell)[:, None]).reshape(-1)
            old = self.inner(um).clone() if brackets is not None else None
            self.step(u, um, lambda lap: lap.index_add_(0, src[0].reshape(-1), q))
            if brackets is not None:
                new = self.inner(um)
                brackets.append(new - 2.0 * self.inner(u) + old + self.s * (new - old))
            u, um = um, u
            out.append(self.sample(u, rec))
        return torch.stack(out), self.inner(u), self.inner(um)

    def adjoint(self, resid, src, rec, brackets=None):
        """F^T resid, and the gradient in m when the brackets are given."""
        u, um = self.field(), self.field()
        g = torch.zeros(self.n, dtype=torch.float64, device=self.dev) if brackets is not None else None
        out = [None] * resid.shape[0]
        for n in reversed(range(resid.shape[0])):
            q = (rec[1] * (resid[n] / self.dt ** 2)[:, None]).reshape(-1)
            self.step(u, um, lambda lap: lap.index_add_(0, rec[0].reshape(-1), q))
            u, um = um, u
            out[n] = self.sample(u, src) * (self.dt ** 2 / self.cell)
            if brackets is not None:
                g.addcmul_(self.inner(u), brackets[n], value=-1.0)
        return torch.stack(out), g


def _exact_diffusion(c, u0):
    r, dt = c["so"] // 2, _diffusion_dt(c)
    w = [NU * dt * x / (H * H) for x in _weights(r)]
    nz, nx = u0.shape
    u = torch.zeros(nz + 2 * r, nx + 2 * r, dtype=torch.float64, device=u0.device)
    inner = u[r:r + nz, r:r + nx]
    inner.copy_(u0)
    for _ in range(c["nt"]):
        d = torch.mul(inner, 2.0 * w[0])
        for j in range(1, r + 1):
            for k in (r + j, r - j):
                d.add_(u[k:k + nz, r:r + nx], alpha=w[j])
                d.add_(u[r:r + nz, k:k + nx], alpha=w[j])
        inner.add_(d)
    return inner.clone()


def exact(case, seed):
    c = case
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    k = c["kind"]
    if k == "diffusion":
        return _exact_diffusion(c, _hat(c, seed, dev))
    if k == "serve":
        out = []
        for s in _shots(c, seed):
            v = _velocity(s["shape"], c["medium"], s["seed"], "cpu").to(dev)
            e = _Exact(s["shape"], s["so"], c["nbl"], _edge(v, c["nbl"]), _dt())
            out.append(e.forward(torch.from_numpy(s["wav"]).to(dev).double(), e.points(s["src"], 0),
                                 e.points(s["rec"], 0))[0].cpu().numpy())
        return out
    shape = _shape(c)
    src, rec = _geometry(shape, c["nsrc"], c["nrec"], seed)
    v = _edge(_velocity(shape, c["medium"], seed, dev), c["nbl"])
    e = _Exact(shape, c["so"], c["nbl"], v, _dt())
    ps, pr = e.points(src, c["sinc"]), e.points(rec, c["sinc"])
    wav = torch.from_numpy(_ricker(c["nt"], c["nsrc"], seed)).to(dev).double()
    if k == "forward":
        out = e.forward(wav, ps, pr)
        return out if c["state"] else out[0]
    if k == "adjoint":
        return e.adjoint(_traces(c["nt"], c["nrec"], seed, dev, 5e-4).double(), ps, pr)[0]
    br = []
    tr = e.forward(wav, ps, pr, br)[0]
    obs = _traces(c["nt"], c["nrec"], seed, dev, 3e-2 if k == "modeling" else 5e-4).double()
    gw, gm = e.adjoint(tr - obs, ps, pr, br)
    if k == "modeling":
        return tr, -2.0 * gm / v.double() ** 3, gw
    return 0.5 * ((tr - obs) ** 2).sum().reshape(1), gm, tr
