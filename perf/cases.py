"""The work that a user of the library has it do, as cases to be timed and compared.

A case is a dict of plain values:

  kind      what one pass does (see run)
  n_mesh    particle-mesh side
  ratio     mesh cells per compression cell and axis (n_cell = n_mesh / ratio)
  n_cdm     cold-dark-matter lattice side (n_cdm^3 particles)
  n_nu      neutrino count per side (n_nu^3 particles), 0 for no neutrinos
  pos, vel  code bytes per axis of the compressed format
  slope     slope of the initial power spectrum
  dt        time step
  steps     steps of a pass

The sizes are those of the repository's workloads (the 64^3 float box, the 256^3 box of
two species, the 128^3 differentiable box, the 1024^3 tile) and of their recipes at other
sizes: the tile's is n_cdm = n_mesh / 4 on 4 mesh cells per compression cell with 8
neutrinos per cold particle, the two-species box's n_cdm = n_mesh / 2 on 2. Inputs follow
the same recipes (a displaced lattice with a power-law spectrum, uniform neutrinos with
Fermi-Dirac speeds), drawn on the GPU.
"""

import math

import numpy as np
import torch

from paper_1611_01545_amd import PMContext
from paper_1611_01545_amd.autodiff import density_loss, trajectory
from paper_1611_01545_amd.pm import widths_word

DEV = "cuda"


def _case(kind, n_mesh, ratio, n_cdm, n_nu, pos=1, vel=2, slope=-1.0, dt=0.005, steps=1):
    return {"kind": kind, "n_mesh": n_mesh, "ratio": ratio, "n_cdm": n_cdm, "n_nu": n_nu,
            "pos": pos, "vel": vel, "slope": slope, "dt": dt, "steps": steps}


def listed():
    cases = [
        # an uncompressed test box: the smallest step, where launches and host time count
        ("float_step_64", _case("float_step", 64, 4, 32, 0, slope=-2.0, dt=0.01)),
        # the compressed step at the size of a test or a tutorial: all latency
        ("step_64", _case("step", 64, 4, 16, 32)),
        # the ordinary production step of two species; mesh and particles fit the cache
        ("step_256", _case("step", 256, 2, 128, 256, slope=-1.5, dt=0.01)),
        # particle counts that are no power of two, with the wide (2 + 2 byte) codes
        ("step_512_wide", _case("step", 512, 4, 121, 243, pos=2)),
        # the largest step of which several states fit the card: the memory-bound regime
        ("step_1024", _case("step", 1024, 4, 256, 512)),
        # the two-level force with the particle-particle term: the method's full step
        ("p3m_512", _case("p3m", 512, 4, 128, 256)),
        # gradient of a density loss through ten compressed steps: an inference loop's pass
        ("trajectory_128", _case("trajectory", 128, 4, 64, 0, slope=-2.0, dt=0.02, steps=10)),
        # one adjoint step at a size where memory counts
        ("vjp_512", _case("vjp", 512, 4, 128, 256)),
        # density and force meshes for analysis, without a step
        ("force_512", _case("force", 512, 4, 128, 256)),
        # start of a run: float initial conditions into the compressed format
        ("encode_256", _case("encode", 256, 2, 128, 256, slope=-1.5)),
        # a checkpoint written: compressed state to a byte stream on the host
        ("save_256", _case("save", 256, 2, 128, 256, slope=-1.5)),
        # and read back: host bytes to a compressed state, decoded for analysis
        ("restart_256", _case("restart", 256, 2, 128, 256, slope=-1.5)),
    ]
    return [dict(c, name=name) for name, c in cases]


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "float_step", "p3m", "trajectory",
                       "vjp", "force", "encode", "save", "restart"])
    top = {"step": 1024, "float_step": 256, "p3m": 512, "trajectory": 128, "vjp": 512,
           "force": 512, "encode": 256, "save": 256, "restart": 256}[kind]
    low = 128 if kind == "p3m" else 64
    n_mesh = rng.choice([n for n in (64, 128, 256, 512, 1024) if low <= n <= top])
    ratio = 4 if n_mesh >= 512 or kind == "p3m" else rng.choice([2, 4])
    # the lattice side about n_mesh / ratio, log-uniform from 0.6 times to just that
    full = min(n_mesh // ratio, 128 if kind != "step" else 256)
    n_cdm = max(8, int(round(full * math.exp(rng.uniform(math.log(0.6), 0.0)))))
    if kind in ("float_step", "trajectory"):
        n_nu = rng.choice([0, 0, n_cdm + 1])
    else:
        n_nu = 2 * n_cdm - rng.choice([0, 1])
    pos, vel = rng.choice([(1, 2), (1, 2), (1, 2), (2, 2), (1, 1)])
    if kind in ("float_step", "trajectory", "vjp"):
        pos, vel = 1, 2
    return _case(kind, n_mesh, ratio, n_cdm, n_nu, pos, vel, rng.choice([-1.0, -1.5, -2.0]),
                 rng.choice([0.005, 0.01]), rng.randint(2, 10) if kind == "trajectory" else 1)


# ------------------------------------------------------------------------- inputs --
def _lattice(n_p, n_mesh, slope, gen):
    """A lattice displaced along the gradient of a Gaussian random field of power n^slope,
    0.3 mesh cells RMS; the velocity equals the displacement (growing mode)."""
    white = torch.randn((n_p, n_p, n_p), generator=gen, device=DEV)
    k = torch.fft.fftfreq(n_p, d=1.0 / n_p, device=DEV)
    kx = torch.fft.rfftfreq(n_p, d=1.0 / n_p, device=DEV)
    n2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + kx[None, None, :] ** 2
    keep = (n2 > 0) & (n2 < (n_p / 2.0) ** 2)
    n2 = torch.where(keep, n2, torch.ones_like(n2))
    dk = torch.fft.rfftn(white) * torch.where(keep, n2 ** (slope / 4.0 - 1.0), 0.0)
    psi = torch.stack([torch.fft.irfftn(1j * kk * dk, s=(n_p, n_p, n_p)).reshape(-1)
                       for kk in (kx[None, None, :], k[None, :, None], k[:, None, None])], 1)
    psi *= (0.3 / n_mesh) / torch.sqrt((psi.double() ** 2).sum(1).mean()).float()
    i = torch.arange(n_p, device=DEV, dtype=torch.float32) / n_p
    z, y, x = torch.meshgrid(i, i, i, indexing="ij")
    q = torch.stack([x.reshape(-1), y.reshape(-1), z.reshape(-1)], 1)
    x = q + psi
    x -= torch.floor(x)
    return torch.where(x >= 1.0, 0.0, x).contiguous(), psi.contiguous()


def _neutrinos(n_p, mean_speed, gen):
    """Uniform positions, isotropic directions, Fermi-Dirac speeds p^2 / (e^p + 1)."""
    n = n_p ** 3
    p = np.linspace(0.0, 40.0, 1 << 15)
    cdf = np.cumsum(p * p / (np.exp(p) + 1.0))
    table = torch.from_numpy(np.interp(np.linspace(0.0, 1.0, 1 << 15), cdf / cdf[-1], p))
    table = table.to(device=DEV, dtype=torch.float32) * (mean_speed / 3.15137)
    x = torch.rand((n, 3), generator=gen, device=DEV)
    v = torch.randn((n, 3), generator=gen, device=DEV)
    v /= torch.linalg.vector_norm(v, dim=1, keepdim=True).clamp_min(1e-20)
    t = torch.rand(n, generator=gen, device=DEV) * ((1 << 15) - 1)
    i = t.long().clamp_max((1 << 15) - 2)
    v *= (table[i] + (table[i + 1] - table[i]) * (t - i))[:, None]
    return torch.where(x >= 1.0, 0.0, x), v


def _loads(case, seed):
    """(x, v, mass) of each species: total cold mass 1, the neutrinos' 1% of it."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    x, v = _lattice(case["n_cdm"], case["n_mesh"], case["slope"], gen)
    loads = [(x, v, 1.0 / case["n_cdm"] ** 3)]
    if case["n_nu"]:
        xn, vn = _neutrinos(case["n_nu"], 50.0 * 0.3 / case["n_mesh"], gen)
        loads.append((xn, vn, 0.01 / case["n_nu"] ** 3))
    return loads


def _cotangents(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed + 1)
    sizes = [case["n_cdm"] ** 3] + ([case["n_nu"] ** 3] if case["n_nu"] else [])
    return [[torch.randn((n, 3), generator=gen, device=DEV) for n in sizes] for _ in "xv"]


def _target(case, seed):
    """A density mesh to be matched: that of another realisation of the recipe."""
    n = case["n_mesh"]
    x, _, m = _loads(dict(case, n_nu=0), seed + 1)[0]
    return _deposit64([(x.double(), m)], n).float()


# --------------------------------------------------------------------- the passes --
def prepare(case, seed):
    kind, n, nc = case["kind"], case["n_mesh"], case["n_mesh"] // case["ratio"]
    s = {"case": case, "kind": kind, "dt": case["dt"], "loads": _loads(case, seed)}
    if kind == "p3m":
        s["ctx"], s["coarse"] = PMContext.two_level(n, nc)
        s["r_soft"] = 1.0 / (40 * nc)
    else:
        s["ctx"] = PMContext(n, nc)
    ctx, w = s["ctx"], widths_word(case["pos"], case["vel"])
    s["float"] = [ctx.float_species(*load) for load in s.pop("loads")]
    if kind == "vjp":
        s["lam"] = _cotangents(case, seed)
    if kind == "trajectory":
        s["x"] = [f.x.requires_grad_() for f in s["float"]]
        s["v"] = [f.v.requires_grad_() for f in s["float"]]
        s["target"] = _target(case, seed)
    if kind == "encode":
        s["widths"] = w
    if kind in ("step", "p3m", "vjp", "force", "save", "restart"):
        s["state"] = [ctx.encode(f, widths=w) for f in s.pop("float")]
    if kind == "restart":
        s["files"] = [(ctx.pack(c, i), c.n) for i, c in enumerate(s.pop("state"))]
    ctx.sync()
    return s


def _codes(state):
    return [{"count": c.count, "pos": c.pos, "vel": c.vel, "esc": c.esc, "hdr": c.hdr}
            for c in state]


def run(s):
    ctx, kind = s["ctx"], s["kind"]
    if kind == "step":
        return _codes(ctx.step(s["state"], s["dt"]))
    if kind == "p3m":
        return _codes(ctx.step_p3m(s["coarse"], s["state"], s["dt"], s["r_soft"]))
    if kind == "float_step":
        return [[f.x, f.v] for f in ctx.step(s["float"], s["dt"])]
    if kind == "trajectory":
        masses = [f.mass for f in s["float"]]
        x, v = trajectory(ctx, s["x"], s["v"], masses, s["dt"], s["case"]["steps"])
        loss = density_loss(ctx, list(zip(x, masses)), s["target"])
        grads = torch.autograd.grad(loss, s["x"] + s["v"])
        return {"loss": loss, "x": x, "v": v, "grads": list(grads)}
    if kind == "vjp":
        return ctx.step_vjp(s["state"], s["dt"], *s["lam"])
    if kind == "force":
        rho = ctx.deposit(s["state"])
        acc, a_max = ctx.force(rho)
        return {"rho": rho, "acc": acc, "a_max": a_max}
    if kind == "encode":
        return _codes([ctx.encode(f, widths=s["widths"]) for f in s["float"]])
    if kind == "save":
        return [np.frombuffer(ctx.pack(c, i), dtype=np.uint8) for i, c in enumerate(s["state"])]
    if kind == "restart":
        back = [ctx.decode(ctx.unpack(data, n)[0]) for data, n in s["files"]]
        return [[f.x, f.v] for f in back]
    raise ValueError(kind)


def work(case):
    """Bytes of the inputs and outputs, once each, and the operations of the transforms
    (2.5 M log2 M for each real transform of M points) and of the particles."""
    kind, m = case["kind"], case["n_mesh"] ** 3
    n = case["n_cdm"] ** 3 + case["n_nu"] ** 3
    n_sp = 2 if case["n_nu"] else 1
    codes = n * 3 * (case["pos"] + case["vel"]) + n_sp * (case["n_mesh"] // case["ratio"]) ** 3
    fft = 2.5 * m * math.log2(m)
    step = 2 * fft + 16 * m + 150 * n
    adjoint = 6 * fft + 40 * m + 400 * n
    got = {
        "step": (2 * codes, step),
        "float_step": (48 * n, step),
        "p3m": (2 * codes, step * (1 + 1 / 64) + 150 * n),
        "trajectory": (72 * n + 4 * m, case["steps"] * (step + adjoint) + 100 * n),
        "vjp": (codes + 48 * n, adjoint),
        "force": (codes + 16 * m, 2 * fft + 16 * m + 40 * n),
        "encode": (24 * n + codes, 20 * n),
        "save": (2 * codes, 0),
        "restart": (codes + 24 * n, 12 * n),
    }[kind]
    return {"bytes": got[0], "flops": got[1]}


# ------------------------------------------------- the same in 64 bits, plain torch --
def _cic(x, n):
    u = x * n
    i = torch.floor(u.detach())
    f = u - i
    i = i.long() % n
    for dz in (0, 1):
        for dy in (0, 1):
            for dx in (0, 1):
                w = (f[:, 0] if dx else 1 - f[:, 0]) * (f[:, 1] if dy else 1 - f[:, 1]) * \
                    (f[:, 2] if dz else 1 - f[:, 2])
                yield ((i[:, 2] + dz) % n * n + (i[:, 1] + dy) % n) * n + (i[:, 0] + dx) % n, w


def _deposit64(species, n):
    rho = torch.zeros(n ** 3, dtype=torch.float64, device=DEV)
    for x, m in species:
        for idx, w in _cic(x, n):
            rho = rho.index_add(0, idx, w * (m * float(n) ** 3))
    return rho.view(n, n, n)


def _force64(rho):
    """a = IDFT(-i D(k) G(k) DFT(rho)): the softened kernel -eps K1(k eps) / k with eps one
    mesh cell and 4 pi G = 1, D the symbol of the fourth-order central difference."""
    n = rho.shape[0]
    k = torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64, device=DEV)
    kx = k[: n // 2 + 1].abs()
    n2 = (k[:, None, None] ** 2 + k[None, :, None] ** 2 + kx[None, None, :] ** 2)
    table = torch.arange(3 * (n // 2) ** 2 + 1, dtype=torch.float64, device=DEV)
    kk = 2 * math.pi * torch.sqrt(table.clamp_min(1.0))
    green = -torch.special.modified_bessel_k1(kk / n) / (n * kk)
    green[0] = 0.0
    pk = torch.fft.rfftn(rho) * green[n2.long()]

    def symbol(j):
        t = 2 * math.pi * j / n
        d = (8 * torch.sin(t) - torch.sin(2 * t)) * (n / 6.0)
        return torch.where(2 * j.abs() == n, 0.0, d)

    return [torch.fft.irfftn(-1j * symbol(d) * pk, s=(n, n, n))
            for d in (kx[None, None, :], k[None, :, None], k[:, None, None])]


def _keys(u, shift, n_cell, brick):
    c = u >> shift
    b, nb = c // brick, n_cell // brick
    loc = c - b * brick
    return (((b[:, 2] * nb + b[:, 1]) * nb + b[:, 0]) * brick ** 3 +
            (loc[:, 2] * brick + loc[:, 1]) * brick + loc[:, 0])


class _Format:
    def __init__(self, case):
        self.n_cell = case["n_mesh"] // case["ratio"]
        self.brick = PMContext.default_brick(case["n_mesh"], self.n_cell)
        self.shift, self.half = 8 * case["pos"], float(2 ** (8 * case["vel"] - 1))
        self.S = self.n_cell << self.shift

    def velocity(self, v, v_max):
        j = torch.floor(v * (self.half / v_max) + self.half).clamp(0, 2 * self.half - 1)
        return ((j - self.half + 0.5) * (v_max / self.half)).float().double()

    def position(self, u):
        return (u.double() + 0.5) / self.S

    def order(self, u):
        return torch.sort(_keys(u, self.shift, self.n_cell, self.brick), stable=True).indices

    def encode(self, x, v):
        """Position codes and decoded velocities in stream order, and that order."""
        u = torch.floor(x.double() * self.S).long() % self.S
        p = self.order(u)
        return u[p], self.velocity(v.double(), float(v.abs().max()))[p], p


def _accel64(xs, masses, n):
    acc = _force64(_deposit64(list(zip(xs, masses)), n))
    a_max = max(float(a.detach().abs().max()) for a in acc)
    out = []
    for x in xs:
        a = [0.0, 0.0, 0.0]
        for idx, w in _cic(x, n):
            for d in range(3):
                a[d] = a[d] + w * acc[d].reshape(-1)[idx]
        out.append(torch.stack(a, 1))
    return out, a_max


def _step64(fmt, us, xs, vs, masses, n, dt):
    """A compressed step on codes us; xs and vs carry the derivative (straight through)."""
    acc, a_max = _accel64(xs, masses, n)
    out = []
    for u, x, v, a in zip(us, xs, vs, acc):
        v1 = v + dt * a
        bound = float(v.detach().abs().max()) + abs(dt) * a_max
        v_max = 2.0 ** math.ceil(math.log2(bound))
        u1 = (u + torch.floor(v1.detach() * dt * fmt.S + 0.5).long()) % fmt.S
        p = fmt.order(u1)
        x1 = x + dt * v1
        x1 = x1 + (fmt.position(u1) - x1).detach()
        v1 = v1 + (fmt.velocity(v1.detach(), v_max) - v1).detach()
        out.append((u1[p], x1[p], v1[p]))
    return [list(t) for t in zip(*out)]


def exact(case, seed):
    kind, n, dt = case["kind"], case["n_mesh"], case["dt"]
    if kind not in ("float_step", "force", "restart", "vjp", "trajectory"):
        return None  # codes and bytes only
    loads = _loads(case, seed)
    masses = [m for _, _, m in loads]
    if kind == "float_step":
        xs = [x.double() for x, _, _ in loads]
        acc, _ = _accel64(xs, masses, n)
        out = []
        for x, a, (_, v, _) in zip(xs, acc, loads):
            v1 = v.double() + dt * a
            x1 = x + dt * v1
            out.append([x1 - torch.floor(x1), v1])
        return out
    fmt = _Format(case)
    enc = [fmt.encode(x, v) for x, v, _ in loads]
    us, vs = [u for u, _, _ in enc], [v for _, v, _ in enc]
    xs = [fmt.position(u) for u in us]
    if kind == "restart":
        return [[x, v] for x, v in zip(xs, vs)]
    if kind == "force":
        rho = _deposit64(list(zip(xs, masses)), n)
        acc = torch.stack(_force64(rho))
        return {"rho": rho, "acc": acc, "a_max": acc.abs().max().reshape(1)}
    for t in xs + vs:
        t.requires_grad_()
    x, v = xs, vs
    for _ in range(case["steps"]):
        us, x, v = _step64(fmt, us, x, v, masses, n, dt)
    if kind == "vjp":
        lx, lv = _cotangents(case, seed)
        g = torch.autograd.grad(x + v, xs + vs, [t.double() for t in lx + lv])
        return [list(g[: len(xs)]), list(g[len(xs):])]
    rho = _deposit64(list(zip(x, masses)), n)
    loss = ((rho - _target(case, seed).double()) ** 2).sum()
    grads = torch.autograd.grad(loss, xs + vs)
    back = []
    for g, p in zip(grads, [p for _, _, p in enc] * 2):
        back.append(torch.empty_like(g))
        back[-1][p] = g
    return {"loss": loss.detach(), "x": [t.detach() for t in x], "v": [t.detach() for t in v],
            "grads": back}
