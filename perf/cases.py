"""Performance cases of the solver: the calls a simulation program makes,
through the public entry points (Plan, Batch, evolve), over the sizes the
repository's own runs, tests and benchmark use.

A case is a dict of plain values:
  op       collision | step | transport | vjp | evolve | batch
  N, Nx    velocity grid side and number of cells (batch: texts "32,64" with
           one entry per problem)
  J, M     angles and radii of the collision quadrature
  f64      float64 (complex128) or float32 (complex64) plan
  walls    periodic | dirichlet | maxwell | mixed (Dirichlet left, Maxwell right)
  field    a magnetic field B(x)
  moments  per-step float64 moments
  steps    time steps of one call
  tune     the program runs the plan's tuner once before it starts
"""
import math

import numpy as np
import torch

import paper_1408_1782_amd as qb

L, R = 12.0, 7.5


def _case(name, op, N, Nx, J=32, M=None, f64=True, walls="periodic", field=False, moments=False, steps=1,
          tune=False):
    c = {"op": op, "N": N, "Nx": Nx, "J": J, "M": (N if M is None else M), "f64": f64, "walls": walls,
         "field": field, "moments": moments, "steps": steps, "tune": tune}
    return dict({"name": name}, **c) if name else c


def listed():
    return [
        # homogeneous relaxation: one cell, a step at a time (launches and latency)
        _case("homogeneous step N32 f64", "step", 32, 1),
        # quadrature study: one cell, more angles and an odd number of radii
        _case("validation N64 J40 f64", "collision", 64, 1, J=40, M=71),
        # small periodic run with a magnetic field, moments at every step
        _case("periodic field N32 f64", "step", 32, 10, field=True, moments=True),
        # coarse grid, the smallest supported transforms
        _case("coarse N16 f64", "step", 16, 16, moments=True, steps=2),
        # slab between two Maxwell walls, as many cells as the physics runs use
        _case("walls N32 f32", "step", 32, 40, f64=False, walls="maxwell", moments=True),
        # the operator alone over a periodic domain
        _case("periodic collision N32 f64", "collision", 32, 128, tune=True),
        # the operator alone on the fine grid in float64
        _case("fine collision N64 f64", "collision", 64, 37),
        # the benchmark's slab: fine grid, float32 bulk, both wall kinds, field, moments
        _case("slab N64 f32", "step", 64, 256, f64=False, walls="mixed", field=True, moments=True, tune=True),
        # transport alone over the same slab (bandwidth)
        _case("slab transport N64 f32", "transport", 64, 256, f64=False, walls="mixed"),
        # transpose of the operator's linearization, by itself
        _case("collision vjp N32 f64", "vjp", 32, 48, tune=True),
        # gradient of a short trajectory in the initial state and the field
        _case("trajectory gradient N32 f64", "evolve", 32, 12, field=True, steps=2),
        # independent uneven problems replayed as one graph
        _case("uneven batch f32", "batch", "32,64,32,16", "32,16,77,5", M=0, f64=False, moments=True),
    ]


def _grids(c):
    """[(N, Nx, M)] of a case's problems."""
    if c["op"] == "batch":
        return [(int(n), int(x), int(n)) for n, x in zip(str(c["N"]).split(","), str(c["Nx"]).split(","))]
    return [(c["N"], c["Nx"], c["M"])]


def _transforms(N, J, M, reverse):
    """P x P complex transforms of one cell's collision (or of its transpose):
    nodes of the radial quadrature in symmetric pairs, two real fields or
    two directions to a transform."""
    pairs, odd = M // 2, M % 2
    if reverse:
        return J * (38 * pairs + 36 * odd) + 22 * J + 14 + 24
    return J * (20 * pairs + 18 * odd) + 11 * J + 7 + 10


def work(c):
    s = 16 if c["f64"] else 8
    flops = bytes_ = 0.0
    for N, Nx, M in _grids(c):
        P = 2 * N
        fft = 5.0 * P * P * math.log2(P * P)
        fwd, rev = (_transforms(N, c["J"], M, r) * fft * Nx for r in (False, True))
        state = 4.0 * N * N * Nx * s
        flops += {"collision": fwd, "step": 2 * fwd * c["steps"], "batch": 2 * fwd * c["steps"], "vjp": rev,
                  "evolve": 2 * (fwd + rev) * c["steps"], "transport": 100.0 * N * N * Nx}[c["op"]]
        bytes_ += state * (3 if c["op"] == "vjp" else 4 if c["op"] == "evolve" else 2)
        bytes_ += 24.0 * Nx * c["field"] + 56.0 * Nx * (c["steps"] + 1) * c["moments"]
    return {"bytes": bytes_, "flops": flops}


def _cost(c):
    """Rough time of a case, in float32 flops."""
    w = work(c)
    return w["flops"] * (2.2 if c["f64"] else 1.0) + 5.0 * w["bytes"]


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        op = rng.choice(["collision", "collision", "step", "step", "step", "transport", "vjp", "evolve", "batch"])
        N = rng.choice([16, 32, 32, 64])
        Nx = int(round(math.exp(rng.uniform(0.0, math.log(512.0)))))
        J = 2 * rng.randint(4, 20)
        M = rng.choice([N, N, rng.randint(max(7, N // 2), 72)])
        f64 = rng.random() < 0.6
        walls = rng.choice(["periodic", "periodic", "dirichlet", "maxwell", "mixed"])
        if op == "batch":
            n = rng.randint(2, 5)
            Ns = [rng.choice([16, 32, 64]) for _ in range(n)]
            xs = [int(round(math.exp(rng.uniform(0.7, math.log(128.0))))) for _ in range(n)]
            c = _case(None, op, ",".join(map(str, Ns)), ",".join(map(str, xs)), J=J, M=0, f64=f64, walls=walls,
                      moments=True)
        else:
            c = _case(None, op, N, Nx, J=J, M=M, f64=f64, walls=walls, field=op in ("step", "evolve")
                      and rng.random() < 0.5, moments=op == "step" and rng.random() < 0.5,
                      steps=rng.randint(1, 3) if op in ("step", "evolve") else 1, tune=op != "transport" and rng.random() < 0.25)
        if _cost(c) <= most:
            return c


# ------------------------------------------------------------------ inputs
def _dt(Nx):
    return min(1e-3, 1.5 / (L * Nx))


def _walls(c):
    left = dict(kind="dirichlet", inv_kT=0.8, mu_up=1.5, mu_down=-1.5)
    right = dict(kind="maxwell", inv_kT=1.1, mu_up=1.3, mu_down=-0.9, alpha=0.4)
    return {"periodic": (dict(kind="periodic"),) * 2, "dirichlet": (left, dict(left, inv_kT=1.2)),
            "maxwell": (dict(right, inv_kT=0.6), right), "mixed": (left, right)}[c["walls"]]


def _dtype(c):
    return torch.complex128 if c["f64"] else torch.complex64


def _state(gen, N, Nx):
    """Fermi-Dirac state with a smooth chemical potential, plus a Hermitian
    perturbation that keeps the eigenvalues in [0, 1]; complex128."""
    kw = dict(dtype=torch.float64, device="cuda")
    v = (2.0 * L / N) * (torch.arange(N, **kw) - N // 2)
    e = 0.5 * (v[:, None] ** 2 + v[None, :] ** 2)
    x = (torch.arange(Nx, **kw) + 0.5) / Nx
    a = torch.rand(3, generator=gen, **kw)
    mu = (a[0] - 0.5) + 0.5 * torch.sin(2 * math.pi * (x + a[1]))
    f = 1.0 / (torch.exp((0.8 + 0.4 * a[2]) * (e[None] - mu[:, None, None])) + 1.0)
    h = 0.2 * f * (1 - f) * (0.5 * torch.rand((4, Nx, N, N), generator=gen, **kw) - 0.25)
    return _matrix(torch.stack([f + h[0], h[1], h[2], h[3]]))


def _matrix(w):
    """[4, Nx, N, N] Pauli components -> [Nx, N, N, 2, 2] complex."""
    rows = [torch.complex(w[0] + w[3], torch.zeros_like(w[0])), torch.complex(w[1], -w[2]),
            torch.complex(w[1], w[2]), torch.complex(w[0] - w[3], torch.zeros_like(w[0]))]
    return torch.stack(rows, dim=-1).reshape(*w.shape[1:], 2, 2)


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    Ws, Bs = [], []
    for N, Nx, _ in _grids(c):
        Ws.append(_state(gen, N, Nx).to(_dtype(c)).contiguous())
        x = (torch.arange(Nx, dtype=torch.float64, device="cuda") + 0.5) / Nx
        p = torch.rand(2, generator=gen, dtype=torch.float64, device="cuda")
        B = torch.stack([0.3 * torch.cos(2 * math.pi * (x + p[0])), 0.5 + 0.0 * x,
                         0.5 * torch.sin(2 * math.pi * (x + p[1]))], dim=1)
        Bs.append(B.contiguous() if c["field"] else None)
    lam = None
    if c["op"] in ("vjp", "evolve"):
        N, Nx, _ = _grids(c)[0]
        f = Ws[0][..., 0, 0].real.double()
        g = (f + 0.05) * (2 * torch.rand((4, Nx, N, N), generator=gen, dtype=torch.float64, device="cuda") - 1)
        lam = _matrix(g).to(_dtype(c)).contiguous()
    return Ws, Bs, lam


def prepare(c, seed):
    Ws, Bs, lam = _inputs(c, seed)
    lw, rw = _walls(c)
    probs = [qb.Problem(Nx, N, c["J"], M, L, R, "f64" if c["f64"] else "f32", qb.BC(**lw), qb.BC(**rw))
             for N, Nx, M in _grids(c)]
    st = {"case": c, "W": Ws[0], "B": Bs[0], "lam": lam, "dt": min(_dt(p.Nx) for p in probs)}
    if c["op"] == "batch":
        st["plan"], st["W"] = qb.Batch(probs), Ws
        st["mom"] = [torch.empty((c["steps"] + 1, p.Nx, 7), dtype=torch.float64, device="cuda") for p in probs]
        return st
    st["plan"] = qb.Plan(probs[0], adjoint=c["op"] in ("vjp", "evolve"))
    if c["moments"]:
        st["mom"] = torch.empty((c["steps"] + 1, probs[0].Nx, 7), dtype=torch.float64, device="cuda")
    if c["tune"]:
        st["plan"].tune()
    if c["op"] == "evolve":
        st["W"].requires_grad_(True)
        if st["B"] is not None:
            st["B"].requires_grad_(True)
    return st


def run(st):
    c, plan, W, B = st["case"], st["plan"], st["W"], st["B"]
    if c["op"] == "collision":
        return plan.collision(W)
    if c["op"] == "step":
        plan.step(W, B, st["dt"], c["steps"], st.get("mom"))
        return (W, st["mom"]) if c["moments"] else W
    if c["op"] == "transport":
        return plan.transport_step(W, 0.5 * st["dt"])
    if c["op"] == "vjp":
        return plan.collision_vjp(W, st["lam"])
    if c["op"] == "batch":
        plan.step(W, None, st["dt"], c["steps"], st["mom"], graph=True)
        return W, st["mom"]
    WT = qb.evolve(plan, W, B, st["dt"], c["steps"], checkpoint_every=1)
    wrt = [W] if B is None else [W, B]
    return (WT.detach(),) + torch.autograd.grad(WT, wrt, st["lam"])


# ------------------------------------------------------------------ the same in plain torch, 64 bits
def _phi(x):
    s = torch.where(x == 0, torch.ones_like(x), x)
    return torch.where(x == 0, torch.zeros_like(x), 2 * L / (math.pi * s) * torch.sin(math.pi * R * s / (2 * L)) ** 2)


def _psi(x):
    s = torch.where(x == 0, torch.ones_like(x), x)
    return torch.where(x == 0, torch.full_like(x, 2 * R), 2 * L / (math.pi * s) * torch.sin(math.pi * R * s / L))


class _SumOver(torch.autograd.Function):
    """sum_c fn(x, c), one term's graph in memory at a time."""

    @staticmethod
    def forward(ctx, x, fn, terms):
        ctx.save_for_backward(x)
        ctx.fn, ctx.terms = fn, terms
        with torch.no_grad():
            out = fn(x, terms[0])
            for t in terms[1:]:
                out = out + fn(x, t)
        return out

    @staticmethod
    def backward(ctx, g):
        x, = ctx.saved_tensors
        gx = torch.zeros_like(x)
        for t in ctx.terms:
            with torch.enable_grad():
                y = x.detach().requires_grad_(True)
                gx += torch.autograd.grad(ctx.fn(y, t), y, g)[0]
        return gx, None, None


class _Exact:
    """The collision of w[4, cells, N, N] by real FFTs on the padded grid."""

    def __init__(self, N, J, M):
        self.N, self.P, self.J, self.M = N, 2 * N, J, M
        kw = dict(dtype=torch.float64, device="cuda")
        b = torch.fft.fftfreq(self.P, 1.0 / self.P, **kw)
        self.bx, self.by = b[:, None], torch.arange(N + 1, **kw)[None, :]  # half spectrum in the second axis
        a = torch.arange(J, **kw) * math.pi / J
        self.th, self.thp = ((torch.cos(t), torch.sin(t)) for t in (a, a + 0.5 * math.pi / J))
        x, w = np.polynomial.legendre.leggauss(M)
        self.rho, self.wgl = R * x, R * w
        k = torch.fft.fftfreq(N, 1.0 / N, **kw).abs() < N / 2 - 0.5
        self.keep = (k[:, None] & k[None, :]).to(torch.float64)
        dots = self.th[0][:, None] * self.thp[0] + self.th[1][:, None] * self.thp[1]
        self.wG = -((2 * math.pi / J) ** 2) / dots

    def dot(self, t, j):
        return self.bx * t[0][j] + self.by * t[1][j]

    def inv(self, f):
        return torch.fft.irfft2(f, s=(self.P, self.P), norm="forward")

    def fwd(self, f):
        return torch.fft.rfft2(f, norm="forward")

    def half(self, w):
        """Coefficients on the padded half spectrum, unpaired frequency dropped."""
        N, P = self.N, self.P
        f = torch.fft.fft2(torch.fft.ifftshift(w, dim=(-2, -1)), norm="forward") * self.keep
        f = f[..., : N // 2 + 1]
        z = f.new_zeros(f.shape[:-2] + (P - N, f.shape[-1]))
        f = torch.cat([f[..., : N // 2, :], z, f[..., N // 2:, :]], dim=-2)
        return torch.cat([f, f.new_zeros(f.shape[:-1] + (N + 1 - f.shape[-1],))], dim=-1)

    def short(self, r):
        """Padded-grid field -> velocity grid, coefficients on Xi only."""
        N = self.N
        f = torch.fft.fft2(r, norm="forward")
        f = torch.cat([f[..., : N // 2, :], f[..., -(N // 2):, :]], dim=-2)
        f = torch.cat([f[..., : N // 2], f[..., -(N // 2):]], dim=-1) * self.keep
        return torch.fft.fftshift(torch.fft.ifft2(f, norm="forward").real, dim=(-2, -1))

    def i3_term(self, wh, jm):
        """Weighted sum over one direction's nodes m0..m1 of s_a Psi(w_a s_nu), with its signs in a."""
        j, m0, m1 = jm
        kw = dict(dtype=torch.float64, device="cuda")
        al = torch.as_tensor(self.rho[m0:m1], **kw)[:, None, None] * (math.pi / L) * self.dot(self.th, j)
        wt = torch.as_tensor(self.wgl[m0:m1] * math.pi / self.J, **kw)[:, None, None, None, None, None]
        s = self.inv(wh * torch.polar(torch.ones_like(al), al)[:, None, None])  # [m, 4, cells, P, P]
        w = self.inv(wh)
        eta = wh.real.new_tensor([1.0, -1.0, -1.0, -1.0])[:, None, None, None, None]
        psi = _psi(self.bx * -self.th[1][j] + self.by * self.th[0][j])
        x = self.inv(self.fwd(w[:, None] * s[:, None]) * psi)                   # [m, a, nu, cells, P, P]
        return (wt * eta * s[:, :, None] * x).sum(dim=(0, 1))

    def pair_term(self, wh, j):
        """One direction of the I_1 (3), I_4 (4) and I_2 (1) fields, stacked."""
        w = self.inv(wh)
        f0 = 2 * w[0] - 1
        phip, out = _phi(self.dot(self.thp, j)), 0.0
        for i in range(self.J):
            out = out + self.wG[i, j] * _phi(self.dot(self.th, i))
        g = self.inv(-1j * out * self.fwd(f0 * self.inv(1j * phip * wh[1:])))
        ps, pp = _psi(self.dot(self.th, j)), _psi(self.bx * -self.th[1][j] + self.by * self.th[0][j])
        y = self.inv(ps * self.fwd(f0 * self.inv(pp * wh))) * (math.pi / self.J)
        eta = wh.real.new_tensor([1.0, -1.0, -1.0, -1.0])[:, None, None, None]
        S = (eta * self.inv(ps * wh) * self.inv(pp * wh)).sum(dim=0, keepdim=True) * (math.pi / self.J)
        return torch.cat([g, y, S])

    def collision(self, w):
        """c[4, cells, N, N]."""
        cells = max(1, int(4e8 / (4 * 16 * 8 * self.P ** 2 * 4)))
        return torch.cat([self.part(x) for x in w.split(cells, dim=1)], dim=1)

    def part(self, w):
        wh = self.half(w)
        wp = self.inv(wh)
        n = max(1, int(4e8 / (16 * 8 * self.P ** 2 * w.shape[1] * 4)))
        b = _SumOver.apply(wh, self.i3_term, [(j, m, min(m + n, self.M)) for j in range(self.J)
                                              for m in range(0, self.M, n)])
        g1, g2, g3, y0, y1, y2, y3, S = _SumOver.apply(wh, self.pair_term, list(range(self.J)))
        w0, w1, w2, w3 = wp
        pi2 = 2 * math.pi
        r = [pi2 * (S * (1 - w0) - b[0] + y0 * w0 - y1 * w1 - y2 * w2 - y3 * w3),
             -2 * (g2 * w3 - g3 * w2) + pi2 * (-S * w1 + b[1] + y0 * w1 - y1 * w0),
             -2 * (g3 * w1 - g1 * w3) + pi2 * (-S * w2 + b[2] + y0 * w2 - y2 * w0),
             -2 * (g1 * w2 - g2 * w1) + pi2 * (-S * w3 + b[3] + y0 * w3 - y3 * w0)]
        return self.short(torch.stack(r))


def _pauli(W):
    return 0.5 * torch.stack([(W[..., 0, 0] + W[..., 1, 1]).real, (W[..., 0, 1] + W[..., 1, 0]).real,
                              (W[..., 1, 0] - W[..., 0, 1]).imag, (W[..., 0, 0] - W[..., 1, 1]).real])


def _minmod(a, b):
    return torch.where(a * b > 0, torch.where(a.abs() <= b.abs(), a, b), torch.zeros_like(a))


def _transport(w, dt, walls):
    """One limited transport step of w[4, Nx, N, N]."""
    Nx, N = w.shape[1], w.shape[2]
    h = 2.0 * L / N
    v1 = h * (torch.arange(N, dtype=torch.float64, device=w.device) - N // 2)
    vx = v1[:, None].expand(N, N)
    ends = []
    for left, bc in ((True, walls[0]), (False, walls[1])):
        if bc["kind"] == "periodic":
            idx = torch.arange(-2, 0) if left else torch.arange(0, 2)
            ends.append(w[:, (idx % Nx).to(w.device)])
            continue
        adj = w[:, 0] if left else w[:, -1]
        f = [1.0 / (torch.exp((0.5 * (vx ** 2 + vx.T ** 2) - bc[m]) * bc["inv_kT"]) + 1.0) for m in ("mu_up", "mu_down")]
        wall = torch.stack([0.5 * (f[0] + f[1]), 0 * f[0], 0 * f[0], 0.5 * (f[0] - f[1])])
        inflow = vx > 0 if left else vx < 0
        if bc["kind"] == "maxwell":
            if not left:
                inflow = inflow & (torch.arange(N, device=w.device) > 0)[:, None]
            outflow = vx < 0 if left else vx > 0
            F = h * h * (2 * adj[0] * vx.abs() * outflow).sum()
            Z = h * h * (2 * wall[0] * vx.abs() * inflow).sum()
            mirror = adj[:, (N - torch.arange(N, device=w.device)) % N]
            wall = (1 - bc["alpha"]) * mirror + bc["alpha"] * wall * (F / Z)
        ends.append(torch.where(inflow, wall, adj)[:, None].expand(-1, 2, -1, -1))
    we = torch.cat([ends[0], w, ends[1]], dim=1)
    d = we[:, 1:] - we[:, :-1]
    S = _minmod(d[:, 1:], d[:, :-1])
    Sm, S0, Sp = S[:, :-2], S[:, 1:-1], S[:, 2:]
    Wm, W0, Wp = we[:, 1:-3], we[:, 2:-2], we[:, 3:-1]
    av, lim = vx.abs(), 0.5 * (torch.sign(vx) - dt * vx * Nx)
    upd = -vx * (Wp - Wm) + av * (Wp - 2 * W0 + Wm) + lim * (-vx * (Sp - Sm) + av * (Sp - 2 * S0 + Sm))
    return W0 + 0.5 * dt * Nx * upd


def _moments(w):
    N = w.shape[2]
    h = 2.0 * L / N
    v = h * (torch.arange(N, dtype=torch.float64, device=w.device) - N // 2)
    vx, vy, tr = v[:, None], v[None, :], 2 * w[0]
    m = [x.sum(dim=(1, 2)) for x in (*w, vx * tr, vy * tr, 0.5 * (vx ** 2 + vy ** 2) * tr)]
    return h * h * torch.stack(m, dim=1)


def _steps(ex, w, B, dt, n, walls):
    """w after n steps, and the moments before the first and after each."""
    def rhs(w):
        f = ex.collision(w)
        if B is None:
            return f
        b = B.T[:, :, None, None]
        return f + 2 * torch.stack([0 * w[0], b[1] * w[3] - b[2] * w[2], b[2] * w[1] - b[0] * w[3],
                                    b[0] * w[2] - b[1] * w[1]])
    mom = [_moments(w)]
    for _ in range(n):
        w = _transport(w, 0.5 * dt, walls)
        w1 = w + dt * rhs(w)
        w = _transport(0.5 * (w + w1 + dt * rhs(w1)), 0.5 * dt, walls)
        mom.append(_moments(w))
    return w, torch.stack(mom)


def exact(c, seed):
    # passes over the padded products; about 4 TB/s of them fit the time there is
    products = sum((4 if c["op"] in ("vjp", "evolve") else 1) * c["J"] * M * Nx * 16 * 4 * N * N * 8 * 12
                   for N, Nx, M in _grids(c)) * (2 * c["steps"] if c["op"] in ("step", "batch", "evolve") else 1)
    if c["op"] != "transport" and products > 40e12:
        return None
    Ws, Bs, lam = _inputs(c, seed)
    walls = _walls(c)
    dt = min(_dt(Nx) for _, Nx, _ in _grids(c))
    exs = {N: _Exact(N, c["J"], M) for N, _, M in _grids(c)}
    N = _grids(c)[0][0]
    W = Ws[0].to(torch.complex128)
    if c["op"] == "collision":
        return _matrix(exs[N].collision(_pauli(W)))
    if c["op"] == "transport":
        return _matrix(_transport(_pauli(W), 0.5 * dt, walls))
    if c["op"] == "vjp":
        W.requires_grad_(True)
        return torch.autograd.grad(_matrix(exs[N].collision(_pauli(W))), W, lam.to(torch.complex128))[0]
    if c["op"] == "evolve":
        B = Bs[0]
        wrt = [x.requires_grad_(True) for x in ([W] if B is None else [W, B])]
        WT = _matrix(_steps(exs[N], _pauli(W), B, dt, c["steps"], walls)[0])
        return (WT.detach(),) + torch.autograd.grad(WT, wrt, lam.to(torch.complex128))
    out = [_steps(exs[x.shape[1]], _pauli(x.to(torch.complex128)), B, dt, c["steps"], walls) for x, B in zip(Ws, Bs)]
    out = [(_matrix(w), m) for w, m in out]
    if c["op"] == "batch":
        return [w for w, _ in out], [m for _, m in out]
    return out[0] if c["moments"] else out[0][0]
