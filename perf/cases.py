"""Performance cases of the t2s2 library, through its public entry points.

Five kinds of work a program of this framework does on the GPU:

  step       time steps of a flow (Context.step), then its fields: the
             Taylor-Green vortex (periodic), the lid-driven cavity (walls,
             stretched mesh) and the force-driven channel (one walled axis),
             in the schemes and storage forms of the library;
  monitor    what a run reads between its steps: the residual against the
             previous output, the global diagnostics, the velocity field and
             the distributions;
  gradient   forward and backward of the differentiable rollout (T2S2Rollout):
             the gradient of a probe loss with respect to the initial
             velocity and the viscosity, on the cavity;
  adjoint    one reverse step on a large periodic grid;
  stability  a von Neumann stability map.

`exact` restates each of them in plain FP64 torch, from the paper's stages.
"""
import math

import numpy as np
import torch

import paper_1911_12913_amd as t2s2
import workloads as W
from paper_1911_12913_amd.rollout import RolloutSpec, T2S2Rollout

DEVICE = "cuda"
STORED = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16,
          "bf16sr": torch.bfloat16, "f16": torch.float16, "f16sr": torch.float16}
F16_SCALE = 16384.0  # the FP16 forms hold 2^14 times the deviation
BTILDE = (0.25, 0.5, 0.25)  # the member of the eq 2.13 family that is run
LARGEST = 4096 * 4096 * 20  # node-steps of the largest listed case
SPEED, LID = 0.05, 0.1  # velocity of the initial vortices, of the lid


def listed():
    step = dict(kind="step", scheme="fdlbm1", storage="f64")
    return [
        # The paper's Poiseuille validation (Tables 5-8): the smallest mesh, a
        # body force, one walled axis; thousands of steps to a steady state.
        dict(step, name="channel10x21_f64", flow="channel", nx=10, ny=21, steps=100),
        # The 32^2 Taylor-Green run checked against the closed form.
        dict(step, name="tgv32_f64", flow="tgv", nx=32, ny=32, steps=100),
        # The Re 1000 cavity of the paper at 257^2, advanced between outputs.
        dict(step, name="cavity257_f64", flow="cavity", nx=257, ny=257, steps=100),
        # The Re 5000 cavity at 2049^2, in FP64 and in the 16-bit form meant
        # for long runs.
        dict(step, name="cavity2049_f64", flow="cavity", nx=2049, ny=2049, steps=20),
        dict(step, name="cavity2049_bf16sr", flow="cavity", nx=2049, ny=2049, steps=20,
             storage="bf16sr"),
        # The throughput workload: Taylor-Green at 4096^2, FP64 and FP32.
        dict(step, name="tgv4096_f64", flow="tgv", nx=4096, ny=4096, steps=20),
        dict(step, name="tgv4096_f32", flow="tgv", nx=4096, ny=4096, steps=20, storage="f32"),
        # A member of the eq 2.13 family on a ragged grid (three gradients).
        dict(step, name="family1500x1100_f64", flow="tgv", nx=1500, ny=1100, steps=10,
             scheme="family"),
        # Output of a long run: residual, diagnostics, velocity, distributions.
        dict(name="monitor1025_f64", kind="monitor", flow="cavity", storage="f64", nx=1025,
             ny=1025),
        # The differentiation workload (513^2 cavity, FP32 storage, sqrt(N)
        # checkpoints), a training step over 100 time steps.
        dict(name="gradient513_f32", kind="gradient", storage="f32", n=513, steps=100),
        # One reverse step where nothing fits in the caches.
        dict(name="adjoint2048_f64", kind="adjoint", storage="f64", nx=2048, ny=2048),
        # A stability map of the implemented step (Sec. 2C).
        dict(name="stability16x16", kind="stability", model="fdlbm1", points=256, nk=17,
             eta=0.1),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 7 + ["monitor", "gradient", "adjoint", "stability"])
    if kind == "step":
        flow = rng.choice(["tgv", "tgv", "cavity", "cavity", "channel"])
        scheme = rng.choice(["fdlbm1"] * 5 + ["t1s2", "fdlbm2", "family"])
        forms = ["f64", "f64", "f64", "f32", "f32", "bf16", "f16"]
        if scheme in ("fdlbm1", "t1s2"):
            forms += ["bf16sr", "f16sr"]
        storage = rng.choice(forms)
        nx, ny = _size(rng, 10, 4096), _size(rng, 10, 4096)
        if rng.random() < 0.5 or flow == "cavity":
            ny = min(4096, max(10, nx + rng.randint(-9, 9)))
        # Three gradients per step cost up to twice one; short runs cost
        # launches, not nodes.
        cap = LARGEST // (4 if scheme in ("fdlbm2", "family") else 2)
        steps = min(_size(rng, 1, 120), max(1, cap // (nx * ny)))
        return dict(kind="step", flow=flow, scheme=scheme, storage=storage, nx=nx, ny=ny,
                    steps=steps)
    if kind == "monitor":
        return dict(kind="monitor", flow=rng.choice(["tgv", "cavity"]),
                    storage=rng.choice(["f64", "f64", "f32", "bf16sr"]),
                    nx=_size(rng, 60, 2500), ny=_size(rng, 60, 2500))
    if kind == "gradient":
        n = _size(rng, 33, 640)
        return dict(kind="gradient", storage=rng.choice(["f32", "f64"]), n=n,
                    steps=min(_size(rng, 8, 100), max(8, 100 * 513 * 513 // (n * n))))
    if kind == "adjoint":
        return dict(kind="adjoint", storage=rng.choice(["f64", "f64", "f32"]),
                    nx=_size(rng, 200, 2300), ny=_size(rng, 200, 2300))
    return dict(kind="stability", model=rng.choice(["paper", "fdlbm1", "fdlbm2", "family"]),
                points=_size(rng, 16, 300), nk=rng.choice([9, 13, 17]),
                eta=rng.choice([0.01, 0.1]))


# ------------------------------------------------------------------ problems

def _problem(c):
    """Mesh, parameters and scheme of a case, as Context takes them."""
    scheme = c.get("scheme", "fdlbm1")
    kw = dict(eta=0.01, A=0.5, scheme=1, btilde=(0.0, 1.0, 0.0))
    cfl = 0.9
    if scheme == "t1s2":
        kw["A"], cfl = 0.0, 0.25
    elif scheme == "fdlbm2":
        kw["scheme"], cfl = 2, 0.6
    elif scheme == "family":
        kw["scheme"], kw["btilde"], cfl = 3, BTILDE, 0.6
    if c["flow"] == "tgv":
        x, px = W.uniform_periodic(c["nx"], 0.0, 2 * math.pi)
        y, py = W.uniform_periodic(c["ny"], 0.0, 2 * math.pi)
        # dt / tau = 4.6, where the schemes are stable at these steps.
        dt = cfl * min(px / c["nx"], py / c["ny"])
        kw.update(periodic_x=True, periodic_y=True, period_x=px, period_y=py, nu=dt / 4.6 / 3)
    elif c["flow"] == "cavity":
        x, y = W.tanh_walled(c["nx"] - 1, 1.5), W.tanh_walled(c["ny"] - 1, 1.5)
        re = 1000.0 if c["nx"] < 1000 else 5000.0
        uw = np.zeros((4, 2))
        uw[3, 0] = LID
        kw.update(periodic_x=False, periodic_y=False, nu=LID / re, u_wall=uw,
                  eta=0.1 if re < 2000 else 0.05)
    else:
        x = np.arange(c["nx"]) / c["nx"]
        y = W.tanh_walled(c["ny"] - 1, 1.5)
        kw.update(periodic_x=True, periodic_y=False, period_x=1.0,
                  nu=math.sqrt(0.01 / 80.0), force=(0.01, 0.0), eta=0.1)
    return x, y, dict(kw, cfl=cfl)


def _fields(c, x, y, seed):
    """A vortex array with seeded phases and amplitudes plus small noise; at
    rest on walls."""
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    r = torch.rand(6, generator=g, device=DEVICE, dtype=torch.float64)
    X = torch.as_tensor(x, device=DEVICE)[None, :]
    Y = torch.as_tensor(y, device=DEVICE)[:, None]
    amp = SPEED * (0.6 + 0.4 * r[0])
    if c["flow"] == "tgv":
        a, b = 2 * math.pi * r[1], 2 * math.pi * r[2]
        u, v = -amp * torch.cos(X + a) * torch.sin(Y + b), amp * torch.sin(X + a) * torch.cos(Y + b)
        rho = 1.001 - 0.75 * amp * amp * (torch.cos(2 * X + 2 * a) + torch.cos(2 * Y + 2 * b))
        u, v = u + 0.01 + 0.01 * r[3], v - 0.01 - 0.01 * r[4]  # carried by a mean flow
    else:
        walls = c["flow"] == "cavity"
        sx = torch.sin(math.pi * X) if walls else torch.ones_like(X)
        cx = torch.cos(math.pi * X) if walls else torch.zeros_like(X)
        sy, cy = torch.sin(math.pi * Y), torch.cos(math.pi * Y)
        u = 2 * amp * sx * sx * sy * cy * (1 - (0.3 + 0.3 * r[3]) * Y)
        v = -2 * amp * sx * cx * sy * sy * (1 - (0.3 + 0.3 * r[4]) * X)
        rho = 1.0 + 0.2 * amp * amp * (1 + sx * sy)
    noise = 1e-6 * (2 * torch.rand(2, *u.shape, generator=g, device=DEVICE, dtype=torch.float64) - 1)
    u, v = u + noise[0], v + noise[1]
    if c["flow"] != "tgv":
        u[0], u[-1], v[0], v[-1] = 0, 0, 0, 0
    if c["flow"] == "cavity":
        u[:, 0], u[:, -1], v[:, 0], v[:, -1] = 0, 0, 0, 0
        u[-1, 1:-1] = LID
    return rho.expand_as(u).contiguous(), u.contiguous(), v.contiguous()


def _previous(u, v):
    """The velocity of an earlier output, which the residual compares with."""
    return 0.97 * u + 0.01 * v, 0.98 * v


def _planes(raw, dtype, c):
    """The nodes of a raw [9][ny][pitch] buffer."""
    return raw.view(dtype).view(9, c["ny"], -1)[:, :, : c["nx"]]


def _context(c, seed):
    x, y, kw = _problem(c)
    ctx = t2s2.Context(t2s2.make_config(storage=c["storage"], **kw), x, y)
    rho, u, v = _fields(c, x, y, seed)
    ctx.init_macro(rho, u, v)
    return ctx, u, v


def _random(shape, seed, scale):
    g = torch.Generator(device=DEVICE).manual_seed(seed + 1)
    return scale * torch.randn(shape, generator=g, device=DEVICE, dtype=torch.float64)


def _off_equilibrium(c, seed):
    """A state inside a run is off equilibrium by a little."""
    return _random((9, c["ny"], c["nx"]), seed + 1, 1e-4)


def _misfit(c, seed):
    """d loss / d state: the misfit of the distributions to noisy targets."""
    return _off_equilibrium(c, seed) + _random((9, c["ny"], c["nx"]), seed + 2, 3e-5)


def _gradient_inputs(c, seed):
    cc = dict(flow="cavity", nx=c["n"], ny=c["n"])
    x, y, kw = _problem(cc)
    rho, u, v = _fields(cc, x, y, seed)
    probes = torch.as_tensor(W.probe_nodes(c["n"], c["n"], 64, seed=2), device=DEVICE)
    dtype = STORED[c["storage"]]
    targets = _random((2, 64), seed, 0.02)
    return x, y, kw, rho.to(dtype), u.to(dtype), v.to(dtype), probes, targets


def _stability_inputs(c, seed):
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    r = torch.rand(2, c["points"], generator=g, device=DEVICE, dtype=torch.float64)
    kw = dict(eta=c["eta"], u=(0.05, 0.02), nk=c["nk"])
    if c["model"] == "paper":
        kw.update(b2bar=0.5, b2tilde=0.25)
    if c["model"] == "family":
        kw.update(btilde=BTILDE)
    return 0.05 + 4.0 * r[0], 0.05 + 1.5 * r[1], kw


# ----------------------------------------------------------- what is timed

def prepare(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "step":
        ctx, _, _ = _context(c, seed)
        return dict(c=c, ctx=ctx)
    if kind == "monitor":
        ctx, u, v = _context(c, seed)
        u, v = _previous(u, v)
        return dict(c=c, ctx=ctx, u=u, v=v)
    if kind == "adjoint":
        ctx, _, _ = _context(dict(c, flow="tgv"), seed)
        ctx.init_distributions(ctx.read_distributions() + _off_equilibrium(c, seed))
        ctx.enable_adjoint()
        state = ctx.save_state()
        lam = ctx.adjoint_load(_misfit(c, seed))
        return dict(c=c, ctx=ctx, state=state, lam=lam, out=ctx.adjoint_buffer())
    if kind == "gradient":
        x, y, kw, rho, u, v, probes, targets = _gradient_inputs(c, seed)
        spec = RolloutSpec(x=x, y=y, periodic_x=False, periodic_y=False, cfl=kw["cfl"],
                           eta=kw["eta"], u_wall=kw["u_wall"], storage=c["storage"],
                           nsteps=c["steps"], device=DEVICE)
        nu = torch.tensor(kw["nu"], dtype=u.dtype, device=DEVICE)
        return dict(c=c, spec=spec, rho=rho, u=u, v=v, nu=nu, probes=probes, targets=targets)
    omega, r, kw = _stability_inputs(c, seed)
    return dict(c=c, omega=omega, r=r, kw=kw)


def run(s):
    c = s["c"]
    kind = c["kind"]
    if kind == "step":
        s["ctx"].step(c["steps"])
        if c["storage"] == "f64":
            return s["ctx"].moments()
        return _planes(s["ctx"].state_tensor(), STORED[c["storage"]], c)
    if kind == "monitor":
        ctx = s["ctx"]
        gre = ctx.velocity_error(s["u"], s["v"])
        diag = ctx.diagnostics()
        return gre, diag, ctx.moments(), ctx.read_distributions()
    if kind == "adjoint":
        dnu = torch.zeros(1, dtype=torch.float64, device=DEVICE)
        s["ctx"].adjoint_step(s["state"], s["lam"], s["out"], dnu)
        dtype = torch.float64 if c["storage"] == "f64" else torch.float32
        return _planes(s["out"], dtype, c), dnu.to(dtype)
    if kind == "gradient":
        u, v, nu = (t.detach().requires_grad_() for t in (s["u"], s["v"], s["nu"]))
        U, V = T2S2Rollout.apply(s["rho"], u, v, nu, s["spec"])
        i, j = s["probes"][:, 0], s["probes"][:, 1]
        loss = ((U[j, i] - s["targets"][0]) ** 2 + (V[j, i] - s["targets"][1]) ** 2).sum()
        loss.backward()
        return u.grad, v.grad, nu.grad
    return t2s2.stability_map(c["model"], s["omega"], s["r"], **s["kw"])


def work(case):
    c = dict(case)
    if c["kind"] == "stability":
        modes = (2 * c["nk"] - 1) * c["nk"] * c["points"]
        # 30 squarings of a complex 9 x 9 matrix per mode.
        return {"bytes": 24.0 * c["points"], "flops": modes * 30 * 8.0 * 729}
    nx, ny = (c["n"], c["n"]) if c["kind"] == "gradient" else (c["nx"], c["ny"])
    nodes, size = float(nx * ny), STORED[c["storage"]].itemsize
    if c["kind"] == "step":
        out = 24 if c["storage"] == "f64" else 0
        # The state in and out; about 330 operations per node and step.
        return {"bytes": nodes * (18 * size + out), "flops": nodes * c["steps"] * 330.0}
    if c["kind"] == "monitor":
        return {"bytes": nodes * (9 * size + 16 + 24 + 72), "flops": nodes * 60.0}
    if c["kind"] == "adjoint":
        real = 8 if c["storage"] == "f64" else 4
        return {"bytes": nodes * (9 * size + 18 * real), "flops": nodes * 700.0}
    # Fields in, gradients out; forward, recompute and reverse per step.
    return {"bytes": nodes * 5 * size, "flops": nodes * c["steps"] * 1300.0}


# ----------------------------------------------- the same in plain FP64 torch

_EX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
_EY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
_WQ = (4 / 9,) + (1 / 9,) * 4 + (1 / 36,) * 4


class _Exact:
    """One time step of the paper's Sec. 2D, stage by stage, on g = f~ - w."""

    def __init__(self, x, y, *, cfl, nu, eta, A, scheme, btilde, periodic_x, periodic_y,
                 period_x=0.0, period_y=0.0, u_wall=None, force=(0.0, 0.0)):
        self.per = {2: periodic_x, 1: periodic_y}
        dmin = min(np.diff(x).min(), np.diff(y).min())
        if periodic_x:
            dmin = min(dmin, x[0] + period_x - x[-1])
        if periodic_y:
            dmin = min(dmin, y[0] + period_y - y[-1])
        self.dt, self.eta, self.A, self.scheme, self.b = cfl * dmin, eta, A, scheme, btilde
        self.F, self.inv_tau = force, 1.0 / (3.0 * nu)
        self.m = {2: self._metric(x, periodic_x, period_x)[None, :],
                  1: self._metric(y, periodic_y, period_y)[:, None]}
        self.uw = np.zeros((4, 2)) if u_wall is None else np.asarray(u_wall)

    @staticmethod
    def _metric(c, per, period):
        lo = np.concatenate([[c[-1] - period if per else c[0]], c[:-1]])
        hi = np.concatenate([c[1:], [c[0] + period if per else c[-1]]])
        return torch.as_tensor(2.0 / (hi - lo), device=DEVICE)

    def moments(self, a, h):
        s = sum(a[q] for q in range(9))
        ux = (a[1] + a[5] + a[8] - a[3] - a[6] - a[7]) / (1 + s) + h / 2 * self.F[0]
        uy = (a[2] + a[5] + a[6] - a[4] - a[7] - a[8]) / (1 + s) + h / 2 * self.F[1]
        return s, ux, uy

    @staticmethod
    def feq(q, s, ux, uy):
        e = _EX[q] * ux + _EY[q] * uy
        return _WQ[q] * (s + (1 + s) * (3 * e + 4.5 * e * e - 1.5 * (ux * ux + uy * uy)))

    def collide(self, a, h, c_a, c_e, c_f):
        """[c_a a + c_e feq(a) + c_f F(a)], the moments shifted by h/2 F."""
        s, ux, uy = self.moments(a, h)
        out = []
        for q in range(9):
            eq = self.feq(q, s, ux, uy)
            r = c_a * a[q] + c_e * eq
            if self.F != (0.0, 0.0):
                r = r + c_f * 3 * (self.F[0] * (_EX[q] - ux) + self.F[1] * (_EY[q] - uy)) * (_WQ[q] + eq)
            out.append(r)
        return out

    def _diff(self, f, axis, sign):
        """Mixed difference along an axis; at walls the ghost is quadratic."""
        d = axis - 1
        n = f.shape[d]
        if self.per[axis]:
            p = torch.cat([f.narrow(d, n - 2, 2), f, f.narrow(d, 0, 2)], d)
        else:
            at = lambda i: f.narrow(d, i % n, 1)  # noqa: E731
            lo, hi = 3 * at(0) - 3 * at(1) + at(2), 3 * at(-1) - 3 * at(-2) + at(-3)
            p = torch.cat([lo, lo, f, hi, hi], d)
        m2, m1, c, p1, p2 = (p.narrow(d, k, n) for k in range(5))
        up = (3 * c - 4 * m1 + m2) / 2 if sign > 0 else -(3 * c - 4 * p1 + p2) / 2
        return ((1 - self.eta) * (p1 - m1) / 2 + self.eta * up) * self.m[axis]

    def L(self, f, q):
        r = 0.0
        if _EX[q]:
            r = r - _EX[q] * self._diff(f, 2, _EX[q])
        if _EY[q]:
            r = r - _EY[q] * self._diff(f, 1, _EY[q])
        return r

    def walls(self, a, h):
        """Non-equilibrium extrapolation (eq 3.10) onto the wall nodes."""
        if self.per[1] and self.per[2]:
            return a
        ny, nx = a[0].shape
        jj, ii = torch.arange(ny, device=DEVICE), torch.arange(nx, device=DEVICE)
        fj = jj if self.per[1] else jj.clamp(1, ny - 2)
        fi = ii if self.per[2] else ii.clamp(1, nx - 2)
        ub, vb = (torch.zeros(ny, nx, device=DEVICE, dtype=torch.float64) for _ in range(2))
        wall = torch.zeros(ny, nx, device=DEVICE, dtype=torch.bool)
        for k, t in enumerate((ub, vb)):
            if not self.per[1]:
                t[0], t[-1] = float(self.uw[2, k]), float(self.uw[3, k])
            if not self.per[2]:
                t[:, 0], t[:, -1] = float(self.uw[0, k]), float(self.uw[1, k])
        if not self.per[1]:
            wall[0] = wall[-1] = True
        if not self.per[2]:
            wall[:, 0] = wall[:, -1] = True
        near = [f[fj][:, fi] for f in a]
        s, ux, uy = self.moments(near, h)
        return [torch.where(wall, near[q] + self.feq(q, s, ub, vb) - self.feq(q, s, ux, uy), a[q])
                for q in range(9)]

    def inside(self, new, old):
        """new at interior nodes, old on walls."""
        if self.per[1] and self.per[2]:
            return new
        sj = slice(None) if self.per[1] else slice(1, -1)
        si = slice(None) if self.per[2] else slice(1, -1)
        keep = torch.zeros_like(old, dtype=torch.bool)
        keep[sj, si] = True
        return torch.where(keep, new, old)

    def predict(self, start, h, w_h):
        """f at t + h from its transformed start (eqs 2.32-2.35, 3.10)."""
        S = [self.inside(start[q] + h * self.L(start[q], q), start[q]) for q in range(9)]
        R = self.collide(S, h, 2 / (2 + w_h), w_h / (2 + w_h), h / (2 + w_h))
        return self.walls(R, 0.0)

    def step(self, g, inv_tau=None):
        dt, A = self.dt, self.A
        w = dt * (self.inv_tau if inv_tau is None else inv_tau)
        Q = self.collide(g, dt, (2 - w) / (2 + w), 2 * w / (2 + w), 2 * dt / (2 + w))
        T = [0.0] * 9
        b = {1: (0.0, 1.0, 0.0), 2: (0.5, 0.0, 0.5), 3: self.b}[self.scheme]
        if b[0]:
            f = self.collide(g, dt, 2 / (2 + w), w / (2 + w), dt / (2 + w))
            T = [T[q] + b[0] * f[q] for q in range(9)]
        if b[1]:
            P = self.collide(g, dt, (2 - A * w) / (2 + w), (1 + A) * w / (2 + w),
                             (1 + A) * dt / (2 + w))
            f = self.predict(P, A * dt, A * w)
            T = [T[q] + b[1] * f[q] for q in range(9)]
        if b[2]:
            f = self.predict(Q, dt, w)
            T = [T[q] + b[2] * f[q] for q in range(9)]
        return self.walls([self.inside(Q[q] + dt * self.L(T[q], q), Q[q]) for q in range(9)], dt)

    def start(self, rho, u, v):
        return [self.feq(q, rho - 1, u, v) for q in range(9)]


def _exact_step(c, seed):
    x, y, kw = _problem(c)
    e = _Exact(x, y, **kw)
    g = e.start(*_fields(c, x, y, seed))
    for _ in range(c["steps"]):
        g = e.step(g)
    if c["storage"] == "f64":
        return e.moments(g, e.dt)
    return torch.stack(g) * (F16_SCALE if c["storage"].startswith("f16") else 1.0)


def _stored(g, c):
    """The state as its storage form holds it (rounded to nearest)."""
    k = F16_SCALE if c["storage"].startswith("f16") else 1.0
    return (g * k).to(STORED[c["storage"]]).double() / k


def _exact_monitor(c, seed):
    x, y, kw = _problem(c)
    e = _Exact(x, y, **kw)
    rho, u0, v0 = _fields(c, x, y, seed)
    g = _stored(torch.stack(e.start(rho, u0, v0)), c)
    u0, v0 = _previous(u0, v0)
    s, u, v = e.moments(g, e.dt)
    d2, r2, u2 = ((u - u0) ** 2 + (v - v0) ** 2).sum(), (u0**2 + v0**2).sum(), (u**2 + v**2).sum()
    gre = dict(sum_diff2=d2, sum_ref2=r2, sum_u2=u2, gre=(d2 / r2).sqrt(), residual=(d2 / u2).sqrt())
    J = []
    for z, axis in ((y, "y"), (x, "x")):
        per, period = kw["periodic_" + axis], kw.get("period_" + axis, 0)
        lo = np.concatenate([[z[-1] - period if per else z[0]], z[:-1]])
        hi = np.concatenate([z[1:], [z[0] + period if per else z[-1]]])
        J.append(torch.as_tensor((hi - lo) / 2, device=DEVICE))
    J = J[0][:, None] * J[1][None, :]
    diag = dict(mass_excess=(J * s).sum(), kinetic_energy=(J * (1 + s) * (u * u + v * v) / 2).sum(),
                max_speed=(u * u + v * v).max().sqrt(), nonfinite=0.0,
                momentum_x=(J * (1 + s) * u).sum(), momentum_y=(J * (1 + s) * v).sum())
    floats = lambda d: {k: float(t) for k, t in d.items()}  # noqa: E731
    return floats(gre), floats(diag), (s, u, v), g


def _exact_adjoint(c, seed):
    cc = dict(c, flow="tgv")
    x, y, kw = _problem(cc)
    e = _Exact(x, y, **kw)
    # The state in hand is near the equilibrium, rounded to the storage.
    start = torch.stack(e.start(*_fields(cc, x, y, seed)))
    g = _stored(start + _off_equilibrium(c, seed), c)
    lam = list(_misfit(c, seed).unbind(0))
    nu = torch.tensor(kw["nu"], dtype=torch.float64, device=DEVICE, requires_grad=True)
    leaves = [t.requires_grad_() for t in g.unbind(0)]
    out = e.step(leaves, 1.0 / (3.0 * nu))
    got = torch.autograd.grad(out, leaves + [nu], lam)
    return torch.stack(got[:9]), got[9].reshape(1)


def _exact_gradient(c, seed):
    from torch.utils.checkpoint import checkpoint

    x, y, kw, rho, u, v, probes, targets = _gradient_inputs(c, seed)
    e = _Exact(x, y, **kw)
    u, v = u.double().requires_grad_(), v.double().requires_grad_()
    nu = torch.tensor(kw["nu"], dtype=u.dtype, device=DEVICE)
    nu = nu.to(STORED[c["storage"]]).double().requires_grad_()
    g = torch.stack(e.start(rho.double(), u, v))
    one = lambda t, n: torch.stack(e.step(list(t.unbind(0)), 1.0 / (3.0 * n)))  # noqa: E731
    for _ in range(c["steps"]):
        g = checkpoint(one, g, nu, use_reentrant=False)
    _, U, V = e.moments(g, e.dt)
    i, j = probes[:, 0], probes[:, 1]
    loss = ((U[j, i] - targets[0]) ** 2 + (V[j, i] - targets[1]) ** 2).sum()
    return torch.autograd.grad(loss, (u, v, nu))


def _exact_stability(c, seed):
    omega, r, kw = _stability_inputs(c, seed)
    nk, (ux, uy), eta, A = kw["nk"], kw["u"], kw["eta"], 0.5
    dev = dict(device=DEVICE, dtype=torch.float64)
    ex, ey, wq = (torch.tensor(t, **dev) for t in (_EX, _EY, _WQ))
    eu, uu = ex * ux + ey * uy, ux * ux + uy * uy
    G = ((wq * (1 - 4.5 * eu * eu + 1.5 * uu))[:, None]
         + (wq * (3 * ex + 9 * eu * ex - 3 * ux))[:, None] * ex
         + (wq * (3 * ey + 9 * eu * ey - 3 * uy))[:, None] * ey).to(torch.complex128)
    eye = torch.eye(9, device=DEVICE, dtype=torch.complex128)
    tx = torch.linspace(-math.pi, math.pi, 2 * nk - 1, **dev).repeat_interleave(nk)
    ty = torch.linspace(0, math.pi, nk, **dev).repeat(2 * nk - 1)
    S = torch.zeros(tx.numel(), 9, device=DEVICE, dtype=torch.complex128)
    for th in (tx[:, None] * ex, ty[:, None] * ey):
        S += 1j * (1 - eta) * torch.sin(th) + eta / 2 * (3 - 4 * torch.exp(-1j * th) + torch.exp(-2j * th))
    out = []
    for w, rr in zip(omega.tolist(), r.tolist()):
        rS = torch.diag_embed(rr * S)
        J = lambda a, e: a * eye + e * G  # noqa: E731
        JP = J((2 - A * w) / (2 + w), (1 + A) * w / (2 + w))
        JQ, Jf = J((2 - w) / (2 + w), 2 * w / (2 + w)), J(2 / (2 + w), w / (2 + w))
        JR = J(2 / (2 + A * w), A * w / (2 + A * w))
        if c["model"] == "paper":
            bb, bt = kw["b2bar"], kw["b2tilde"]
            lhs = (1 + w * bb) * eye + w * (0.5 - 2 * bb) * G + rS @ (bt * eye + (0.5 - bt) * G)
            rhs = (1 - w * (1 - bb)) * eye + w * (1.5 - 2 * bb) * G - rS @ ((1 - bt) * eye - (0.5 - bt) * G)
            M = torch.linalg.solve(lhs, rhs)
        elif c["model"] == "fdlbm1":
            M = JQ - rS @ JR @ (eye - A * rS) @ JP
        elif c["model"] == "fdlbm2":
            M = JQ - 0.5 * rS @ (Jf + Jf @ (eye - rS) @ JQ)
        else:
            b = kw["btilde"]
            M = JQ - rS @ (b[0] * Jf + b[1] * JR @ (eye - A * rS) @ JP + b[2] * Jf @ (eye - rS) @ JQ)
        ell = torch.zeros(M.shape[0], **dev)
        for k in range(31):
            n = M.abs().amax((1, 2))
            M, ell = M / n[:, None, None], ell + torch.log(n) / 2.0**k
            if k < 30:
                M = (M[:, :, :, None] * M[:, None, :, :]).sum(2)
        out.append(torch.exp(ell).max())
    return torch.stack(out)


def exact(case, seed):
    c = dict(case)
    return {"step": _exact_step, "monitor": _exact_monitor, "adjoint": _exact_adjoint,
            "gradient": _exact_gradient, "stability": _exact_stability}[c["kind"]](c, seed)
