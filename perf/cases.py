"""The work that a user of this package has it do, as timed cases.

Seven kinds, each through the package's public entry points:

  solve   one implicit pressure solve from a zero guess (Solver.solve), FP64 or mixed precision
  next    the pressure part of a time step: new coefficients, then a solve from the previous pressure
          (Solver.update_coefficients, Solver.solve)
  update  new coefficients, then the residual that the previous pressure leaves under them
          (Solver.update_coefficients, Solver.residual)
  hydro   the steps either side of a solve (Solver.eos_ideal, advect, pressure_rhs, pressure_update)
  step    one whole two-stage time step of the Gresho vortex (stepper.SemiImplicitStepper.step)
  net     the learned estimate of a solution (Net.forward)
  train   one training step of that network on the A-norm error (Solver.train_step_anorm)

Arrays are (nz, ny, nx), momenta (3, nz, ny, nx). Boxes are periodic in x and y and closed in z, x
also closed where a case says so. Sizes, Mach numbers and fields are those of the package's own
workloads, drawn on the GPU from the case's seed.
"""
import math

import numpy as np
import torch

import paper_1112_3507_amd as hp
from paper_1112_3507_amd.stepper import SemiImplicitStepper

TOL = 1e-10
GAMMA = 5.0 / 3.0
LR = 1e-3
MODES = {"fp64": hp.MODE_FP64_MGPCG, "mixed": hp.MODE_MIXED_IR}
# (input channels, output channels, level) of the network's ten convolutions
CONVS = [(4, 16, 0), (16, 16, 0), (16, 32, 1), (32, 32, 1), (32, 64, 2), (64, 64, 2), (96, 32, 1),
         (32, 32, 1), (48, 16, 0), (16, 16, 0)]


# ---- the cases ---------------------------------------------------------------------------------

def _solve(nx, ny, nz, mach, mode, closed_x=False):
    return {"kind": "solve", "nx": nx, "ny": ny, "nz": nz, "mach": mach, "mode": mode, "closed_x": closed_x}


def _box(kind, nx, ny, nz, **more):
    return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, **more}


def listed():
    return [
        # the smallest solve in use: the 2D validation problem, where launches and latency count
        {"name": "solve 64x1x64", **_solve(64, 1, 64, 0.1, "fp64")},
        # a resolution study's small box
        {"name": "solve 64x64x64", **_solve(64, 64, 64, 0.01, "fp64")},
        # a box whose sizes carry few factors of two: it stops coarsening early
        {"name": "solve 160x96x72", **_solve(160, 96, 72, 0.01, "fp64")},
        # the benchmark's box, in the default precision and in the mixed one
        {"name": "solve 256x256x256", **_solve(256, 256, 256, 0.01, "fp64")},
        {"name": "solve 256x256x256 mixed", **_solve(256, 256, 256, 0.001, "mixed")},
        # a production box in a running simulation: coefficients of the new time, previous pressure
        {"name": "next 512x512x256 mixed", **_box("next", 512, 512, 256, mach=0.001, mode="mixed")},
        # whether a previous pressure still holds after the coefficients moved
        {"name": "update 256x256x256", **_box("update", 256, 256, 256, mach=0.01)},
        # explicit and update steps of the benchmark's box, and of a small two-component one
        {"name": "hydro 256x256x256", **_box("hydro", 256, 256, 256, mach=0.01, two=False)},
        {"name": "hydro 96x80x72 two", **_box("hydro", 96, 80, 72, mach=0.01, two=True)},
        # a whole time step of the Mach ladder's vortex, many small launches
        {"name": "step 256x256", **_box("step", 256, 256, 1, mach=0.1)},
        # the network's estimate on the benchmark's box, and its training at the size it is trained at
        {"name": "net 256x256x256", **_box("net", 256, 256, 256)},
        {"name": "train 128x128x128", **_box("train", 128, 128, 128, mach=0.001)},
    ]


def _size(rng, low, high, odd_part):
    """A size near a log-uniform draw in [low, high]: a power of two times one of `odd_part`."""
    want = math.exp(rng.uniform(math.log(low), math.log(high)))
    every = [a << k for a in odd_part for k in range(12) if low <= (a << k) <= high]
    near = sorted(every, key=lambda n: abs(math.log(n / want)))[:3]
    return rng.choice(near)


# factors that leave the coarsest level small enough for the solver: periodic axes stop at twice
# an odd number, closed ones at an odd one
PERIODIC_PART = (2, 6, 10, 14)
CLOSED_PART = (2, 3, 5, 7, 9, 11)


def _draw_box(rng, low, high, cells):
    while True:
        n = (_size(rng, low, high, PERIODIC_PART), _size(rng, low, high, PERIODIC_PART),
             _size(rng, max(low // 2, 6), high, CLOSED_PART))
        if n[0] * n[1] * n[2] <= cells:
            return n


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "next", "update", "hydro", "step", "net", "train"])
    mach = rng.choice([0.1, 0.01, 0.001])
    mode = rng.choice(["fp64", "mixed"])
    if kind == "solve":
        closed = rng.random() < 0.25
        if rng.random() < 0.3:  # two dimensions, as the validation problems
            nx = _size(rng, 32, 512, CLOSED_PART if closed else PERIODIC_PART)
            return _solve(nx, 1, _size(rng, 32, 512, CLOSED_PART), mach, mode, closed)
        nx, ny, nz = _draw_box(rng, 24, 320, 256 ** 3)
        return _solve(nx, ny, nz, mach, mode, closed)
    if kind == "next":
        nx, ny, nz = _draw_box(rng, 32, 512, 256 ** 3)
        return _box("next", nx, ny, nz, mach=mach, mode=mode)
    if kind == "update":
        nx, ny, nz = _draw_box(rng, 32, 320, 256 ** 3)
        return _box("update", nx, ny, nz, mach=mach)
    if kind == "hydro":
        nx, ny, nz = _draw_box(rng, 24, 320, 256 ** 3)
        return _box("hydro", nx, ny, nz, mach=rng.choice([0.1, 0.01]), two=rng.random() < 0.5)
    if kind == "step":
        n = _size(rng, 32, 320, PERIODIC_PART)
        return _box("step", n, n, 1, mach=rng.choice([0.1, 0.03, 0.01]))
    nets = (4, 12, 20, 28)  # the network takes multiples of four
    if kind == "net":
        return _box("net", *(_size(rng, 32, 256, nets) for _ in range(3)))
    return _box("train", *(_size(rng, 32, 128, (4, 12)) for _ in range(3)), mach=0.001)


# ---- inputs ------------------------------------------------------------------------------------

class Fields:
    """Seeded fields of one box on the GPU."""

    def __init__(self, case, seed):
        self.n = (case["nx"], case["ny"], case["nz"])
        self.shape = self.n[::-1]
        # the flat cases' spacing is that of their x axis (z has one cell)
        self.d = 1.0 / (self.n[2] if self.n[2] > 1 else self.n[0])
        self.h = (self.d,) * 3
        self.bc = (hp.NEUMANN if case.get("closed_x") else hp.PERIODIC, hp.PERIODIC, hp.NEUMANN)
        self.gen = torch.Generator(device="cuda").manual_seed(int(seed))
        self.z = (torch.arange(self.n[2], dtype=torch.float64, device="cuda") + 0.5) * self.d

    def uniform(self, *lead):
        """uniform(-1, 1) per cell"""
        return 2.0 * torch.rand(*lead, *self.shape, dtype=torch.float64, device="cuda", generator=self.gen) - 1.0

    def white(self):
        """N(0, 1) per cell minus the mean"""
        b = torch.randn(self.shape, dtype=torch.float64, device="cuda", generator=self.gen)
        return b.sub_(b.mean())

    def polytrope(self):
        """rho and c2 of the stratified layer, T = 1 + 9 z, with 1% of noise per cell"""
        t = (1.0 + 9.0 * self.z)[:, None, None]
        rho = t ** 1.5 * (1.0 + 0.01 * self.uniform())
        return rho, t * (1.0 + 0.01 * self.uniform())

    def velocity(self, mach):
        """a smooth velocity of size ~mach that vanishes at the closed ends of z"""
        x, y = ((torch.arange(k, dtype=torch.float64, device="cuda") + 0.5) / k for k in self.n[:2])
        u = torch.zeros(3, *self.shape, dtype=torch.float64, device="cuda")
        r = torch.rand(4, 8, dtype=torch.float64, generator=torch.Generator().manual_seed(self.gen.initial_seed()))
        for kx, ky, kz, ph, a0, a1, a2, pv in r.tolist():
            kx, ky, kz = int(7 * kx) - 3, int(7 * ky) - 3, 1 + int(3 * kz)
            flat = torch.cos(2 * math.pi * (kx * x[None, :] + ky * y[:, None] + ph))[None]
            up = math.pi * kz * self.z
            u[0] += mach * (2 * a0 - 1) * flat * torch.cos(up + pv)[:, None, None]
            u[1] += mach * (2 * a1 - 1) * flat * torch.cos(up - pv)[:, None, None]
            u[2] += mach * (2 * a2 - 1) * flat * torch.sin(up)[:, None, None]
        return u


def _solve_inputs(case, seed):
    f = Fields(case, seed)
    rho, c2 = f.polytrope()
    return f, rho, c2, f.white(), f.d / case["mach"]


def _next_inputs(case, seed):
    """Coefficients before and after a step, and the right-hand sides of either time."""
    f, rho, c2, b, dt = _solve_inputs(case, seed)
    rho1, c21 = (torch.roll(a, 1, 2) * (1.0 + 0.001 * f.uniform()) for a in (rho, c2))
    return f, (rho, c2), (rho1, c21), b, b + 0.1 * f.white(), dt


def _hydro_inputs(case, seed):
    f = Fields(case, seed)
    t = (1.0 + 9.0 * f.z)[:, None, None]
    rho = t ** 1.5 * (1.0 + 0.01 * f.uniform())
    u = f.velocity(case["mach"])
    mom = rho * u
    p = t ** 2.5 * (1.0 + 1e-4 * f.uniform())
    e = p / (GAMMA - 1.0) + 0.5 * rho * (u * u).sum(0)
    more = {}
    if case["two"]:
        ones = torch.ones(f.shape, dtype=torch.float64, device="cuda")
        more = {"visc": case["mach"] ** 2 * f.uniform(), "temp_n": t * ones,
                "conc_n": (0.25 + 0.05 * torch.tanh((f.z - 0.5) / 0.02))[:, None, None] * ones,
                "rkc_n": 1e-3 * rho}
    new = p * (1.0 + 1e-5 * f.uniform())  # the pressure a solve would return
    return f, rho, mom, e, new, more, 0.5 * f.d


def _gresho(case, seed):
    """The Gresho vortex with 0.1% of density noise, and the sound-speed step of its Mach number."""
    f = Fields(case, seed)
    n, mach = case["nx"], case["mach"]
    c = (torch.arange(n, dtype=torch.float64, device="cuda") + 0.5) / n - 0.5
    dx, dy = c[None, :].expand(n, n), c[:, None].expand(n, n)
    r = torch.sqrt(dx * dx + dy * dy).clamp_min(1e-300)
    u = torch.where(r <= 0.2, 5.0 * r, torch.where(r <= 0.4, 2.0 - 5.0 * r, torch.zeros_like(r)))
    p0 = 1.0 / (GAMMA * mach * mach)
    p = torch.where(r <= 0.2, p0 + 12.5 * r * r, torch.where(
        r <= 0.4, p0 + 12.5 * r * r + 4.0 * (1.0 - 5.0 * r - math.log(0.2) + torch.log(r)),
        torch.full_like(r, p0 - 2.0 + 4.0 * math.log(2.0))))
    rho = 1.0 + 0.001 * f.uniform()
    mom = torch.stack([-dy / r * u, dx / r * u, torch.zeros_like(u)]).reshape(3, 1, n, n) * rho
    e = p.reshape(1, n, n) / (GAMMA - 1.0) + 0.5 * (mom * mom).sum(0) / rho
    return f, rho, mom, e, 0.5 * f.d / (1.0 + 1.0 / mach)


def _theta(seed):
    """He-uniform parameters as training starts from, with small biases."""
    rng = np.random.default_rng(seed)
    parts = []
    for ci, co, _ in CONVS:
        a = math.sqrt(6.0 / (27 * ci))
        parts += [rng.uniform(-a, a, 27 * ci * co), rng.uniform(-0.01, 0.01, co)]
    a = math.sqrt(6.0 / 16)
    parts += [rng.uniform(-a, a, 16), rng.uniform(-0.01, 0.01, 1)]
    return torch.from_numpy(np.concatenate(parts).astype(np.float32)).cuda()


NET_SCALE = 1e-2


def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        f, rho, c2, b, dt = _solve_inputs(case, seed)
        s = hp.setup(f.n, f.h, f.bc, rho, c2, dt, MODES[case["mode"]])
        return {"kind": kind, "s": s, "b": b, "p": torch.zeros_like(b)}
    if kind in ("next", "update"):
        f, old, new, b, b1, dt = _next_inputs(case, seed)
        s = hp.setup(f.n, f.h, f.bc, *old, dt, MODES[case.get("mode", "fp64")])
        before = torch.zeros_like(b)
        if kind == "next":
            s.solve(b, before, TOL)
        else:
            before = f.velocity(1.0)[2].clone()
        return {"kind": kind, "s": s, "new": new, "dt": dt, "b": b1, "before": before, "p": torch.empty_like(b)}
    if kind == "hydro":
        f, rho, mom, e, new, more, dt = _hydro_inputs(case, seed)
        s = hp.setup(f.n, f.h, f.bc, rho, rho, dt)
        a = lambda *lead: torch.empty(*lead, *f.shape, dtype=torch.float64, device="cuda")  # noqa: E731
        out = {"p": a(), "c2": a(), "rho1": a(), "mom_s": a(3), "e_s": a(), "b": a(), "mom1": a(3), "uf": a(3),
               "e1": a()}
        return {"kind": kind, "s": s, "rho": rho, "mom": mom, "e": e, "new": new, "more": more, "out": out}
    if kind == "step":
        f, rho, mom, e, dt = _gresho(case, seed)
        return {"kind": kind, "st": SemiImplicitStepper(f.n, f.h, f.bc, dt, GAMMA, rho, mom, e, TOL)}
    f, rho, c2, b, dt = _solve_inputs({"mach": 0.001, **case}, seed)
    net = hp.Net(f.n, training=kind == "train")
    net.set_params(_theta(seed))
    if kind == "net":
        net.set_output_scale(NET_SCALE)
        return {"kind": kind, "net": net, "b": b, "rho": rho, "c2": c2, "prev": 1e-2 * f.uniform(),
                "x": torch.empty_like(b)}
    s = hp.setup(f.n, f.h, f.bc, rho, c2, dt)
    x = torch.zeros_like(b)
    s.solve(b, x, TOL)
    net.set_output_scale(float(x.norm() / b.norm()))
    return {"kind": kind, "net": net, "s": s, "b": b, "x": x}


def run(state):
    kind = state["kind"]
    if kind == "solve":
        state["p"].zero_()
        state["s"].solve(state["b"], state["p"], TOL)
        return state["p"]
    if kind == "next":
        state["s"].update_coefficients(*state["new"], state["dt"])
        state["p"].copy_(state["before"])
        state["s"].solve(state["b"], state["p"], TOL)
        return state["p"]
    if kind == "update":
        state["s"].update_coefficients(*state["new"], state["dt"])
        state["s"].residual(state["b"], state["before"], state["p"])
        return state["p"]
    if kind == "hydro":
        s, o = state["s"], state["out"]
        s.eos_ideal(state["rho"], state["mom"], state["e"], GAMMA, o["p"], o["c2"])
        s.advect(state["rho"], state["mom"], state["e"], o["rho1"], o["mom_s"], o["e_s"])
        s.pressure_rhs(state["rho"], o["c2"], o["p"], state["mom"], o["rho1"], o["mom_s"], o["b"], **state["more"])
        s.pressure_update(state["new"], o["rho1"], o["mom_s"], o["e_s"], o["mom1"], o["uf"], o["e1"])
        return o
    if kind == "step":
        st = state["st"]
        st.step()
        return {"rho": st.rho, "mom": st.mom, "e": st.e}
    if kind == "net":
        state["net"].forward(state["b"], state["rho"], state["c2"], state["prev"], state["x"])
        return state["x"]
    loss = state["s"].train_step_anorm(state["net"], state["b"], state["x"], LR)
    return {"loss": loss, "grad": state["net"].get_grad(), "params": state["net"].get_params()}


def work(case):
    """Bytes: each input read and each output written once; operations: of the network's
    convolutions (three products per multiply in training), of one pass over the stencil else."""
    cells = case["nx"] * case["ny"] * case["nz"]
    conv = sum(2 * 27 * ci * co * cells / 8 ** lev for ci, co, lev in CONVS)
    kind = case["kind"]
    arrays = {"solve": 3, "next": 5, "update": 5, "hydro": 5 + 15 + (4 if case.get("two") else 0) + 1, "step": 10,
              "net": 5, "train": 3}[kind]
    flops = {"net": conv, "train": 3 * conv}.get(kind, 40.0 * cells)
    return {"bytes": 8.0 * arrays * cells, "flops": flops}


# ---- 64-bit reference --------------------------------------------------------------------------

class Box:
    """The discrete operator and the explicit formulas of one box in plain torch."""

    def __init__(self, f, dt):
        self.n, self.h, self.bc, self.dt = f.n, f.h, f.bc, dt
        self.axes = [d for d in range(3) if self.n[d] > 1]

    def closed(self, d):
        return self.bc[d] == hp.NEUMANN

    def end(self, a, d, value, last=True):
        """a with its cells at one closed end of axis d set to `value`'s."""
        if not self.closed(d):
            return a
        i = a.shape[2 - d] - 1 if last else 0
        a = a.clone()
        v = value.select(2 - d, i) if torch.is_tensor(value) else value
        a.select(2 - d, i).copy_(v) if torch.is_tensor(v) else a.select(2 - d, i).fill_(v)
        return a

    def up(self, a, d):
        return torch.roll(a, -1, 2 - d)

    def low(self, a, d, own):
        """The low interface of each cell from high-interface values; `own` at a closed low end."""
        return self.end(torch.roll(a, 1, 2 - d), d, own, last=False)

    def weights(self, rho):
        """dt^2 kappa / h^2 on the high interface of every cell, per axis."""
        return {d: self.end(self.dt ** 2 / self.h[d] ** 2 * 2.0 / (rho + self.up(rho, d)), d, 0.0) for d in self.axes}

    def apply(self, m, w, p):
        y = m * p
        for d in self.axes:
            flux = w[d] * (p - self.up(p, d))
            y += flux
            y -= torch.roll(flux, 1, 2 - d)
        return y

    def basis(self, d):
        """Orthonormal eigenvectors (columns) and eigenvalues of the second difference on axis d."""
        k = self.n[d]
        i = torch.arange(k, dtype=torch.float64, device="cuda")
        if k == 1:
            return torch.ones(1, 1, dtype=torch.float64, device="cuda"), torch.zeros_like(i)
        if self.closed(d):
            q = torch.cos(math.pi / k * (i[:, None] + 0.5) * i[None, :])
            lam = 2.0 - 2.0 * torch.cos(math.pi * i / k)
        else:
            f = torch.div(i + 1, 2, rounding_mode="floor")  # 0, 1, 1, 2, 2, ...
            a = 2.0 * math.pi / k * i[:, None] * f[None, :]
            q = torch.where((i[None, :] % 2 == 1), torch.cos(a), torch.sin(a))
            q[:, 0] = 1.0
            lam = 2.0 - 2.0 * torch.cos(2.0 * math.pi * f / k)
        return q / q.norm(dim=0, keepdim=True), lam

    def separable(self, m, rho):
        """Solver of the operator with coefficients averaged over each horizontal plane."""
        nx, ny, nz = self.n
        qx, lx = self.basis(0)
        qy, ly = self.basis(1)
        cx, cy, cz = (self.dt ** 2 / v ** 2 for v in self.h)
        mz, rz = m.mean((1, 2)), rho.mean((1, 2))
        diag = mz[:, None, None] + (cx * lx[None, None, :] + cy * ly[None, :, None]) / rz[:, None, None]
        wz = cz * 2.0 / (rz[1:] + rz[:-1])
        if nz > 1 and not self.closed(2):
            raise ValueError("z is closed in every case")
        diag[:-1] += wz[:, None, None]
        diag[1:] += wz[:, None, None]
        wl = wz.tolist()
        piv = torch.empty_like(diag)
        piv[0] = 1.0 / diag[0]
        for k in range(1, nz):
            piv[k] = 1.0 / (diag[k] - wl[k - 1] ** 2 * piv[k - 1])
        del diag

        def solve(r):
            s = torch.matmul(r.reshape(-1, nx), qx).reshape(nz, ny, nx)
            s = torch.matmul(qy.T.contiguous(), s) if ny > 1 else s
            s[0] *= piv[0]
            for k in range(1, nz):
                s[k].add_(s[k - 1], alpha=wl[k - 1]).mul_(piv[k])
            for k in range(nz - 2, -1, -1):
                s[k].addcmul_(piv[k], s[k + 1], value=wl[k])
            s = torch.matmul(qy, s) if ny > 1 else s
            return torch.matmul(s.reshape(-1, nx), qx.T.contiguous()).reshape(nz, ny, nx)

        return solve

    def solve(self, m, rho, b, x=None):
        """The solution as conjugate gradients with the separable preconditioner reach it, down to
        where the residual no longer falls."""
        w, pre = self.weights(rho), self.separable(m, rho)
        x = torch.zeros_like(b) if x is None else x.clone()
        bn = float(b.norm())
        best, kept = math.inf, x
        for _ in range(3):  # from the true residual each time
            r = b - self.apply(m, w, x)
            rel = float(r.norm()) / bn
            if not rel < 0.5 * best:
                break
            best, kept = rel, x.clone()
            p, rz = None, 1.0
            for _ in range(30):
                z = pre(r)
                new = float((r * z).sum())
                p = z if p is None else z + (new / rz) * p
                rz = new
                q = self.apply(m, w, p)
                alpha = rz / float((p * q).sum())
                x = x + alpha * p
                r = r - alpha * q
                if float(r.norm()) <= 1e-15 * bn:
                    break
        r = b - self.apply(m, w, x)
        return x if float(r.norm()) / bn < best else kept

    # the explicit steps and the updates around a solve

    def face_u(self, mom, rho, d):
        return self.end((mom[d] + self.up(mom[d], d)) / (rho + self.up(rho, d)), d, 0.0)

    def div(self, faces):
        out = 0.0
        for d in self.axes:
            out = out + (faces[d] - self.low(faces[d], d, 0.0)) / self.h[d]
        return out

    def grad(self, p, rho):
        g = [torch.zeros_like(p) for _ in range(3)]
        for d in self.axes:
            face = (self.up(p, d) * rho + p * self.up(rho, d)) / (rho + self.up(rho, d))
            face = self.end(face, d, p)
            g[d] = (face - self.low(face, d, p)) / self.h[d]
        return torch.stack(g)

    def eos(self, rho, mom, e):
        p = (GAMMA - 1.0) * (e - 0.5 * (mom * mom).sum(0) / rho)
        return p, GAMMA * p / rho

    def near(self, q, d, s):
        k = q.shape[2 - d]
        i = torch.arange(k, device=q.device) + s
        return q.index_select(2 - d, i.clamp(0, k - 1) if self.closed(d) else i % k)

    def advect(self, rho, mom, e):
        new = []
        u = {d: self.face_u(mom, rho, d) for d in self.axes}
        for q in (rho, mom[0], mom[1], mom[2], e):
            o = q.clone()
            for d in self.axes:
                qm, qp, qpp = (self.near(q, d, s) for s in (-1, 1, 2))
                a, b, c = q - qm, qp - q, qpp - qp
                left = q + 0.5 * torch.where(a.abs() < b.abs(), a, b)
                right = qp - 0.5 * torch.where(b.abs() < c.abs(), b, c)
                flux = u[d] * torch.where(u[d] >= 0, left, right)
                o -= self.dt * (flux - self.low(flux, d, 0.0)) / self.h[d]
            new.append(o)
        return new[0], torch.stack(new[1:4]), new[4]

    def rhs(self, rho, c2, p, mom, rho1, mom_s, visc=None, temp_n=None, conc_n=None, rkc_n=None):
        m, dt = 1.0 / (rho * c2), self.dt
        b = m * (p - dt * (mom / rho * self.grad(p, rho)).sum(0))
        b = b - dt * self.div({d: self.face_u(mom_s, rho1, d) for d in self.axes})
        if visc is not None:
            b = b - 2.0 * dt / 3.0 * m / rho * visc
        if temp_n is not None:
            flux = {d: self.end(0.5 * (rkc_n + self.up(rkc_n, d)) * (self.up(conc_n, d) - conc_n) / self.h[d], d, 0.0)
                    for d in self.axes}
            b = b - 3.0 * dt / 4.0 * m * temp_n * self.div(flux)
        return b

    def updated(self, p, rho1, mom_s, e_s):
        g = self.grad(p, rho1)
        mom = mom_s - self.dt * g
        uf = torch.zeros_like(mom_s)
        for d in self.axes:
            du = self.dt * (self.up(p, d) - p) / self.h[d] * 2.0 / (self.up(rho1, d) + rho1)
            uf[d] = self.face_u(mom_s, rho1, d) - self.end(du, d, 0.0)
        return mom, uf, e_s - self.dt * (p * self.div(uf) + (mom / rho1 * g).sum(0))

    def stage(self, rho, mom, e):
        p, c2 = self.eos(rho, mom, e)
        rho1, mom_s, e_s = self.advect(rho, mom, e)
        b = self.rhs(rho, c2, p, mom, rho1, mom_s)
        x = self.solve(1.0 / (rho * c2), rho1, b, p)
        mom1, _, e1 = self.updated(x, rho1, mom_s, e_s)
        return rho1, mom1, e1


class Net64:
    """The network in 64 bits: 3x3x3 correlations, periodic in x and y, zero beyond z."""

    def __init__(self, theta):
        self.layers, at = [], 0
        for ci, co, _ in CONVS:
            k = 27 * ci * co
            self.layers.append((theta[at:at + k].view(co, 27, ci), theta[at + k:at + k + co]))
            at += k + co
        self.head, self.bias = theta[at:at + 16], theta[at + 16]

    @staticmethod
    def conv(x, w, b):
        nz, ny, nx, ci = x.shape
        pad = torch.cat([x[:, -1:], x, x[:, :1]], 1)
        pad = torch.cat([pad[:, :, -1:], pad, pad[:, :, :1]], 2)
        zero = torch.zeros_like(pad[:1])
        pad = torch.cat([zero, pad, zero], 0)
        planes = []
        step = max(1, (1 << 21) // (ny * nx))  # planes at a time, so that the gathered taps stay small
        for k in range(0, nz, step):
            e = min(nz, k + step)
            taps = [pad[k + t // 9:e + t // 9, t // 3 % 3:t // 3 % 3 + ny, t % 3:t % 3 + nx] for t in range(27)]
            col = torch.cat([t.reshape(-1, ci) for t in taps], 1)
            planes.append((col @ w.reshape(w.shape[0], -1).T + b).view(e - k, ny, nx, -1))
        return torch.cat(planes, 0)

    def __call__(self, x):
        def block(x, i, keep):
            for w, b in self.layers[i:i + 2]:
                call = lambda v, w=w, b=b: torch.relu(self.conv(v, w, b))  # noqa: E731
                x = torch.utils.checkpoint.checkpoint(call, x, use_reentrant=False) if keep else call(x)
            return x

        def pool(x):
            nz, ny, nx, c = x.shape
            return x.view(nz // 2, 2, ny // 2, 2, nx // 2, 2, c).mean((1, 3, 5))

        def grow(x):
            for d in range(3):
                x = x.repeat_interleave(2, d)
            return x

        keep = torch.is_grad_enabled()
        e1 = block(x, 0, keep)
        e2 = block(pool(e1), 2, keep)
        e3 = block(pool(e2), 4, keep)
        d2 = block(torch.cat([grow(e3), e2], -1), 6, keep)
        d1 = block(torch.cat([grow(d2), e1], -1), 8, keep)
        return (d1 * self.head).sum(-1) + self.bias


def _features(b, rho, c2, prev):
    s = b.square().mean().sqrt()
    return torch.stack([b / s, rho.log(), c2.log(), prev / s], -1), s


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        f, rho, c2, b, dt = _solve_inputs(case, seed)
        return Box(f, dt).solve(1.0 / (rho * c2), rho, b)
    if kind in ("next", "update"):
        f, (rho, c2), (rho1, c21), b, b1, dt = _next_inputs(case, seed)
        box = Box(f, dt)
        if kind == "next":
            return box.solve(1.0 / (rho1 * c21), rho1, b1)
        return b1 - box.apply(1.0 / (rho1 * c21), box.weights(rho1), f.velocity(1.0)[2])
    if kind == "hydro":
        f, rho, mom, e, new, more, dt = _hydro_inputs(case, seed)
        box = Box(f, dt)
        p, c2 = box.eos(rho, mom, e)
        rho1, mom_s, e_s = box.advect(rho, mom, e)
        mom1, uf, e1 = box.updated(new, rho1, mom_s, e_s)
        return {"p": p, "c2": c2, "rho1": rho1, "mom_s": mom_s, "e_s": e_s,
                "b": box.rhs(rho, c2, p, mom, rho1, mom_s, **more), "mom1": mom1, "uf": uf, "e1": e1}
    if kind == "step":
        f, rho, mom, e, dt = _gresho(case, seed)
        box = Box(f, dt)
        two = box.stage(*box.stage(rho, mom, e))
        rho, mom, e = (0.5 * (a + c) for a, c in zip((rho, mom, e), two))
        return {"rho": rho, "mom": mom, "e": e}
    f, rho, c2, b, dt = _solve_inputs({"mach": 0.001, **case}, seed)
    theta = _theta(seed).double()
    if kind == "net":
        with torch.no_grad():
            x, s = _features(b, rho, c2, 1e-2 * f.uniform())
            return s * NET_SCALE * Net64(theta)(x)
    box = Box(f, dt)
    m = 1.0 / (rho * c2)
    true = box.solve(m, rho, b)
    w = box.weights(rho)
    x, s = _features(b, rho, c2, torch.zeros_like(b))
    theta.requires_grad_(True)
    d = s * (true.norm() / b.norm()) * Net64(theta)(x) - true
    with torch.no_grad():
        ad, size = box.apply(m, w, d), (true * box.apply(m, w, true)).sum()
        loss = float((d * ad).sum() / size)
    d.backward(2.0 * ad / size)
    g = theta.grad
    return {"loss": loss, "grad": g, "params": theta.detach() - LR * g / (g.abs() + 1e-8)}
