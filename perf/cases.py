"""The work that a user of this package has it do, as cases to be timed.

Three kinds of pass, each through the package's public handles:

* ``frames``: what a simulation loop repeats -- advance a lattice by ``steps``
  time steps, then take the macroscopic fields for output (``Lattice`` or
  ``Lattice3D``: ``step``, ``moments``). The lattice handle is the user's
  state and goes on from pass to pass.
* ``totals``: the same loop with the conservation check instead of the fields
  (``step``, ``mass``: four totals on the host).
* ``grad``: one gradient of a final-time loss with respect to the initial
  order parameter, surface tension and mobility (``simulate`` and its
  backward pass: checkpointed forward steps, recording replay, adjoint steps,
  initial-state map).

The states are flows in motion: drops (or a wavy layer between walls) with a
smooth random velocity field, not fluid at rest, so that every output has a
magnitude of its own. Relaxation times are those of the stable problems, since
a handle is advanced many times over.
"""
import math
import random

import torch
import torch.utils.checkpoint

from paper_1507_03521_amd import Lattice, Lattice3D
from paper_1507_03521_amd.autograd import simulate

DEV = "cuda"


# ------------------------------------------------------------------ the cases

def _case(kind, precision, nx, ny, nz, walls, trt, steps, every=0):
    """``nz`` 0: two dimensions. ``trt``: magic parameter of the two-relaxation-
    time collision, 0 for BGK. ``every``: checkpoint interval of a gradient."""
    return dict(kind=kind, precision=precision, nx=nx, ny=ny, nz=nz, walls=walls, trt=trt,
                steps=steps, every=every)


def listed():
    return [
        # the smallest call: the 32 x 32 copy that gradient checks run on,
        # looked at after every step
        dict(_case("frames", "fp64", 32, 32, 0, False, 0.0, 1), name="look32_fp64"),
        # the static-droplet validation lattice, fields every 100 steps
        dict(_case("frames", "fp64", 64, 64, 0, False, 0.0, 100), name="droplet64_fp64"),
        # the Laplace-law and phase-separation lattice, totals every 100 steps
        dict(_case("totals", "fp32", 100, 100, 0, False, 0.0, 100), name="droplet100_fp32"),
        # the Rayleigh-Taylor channel that parity and precision are stated on
        dict(_case("frames", "fp64", 256, 1024, 0, True, 0.0, 50), name="rt256_fp64"),
        # the same channel in single precision with the collision that keeps
        # it stable longest
        dict(_case("frames", "fp32", 256, 1024, 0, True, 0.25, 50), name="rt256_fp32_trt"),
        # half-precision storage, odd sizes, a medium lattice
        dict(_case("frames", "fp16", 701, 1333, 0, True, 0.0, 50), name="ragged701_fp16"),
        # the gradient workload: 512 x 512, two checkpointed segments
        dict(_case("grad", "fp64", 512, 512, 0, False, 0.0, 20, 10), name="grad512_fp64"),
        # a single-precision gradient between walls at a ragged size
        dict(_case("grad", "fp32", 1001, 2003, 0, True, 0.0, 12, 6), name="grad1001_fp32"),
        # the production Rayleigh-Taylor lattice, in both precisions
        dict(_case("frames", "fp32", 2048, 8192, 0, True, 0.0, 40), name="rt2048_fp32"),
        dict(_case("frames", "fp64", 2048, 8192, 0, True, 0.0, 20), name="rt2048_fp64"),
        # three dimensions: the droplet cube and the Rayleigh-Taylor box
        dict(_case("frames", "fp64", 32, 32, 32, False, 0.0, 50), name="droplet3d_fp64"),
        dict(_case("frames", "fp32", 256, 256, 256, True, 0.0, 20), name="rt3d_fp32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the same ranges: lattices from 32 x 32 to 2048 x 8192
    and from 16^3 to 256^3 in any aspect between, any precision, boundary and
    collision the kind of pass offers, one step to a hundred."""
    kind = rng.choice(("frames", "frames", "frames", "totals", "grad", "grad", "frames3", "frames3"))
    walls = rng.random() < 0.5
    if kind == "frames3":
        n = [_log(rng, 16, 256) for _ in range(3)]
        precision = rng.choice(("fp32", "fp64"))
        budget = 2.0e8 if precision == "fp32" else 8.0e7
        return _case("frames", precision, n[0], n[1], n[2], walls, rng.choice((0.0, 0.0, 0.25)),
                     max(1, min(_log(rng, 1, 50), int(budget / (n[0] * n[1] * n[2])))))
    if kind == "grad":
        nx, ny = _log(rng, 32, 1024), _log(rng, 32, 2048)
        steps = max(2, min(_log(rng, 4, 40), int(2.4e7 / (nx * ny))))
        return _case("grad", rng.choice(("fp32", "fp64")), nx, ny, 0, walls, 0.0, steps,
                     rng.randint(2, steps))
    nx, ny = _log(rng, 32, 2048), _log(rng, 32, 8192)
    precision = rng.choice(("fp64", "fp64", "fp32", "fp32", "fp16"))
    budget = 6.0e8 if precision != "fp64" else 3.0e8
    steps = max(1, min(_log(rng, 1, 100), int(budget / (nx * ny))))
    return _case(kind, precision, nx, ny, 0, walls, rng.choice((0.0, 0.0, 0.25)), steps)


# ----------------------------------------------------------------- the inputs

def _params(case):
    """Density ratio 10 and sigma = 0.01 for drops in a periodic box; the
    Rayleigh-Taylor values (ratio 3, weak tension, gravity) between walls."""
    if case["walls"]:
        p = dict(rho_A=1.0, rho_B=1.0 / 3.0, sigma=4e-4, W=4.0, M=0.02, tau_f=0.582, tau_g=1.0,
                 gx=0.0, gy=0.0, rho_ref=1.0, bc=1)
        p["gz" if case["nz"] else "gy"] = -6.25e-6
    else:
        p = dict(rho_A=1.0, rho_B=0.1, sigma=0.01, W=4.0, M=0.1, tau_f=0.8, tau_g=0.8,
                 gx=0.0, gy=0.0, rho_ref=1.0, bc=0)
    p.update(nx=case["nx"], ny=case["ny"])
    if case["nz"]:
        p["nz"] = case["nz"]
        p.setdefault("gz", 0.0)
    if case["trt"]:
        p["trt_magic"] = case["trt"]
    return p


def _shape(case):
    return ((case["nz"],) if case["nz"] else ()) + (case["ny"], case["nx"])


def _grid(case):
    """Coordinates x, y[, z] as broadcastable float64 arrays."""
    shape = _shape(case)
    out = []
    for a in reversed(range(len(shape))):
        v = torch.arange(shape[a], dtype=torch.float64, device=DEV)
        out.append(v.reshape([-1 if b == a else 1 for b in range(len(shape))]))
    return out


def _waves(rng, xs, sizes, count=4):
    """A smooth field of order one: ``count`` periodic Fourier modes."""
    acc = 0.0
    for _ in range(count):
        arg = rng.uniform(0.0, 2.0 * math.pi)
        for x, n in zip(xs, sizes):
            arg = arg + (2.0 * math.pi * rng.randint(-2, 2) / n) * x
        acc = acc + rng.uniform(0.3, 1.0) * torch.cos(arg)
    return acc / math.sqrt(count)


def _phi0(case, seed):
    """Initial order parameter: drops, or heavy over light fluid with a wavy
    interface between walls; the profile is wider than the equilibrium one and
    lightly perturbed, so the interface relaxes."""
    rng = random.Random(seed * 2 + 1)
    xs = _grid(case)
    sizes = [case["nx"], case["ny"]] + ([case["nz"]] if case["nz"] else [])
    if case["walls"]:
        up, n = xs[-1], sizes[-1]
        h = n / 2 + 0.08 * n * _waves(rng, xs[:-1], sizes[:-1])
        phi = 0.5 + 0.5 * torch.tanh(2.0 * (up - h) / 5.5)
    else:
        phi = 0.0
        for k in range(2):
            r2 = 0.0
            for x, n in zip(xs, sizes):
                d = torch.remainder(x - n * (0.25 + 0.5 * k + rng.uniform(-0.06, 0.06)) + n / 2,
                                    n) - n / 2
                r2 = r2 + d * d
            r = min(sizes) * rng.uniform(0.14, 0.2)
            phi = phi + 0.5 + 0.5 * torch.tanh(2.0 * (r - torch.sqrt(r2)) / 5.5)
    phi = phi + 0.01 * _waves(rng, xs, sizes)
    return phi.expand(_shape(case)).contiguous()


def _state(case, seed):
    """Populations of a flow in motion, canonical pre-collision layout:
    f = w (p + rho s(u) / 3) and g = phi in the rest slot plus w phi s(u)."""
    c, w = _lattice(case)
    rng = random.Random(seed * 2)
    xs = _grid(case)
    sizes = [case["nx"], case["ny"]] + ([case["nz"]] if case["nz"] else [])
    prm = _params(case)
    phi = _phi0(case, seed)
    rho = prm["rho_B"] + (prm["rho_A"] - prm["rho_B"]) * phi
    p = 1e-3 * _waves(rng, xs, sizes) + 2e-3
    u = [0.02 * _waves(rng, xs, sizes) for _ in sizes]
    f, g = [], []
    for ci, wi in zip(c, w):
        s = _s(ci, u)
        f.append((wi * (p + rho * s / 3.0)).expand(phi.shape))
        g.append((wi * phi * s).expand(phi.shape))
    g[0] = phi - sum(g[1:])
    return phi, torch.stack(f), torch.stack(g)


def prepare(case, seed):
    if case["kind"] == "grad":
        # a single-precision run takes and returns single-precision tensors
        dt = torch.float32 if case["precision"] == "fp32" else torch.float64
        prm = _params(case)
        phi0 = _phi0(case, seed).to(dt).requires_grad_()
        sigma = torch.tensor(prm["sigma"], dtype=dt, requires_grad=True)
        M = torch.tensor(prm["M"], dtype=dt, requires_grad=True)
        # cotangent of a quadratic distance to a smooth target
        rng = random.Random(seed * 2)
        target = 0.5 + 0.2 * _waves(rng, _grid(case), [case["nx"], case["ny"]])
        return dict(case=case, params=prm, phi0=phi0, sigma=sigma, M=M,
                    weight=(phi0.detach() - target).to(dt).contiguous())
    phi, f, g = _state(case, seed)
    lat = (Lattice3D if case["nz"] else Lattice)(_params(case), phi, precision=case["precision"])
    lat.set_state(f, g)
    return dict(case=case, lat=lat)


#: Type that a program keeps the output fields in, by the lattice's storage.
KEEP = dict(fp64=torch.float64, fp32=torch.float32, fp16=torch.float16)


def run(state):
    case = state["case"]
    if case["kind"] == "grad":
        leaves = (state["phi0"], state["sigma"], state["M"])
        phi = simulate(*leaves, state["params"], case["steps"], checkpoint=case["every"],
                       precision=case["precision"]).to(state["phi0"].dtype)
        got = torch.autograd.grad(phi, leaves, state["weight"])
        return dict(phi=phi.detach(), dphi0=got[0], dsigma=got[1], dM=got[2])
    lat = state["lat"]
    lat.step(case["steps"])
    if case["kind"] == "totals":
        return list(lat.mass())
    names = ("phi", "ux", "uy", "uz") if case["nz"] else ("phi", "ux", "uy", "p")
    return {k: v.to(KEEP[case["precision"]]) for k, v in lat.moments(names).items()}


def work(case):
    """Populations in and out once, the outputs once; operations of Sec. III's
    step as written (moments, three stencils, two collisions). A gradient: the
    forward steps, their replay, and adjoint steps of twice a step's work."""
    n = case["nx"] * case["ny"] * max(1, case["nz"])
    q = 19 if case["nz"] else 9
    word = dict(fp64=8, fp32=4, fp16=2)[case["precision"]]
    per = 1250 if case["nz"] else 560
    if case["kind"] == "grad":
        return dict(bytes=n * word * (3 + 2 * q * 2), flops=float(per) * 4 * n * case["steps"])
    out = 0 if case["kind"] == "totals" else 4 * word * n
    return dict(bytes=n * word * 2 * q * 2 + out, flops=float(per) * n * case["steps"])


# ------------------------------------------------- the same in plain 64 bits

def _lattice(case):
    if not case["nz"]:
        c = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]
        w = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
    else:
        c = [(0, 0, 0)]
        for a in range(3):
            for s in (1, -1):
                c.append(tuple(s if b == a else 0 for b in range(3)))
        for a, b in ((0, 1), (0, 2), (1, 2)):
            for s, t in ((1, 1), (-1, -1), (1, -1), (-1, 1)):
                c.append(tuple(s if d == a else t if d == b else 0 for d in range(3)))
        w = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
    return c, w


def _dot(ci, v):
    acc = 0.0
    for k, x in zip(ci, v):
        if k:
            acc = acc + k * x
    return acc


def _s(ci, u):
    cu = _dot(ci, u)
    return 3.0 * cu + 4.5 * cu * cu - 1.5 * sum(x * x for x in u)


def _at(v, ci, walls):
    """v(x + c): periodic, or with the boundary layer mirrored beyond a wall."""
    nd = v.dim()
    for a, k in enumerate(ci):
        d = nd - 1 - a
        if not k:
            continue
        if walls and d == 0:
            v = torch.cat((v[1:], v[-1:])) if k > 0 else torch.cat((v[:1], v[:-1]))
        else:
            v = torch.roll(v, -k, d)
    return v


class _Plain:
    """The coupled step on whole-lattice float64 tensors."""

    def __init__(self, case, sigma=None, M=None):
        q = _params(case)
        self.c, self.w = _lattice(case)
        self.walls = case["walls"]
        self.q = q
        self.trt = case["trt"]
        sigma = q["sigma"] if sigma is None else sigma
        self.M = q["M"] if M is None else M
        self.beta, self.kappa = 12.0 * sigma / q["W"], 1.5 * sigma * q["W"]
        self.alpha = 3.0 * self.M / (q["tau_g"] - 0.5)
        self.gamma = q["rho_A"] / q["rho_B"] - 1.0
        self.drho = q["rho_A"] - q["rho_B"]
        self.grav = [q["gx"], q["gy"]] + ([q["gz"]] if case["nz"] else [])
        self.opp = [self.c.index(tuple(-k for k in ci)) for ci in self.c]

    def stencil(self, v):
        grad = [0.0] * len(self.grav)
        lap = 0.0
        for ci, wi in zip(self.c[1:], self.w[1:]):
            n = _at(v, ci, self.walls)
            for a, k in enumerate(ci):
                if k:
                    grad[a] = grad[a] + 3.0 * wi * k * n
            lap = lap + 6.0 * wi * (n - v)
        return grad, lap

    def mu(self, phi, lap):
        return 4.0 * self.beta * (phi - 1.0) * phi * (phi - 0.5) - self.kappa * lap

    def macro(self, f, g):
        q = self.q
        phi, S = g.sum(0), f.sum(0)
        j = [sum(ci[a] * fi for ci, fi in zip(self.c, f) if ci[a]) for a in range(len(self.grav))]
        dphi, lap = self.stencil(phi)
        mu = self.mu(phi, lap)
        dmu, lapmu = self.stencil(mu)
        rho = q["rho_B"] + self.drho * phi
        F = [-phi * m + (rho - q["rho_ref"]) * b for m, b in zip(dmu, self.grav)]
        u = [3.0 * (a + b / 6.0) / rho for a, b in zip(j, F)]
        drho = [self.drho * d for d in dphi]
        D = self.M * lapmu
        p = S + (sum(a * b for a, b in zip(u, drho)) - self.gamma * rho * D) / 6.0
        return phi, mu, rho, F, u, drho, D, p

    def start(self, phi0):
        amu = self.alpha * self.mu(phi0, self.stencil(phi0)[1])
        g = [phi0 - (1.0 - self.w[0]) * amu] + [wi * amu for wi in self.w[1:]]
        g = torch.stack(g)
        return torch.zeros_like(g), g

    def step(self, f, g):
        q = self.q
        phi, mu, rho, F, u, drho, D, p = self.macro(f, g)
        dp = self.stencil(p)[0]
        tf, tg = q["tau_f"], q["tau_g"]
        feq, Fs, gn = [], [], []
        for i, (ci, wi) in enumerate(zip(self.c, self.w)):
            s = _s(ci, u)
            cu = [k - x for k, x in zip(ci, u)]
            feq.append(wi * (p + rho * s / 3.0))
            Fs.append(wi * (sum(a * ((1.0 + s) * b + s * d / 3.0)
                                for a, b, d in zip(cu, F, drho)) - rho * self.gamma * D / 3.0))
            H = phi - (1.0 - wi) * self.alpha * mu if i == 0 else wi * self.alpha * mu
            G = -3.0 * phi / rho * wi * (1.0 + s) * sum(a * (d - b)
                                                       for a, d, b in zip(cu, dp, F))
            geq = H + wi * phi * s
            gn.append(g[i] - (g[i] - geq) / tg + (1.0 - 0.5 / tg) * G)
        if self.trt:
            tm = 0.5 + self.trt / (tf - 0.5)
            fn = []
            for i, o in enumerate(self.opp):
                even = [0.5 * (x[i] + x[o]) for x in (f, feq, Fs)]
                odd = [0.5 * (x[i] - x[o]) for x in (f, feq, Fs)]
                fn.append(f[i] - (even[0] - even[1]) / tf + (1.0 - 0.5 / tf) * even[2]
                          - (odd[0] - odd[1]) / tm + (1.0 - 0.5 / tm) * odd[2])
        else:
            fn = [f[i] - (f[i] - feq[i]) / tf + (1.0 - 0.5 / tf) * Fs[i] for i in range(len(feq))]
        return self.stream(fn), self.stream(gn)

    def stream(self, x):
        out = []
        for i, ci in enumerate(self.c):
            v = x[i]
            nd = v.dim()
            for a, k in enumerate(ci):
                if k:
                    v = torch.roll(v, k, nd - 1 - a)
            if self.walls and ci[-1]:
                # half-way bounce-back: the layer that a wall feeds
                o = x[self.opp[i]]
                v = torch.cat((o[:1], v[1:])) if ci[-1] > 0 else torch.cat((v[:-1], o[-1:]))
            out.append(v)
        return torch.stack(out)


def exact(case, seed):
    if case["kind"] == "grad":
        s = prepare(case, seed)
        phi0, sigma, M = (s[k].detach().to(DEV, torch.float64).requires_grad_()
                          for k in ("phi0", "sigma", "M"))

        def many(f, g, sigma, M):
            return _Plain(case, sigma, M).step(f, g)

        f, g = _Plain(case, sigma, M).start(phi0)
        for _ in range(case["steps"]):
            f, g = torch.utils.checkpoint.checkpoint(many, f, g, sigma, M, use_reentrant=False)
        phi = g.sum(0)
        got = torch.autograd.grad(phi, (phi0, sigma, M), s["weight"].to(torch.float64))
        return dict(phi=phi.detach(), dphi0=got[0], dsigma=got[1], dM=got[2])
    plain = _Plain(case)
    _, f, g = _state(case, seed)
    with torch.no_grad():
        for _ in range(case["steps"]):
            f, g = plain.step(f, g)
        phi, mu, rho, F, u, drho, D, p = plain.macro(f, g)
        if case["kind"] == "totals":
            return [float(x.sum()) for x in (phi, rho, rho * u[0], rho * u[1])]
        out = dict(phi=phi, ux=u[0], uy=u[1])
        out["uz" if case["nz"] else "p"] = u[2] if case["nz"] else p
        return out
