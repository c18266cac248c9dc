"""What this library is timed on: the calls a solver makes, over the sizes it makes them at.

A solver on a Cartesian grid with an embedded body builds a plan (`gcr.Plan`, or `gcr.Batch` for a sweep of
many bodies) when the body is placed, moves it (`Plan.update`) when the body moves, and in every time step fills
its fields' ghost cells and reads values, gradients and forces off the body (`Plan.fill`, `Plan.surface`,
`Plan.forces`, or `Batch.forward`); a design loop differentiates that step (`autograd`).  Each case is one such
call or step.  Grids, bodies and boundary data are of the kinds `synth.workloads` has, at its sizes and between
them; positions, coefficients and fields come from the seed.

`exact` is the same mathematics in plain torch, in float64, without the library.
"""
import itertools
import math
import random

import numpy as np
import torch

import paper_2609_10165_amd as gcr
from paper_2609_10165_amd import autograd as gcr_autograd

CGC, CGC_ES, HGC, LAYER2 = gcr.CGC, gcr.CGC_ES, gcr.HGC, gcr.LAYER2
DIRICHLET, NEUMANN, MIXED = gcr.DIRICHLET, gcr.NEUMANN, gcr.MIXED
F64 = torch.float64
SCHEMES = {"cgc": CGC, "cgc_es": CGC_ES, "hgc": HGC, "hgc2": HGC | LAYER2, "cgc_es2": CGC_ES | LAYER2}
THREE_D = ("sphere", "shstar")


# ----------------------------------------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------------------------------------

def listed():
    return [
        # one small body placed and its first fill and surface values: the shortest build, where launches and the
        # two waits for the host count
        {"name": "plan_circle128", "do": "plan", "body": "circle", "n": 128, "scheme": "hgc", "stretch": 1.0,
         "nf": 1, "bc": "plain", "nq": 256},
        # a thin 2D section on a fine grid of odd size: a long chain of levels
        {"name": "plan_airfoil2731", "do": "plan", "body": "airfoil", "n": 2731, "scheme": "hgc", "stretch": 1.0,
         "nf": 3, "bc": "plain", "nq": 2048},
        # a stretched 3D grid with a second ghost layer, as flow runs near a moving or high-order wall use
        {"name": "plan_sphere190_stretched_l2", "do": "plan", "body": "sphere", "n": 190, "scheme": "hgc2",
         "stretch": 1.01, "nf": 4, "bc": "plain", "nq": 2048},
        # a large 3D build: the classification of every cell and a graph beyond one workgroup
        {"name": "plan_sphere512", "do": "plan", "body": "sphere", "n": 512, "scheme": "hgc", "stretch": 1.0,
         "nf": 1, "bc": "plain", "nq": 2048},
        # a body moving through a 3D grid, four moves: re-plan, the cells each move exposes, a field filled
        {"name": "move_sphere256_l2", "do": "move", "body": "sphere", "n": 256, "scheme": "hgc2", "stretch": 1.0,
         "nf": 1, "bc": "plain"},
        # a sweep over 64 uneven bodies: all plans by shared launches (the benchmark's batch)
        {"name": "build_stars64", "do": "build", "body": "star", "ninst": 64, "nmin": 128, "nmax": 2048, "mix": 1,
         "scheme": "hgc"},
        # the same batch in a time step: fill of three fields with mixed data, surface values, forces
        {"name": "forward_stars64", "do": "forward", "body": "star", "ninst": 64, "nmin": 128, "nmax": 2048,
         "mix": 1, "scheme": "hgc", "nf": 3, "bc": "mixed", "nq": 256},
        # a few 3D bodies in a time step
        {"name": "forward_spheres7", "do": "forward", "body": "sphere", "ninst": 7, "nmin": 60, "nmax": 200,
         "mix": 3, "scheme": "hgc", "nf": 4, "bc": "plain", "nq": 2048},
        # one time step of a static body, plan kept: the smallest, a deep 2D chain, an ordinary 3D one
        {"name": "step_circle128", "do": "step", "body": "circle", "n": 128, "scheme": "hgc", "stretch": 1.0,
         "nf": 3, "bc": "plain", "nq": 256},
        {"name": "step_airfoil4096", "do": "step", "body": "airfoil", "n": 4096, "scheme": "hgc", "stretch": 1.0,
         "nf": 3, "bc": "plain", "nq": 2048},
        {"name": "step_sphere256", "do": "step", "body": "sphere", "n": 256, "scheme": "hgc", "stretch": 1.0,
         "nf": 4, "bc": "plain", "nq": 2048},
        # a design loop: the force on a body and its gradient by the fields and the boundary data
        {"name": "grad_shstar160", "do": "grad", "body": "shstar", "n": 160, "scheme": "hgc", "stretch": 1.0,
         "nf": 4, "bc": "plain", "nq": 2048},
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm, odd as often as even."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(("plan", "plan", "move", "build", "forward", "forward", "step", "step", "grad"))
    if do in ("build", "forward"):
        body = rng.choice(("star", "star", "sphere"))
        case = {"do": do, "body": body, "ninst": _log(rng, 2, 64) if body == "star" else rng.randint(2, 7),
                "nmin": rng.randint(100, 300) if body == "star" else rng.randint(40, 80),
                "nmax": _log(rng, 400, 2048) if body == "star" else rng.randint(90, 200),
                "mix": rng.randrange(1 << 20), "scheme": "hgc"}
        if do == "forward":
            case.update({"nf": 3 if body == "star" else 4, "bc": rng.choice(("plain", "mixed")),
                         "nq": rng.choice((100, 256, 1001))})
        return case
    body = rng.choice(("sphere",) if do == "move" else ("shstar", "sphere", "circle", "star") if do == "grad"
                      else ("circle", "star", "airfoil", "sphere", "sphere", "shstar"))
    lo, hi = {"plan": (48, 512), "step": (48, 256), "move": (48, 256), "grad": (48, 160)}[do] if body in THREE_D \
        else {"plan": (96, 3000), "step": (96, 4096), "grad": (96, 1024)}[do]
    if body == "shstar":
        hi = min(hi, 256)
    if body == "airfoil":
        lo = 300
    round_body = body in ("circle", "sphere")
    scheme = "hgc" if not round_body else rng.choice(("cgc_es", "hgc2", "cgc_es2") if do == "move" else
                                                      ("hgc", "hgc", "cgc", "cgc_es", "hgc2"))
    case = {"do": do, "body": body, "n": _log(rng, lo, hi), "scheme": scheme, "stretch": 1.0}
    if round_body and do != "move" and case["n"] <= 256 and rng.random() < 0.3:
        case["stretch"] = round(1.0 + rng.uniform(0.2, 2.0) / case["n"], 6)
    if do == "move":
        case.update({"nf": 1, "bc": "plain"})
    else:
        nf = 1 if do == "plan" and case["n"] > 256 else 4 if body in THREE_D else 3
        case.update({"nf": nf, "bc": "plain" if do == "plan" else rng.choice(("plain", "mixed")),
                     "nq": rng.choice((256, 777, 2048))})
    return case


def _sizes(case):
    if "n" in case:
        return [case["n"]]
    rng = random.Random(case["mix"])
    return [rng.randint(case["nmin"], case["nmax"]) for _ in range(case["ninst"])]


def _ghosts(case, n):
    """About how many ghosts a body has: its surface in faces of a cell, twice that with a second layer."""
    per = {"circle": 2 * math.pi * 0.5 / 4, "star": 2 * math.pi * 0.45 / 2, "airfoil": 2.06 / 4,
           "sphere": 4 * math.pi * 0.09 / 4, "shstar": 4 * math.pi * 0.09 / 4}[case["body"]]
    t = (n / 2) * math.log(case.get("stretch", 1.0))  # a stretched grid is finer at the body
    n *= math.expm1(t) / t if t else 1.0
    return per * n ** (2 if case["body"] in THREE_D else 1) * (2 if case["scheme"].endswith("2") else 1)


def work(case):
    """Bytes and operations of one pass.  Building: a tag per cell and a ghost's record; a move: its record.
    Filling: per ghost and field the other corners of
    the stencil, the datum and the result, per ghost its record; a surface point: its position, normal and
    weight, and per field the corners read, the value and the gradient.  A gradient: the step, its transpose,
    and the dense copies and gradients that come back."""
    d = 3 if case["body"] in THREE_D else 2
    nc = 2 ** d
    cells = sum(float(n) ** d for n in _sizes(case))
    ng = sum(_ghosts(case, n) for n in _sizes(case))
    record = 4 + 4 + 8 * 2 * d + 8 + 4 * d + 4
    foot = 16 * d
    solve = 60.0 * d * ng  # the closest point, roughly
    nf, nq = case.get("nf", 0), case.get("nq", 0) * len(_sizes(case))
    fill = ng * (nf * 8 * (nc + 1) + 8 + 16 * d)
    read = nq * (8 * (2 * d + 1) + 4 + nf * 8 * (nc + 1 + d))
    flop = ng * nf * 2 * nc + nq * nf * (d + 1) * 2 * nc
    if case["do"] == "plan":
        return {"bytes": cells + ng * record + fill + read, "flops": solve + flop}
    if case["do"] == "move":
        return {"bytes": 4 * (ng * record + fill), "flops": 4 * (solve + flop)}
    if case["do"] == "build":
        return {"bytes": cells + ng * foot, "flops": solve}
    if case["do"] in ("forward", "step"):
        return {"bytes": fill + read, "flops": flop}
    return {"bytes": 2 * (fill + read) + nf * cells * 8 * 3, "flops": 2 * flop}


# ----------------------------------------------------------------------------------------------------------
# grids, bodies, fields and surface points from the seed
# ----------------------------------------------------------------------------------------------------------

class Grid:
    """A grid as gcr.Plan takes it: cells, lower corner, spacing, and the faces of stretched axes."""

    def __init__(self, dim, n, lo, length, stretch):
        self.dim, self.n = dim, (n,) * dim + (1,) * (3 - dim)
        self.lo, self.h = tuple(lo) + (0.0,) * (3 - dim), (length / n,) * dim + (1.0,) * (3 - dim)
        self.faces = None
        if stretch != 1.0:  # widths grow by a fixed ratio from the middle of the axis outward
            faces = []
            for a in range(dim):
                w = (stretch * (1.0 + 0.002 * a / n)) ** np.abs(np.arange(n) - (n - 1) / 2.0)
                f = lo[a] + np.concatenate([[0.0], np.cumsum(w * (length / w.sum()))])
                f[-1] = lo[a] + length
                faces.append(f)
            self.faces = tuple(faces) + (None,) * (3 - dim)

    def centres(self, a):
        f = None if self.faces is None else self.faces[a]
        if f is None:
            return self.lo[a] + (torch.arange(self.n[a], dtype=F64, device="cuda") + 0.5) * self.h[a]
        f = torch.tensor(f, dtype=F64, device="cuda")
        return 0.5 * (f[:-1] + f[1:])

    def widths(self, a):
        f = None if self.faces is None else self.faces[a]
        if f is None:
            return torch.full((self.n[a],), self.h[a], dtype=F64, device="cuda")
        f = torch.tensor(f, dtype=F64, device="cuda")
        return f[1:] - f[:-1]

    def mesh(self):
        """Broadcastable centre coordinates (x fastest: the last axis), x first."""
        out = []
        for a in range(self.dim):
            shape = [1] * self.dim
            shape[self.dim - 1 - a] = self.n[a]
            out.append(self.centres(a).view(shape))
        return out


class Shape:
    def __init__(self, kind, center, r0=0.0, coef=(), ncoef=0, thick=0.12, incidence=0.0):
        self.kind, self.center, self.r0, self.ncoef = kind, tuple(center), r0, ncoef
        self.coef = np.asarray(coef, dtype=np.float64)
        self.chord, self.thick, self.incidence = 1.0, thick, incidence


def _body(body, n, stretch, rng):
    """A grid and a body at a position inside a cell near the middle, as synth.workloads places them."""
    if body in THREE_D:
        g = Grid(3, n, (-1.0,) * 3, 2.0, stretch)
    elif body == "circle":
        g = Grid(2, n, (-2.0,) * 2, 4.0, stretch)
    elif body == "star":
        g = Grid(2, n, (-1.0,) * 2, 2.0, stretch)
    else:
        g = Grid(2, n, (-1.0, -2.0), 4.0, stretch)
    c = tuple(rng.uniform(0.0, g.h[0]) for _ in range(g.dim)) + (0.0,) * (3 - g.dim)
    if body == "circle":
        return g, Shape(gcr.SPHERE, c, 0.5)
    if body == "sphere":
        return g, Shape(gcr.SPHERE, c, 0.3)
    if body == "airfoil":
        return g, Shape(gcr.AIRFOIL, c, incidence=math.radians(8.0))
    if body == "star":
        coef = np.zeros((6, 2))
        for k in range(2, 6):
            a, ph = rng.uniform(0, 0.05), rng.uniform(0, 2 * math.pi)
            coef[k] = a * math.cos(ph), -a * math.sin(ph)
        return g, Shape(gcr.STAR2D, c, rng.uniform(0.3, 0.6), coef.ravel(), 6)
    coef = np.zeros(25)
    coef[4:] = [rng.uniform(0, 0.04) for _ in range(21)]
    return g, Shape(gcr.SHSTAR, c, 0.3, coef, 25)


class Field:
    """A smooth field of two waves, as a velocity component or a pressure near a body is."""

    def __init__(self, dim, rng):
        self.k = [[rng.uniform(-3.0, 3.0) for _ in range(dim)] for _ in range(2)]
        self.p = [rng.uniform(0.0, 2 * math.pi) for _ in range(2)]

    def _arg(self, j, x):
        return sum(k * v for k, v in zip(self.k[j], x)) + self.p[j]

    def value(self, x):
        return torch.sin(self._arg(0, x)) + 0.5 * torch.cos(self._arg(1, x))

    def normal(self, x, n):
        c, s = torch.cos(self._arg(0, x)), torch.sin(self._arg(1, x))
        return sum((a * c - 0.5 * b * s) * m for a, b, m in zip(self.k[0], self.k[1], n))


def _boundary(fields, kinds, center, beta, S, n):
    """Boundary data at the foot points: values where the data are Dirichlet, normal derivatives where Neumann,
    and the kinds of mixed data (Dirichlet on the side of the body that faces the angle beta)."""
    vals, types = [], []
    for f, kind, b in zip(fields, kinds, beta):
        if kind == MIXED:
            t = torch.cos(torch.atan2(S[1] - center[1], S[0] - center[0]) - b) < 0
        else:
            t = torch.full(S.shape[1:], kind == NEUMANN, device="cuda")
        vals.append(torch.where(t, f.normal(S, n), f.value(S)).contiguous())
        types.append(t.to(torch.uint8))
    return vals, types


def _kinds(case):
    return [MIXED] * case["nf"] if case["bc"] == "mixed" else [DIRICHLET] * (case["nf"] - 1) + [NEUMANN]


def _star_radius(s, th):
    r, r1, r2 = torch.ones_like(th), torch.zeros_like(th), torch.zeros_like(th)
    for k in range(s.ncoef):
        a, b = float(s.coef[2 * k]), float(s.coef[2 * k + 1])
        ck, sk = torch.cos(k * th), torch.sin(k * th)
        r, r1, r2 = r + a * ck + b * sk, r1 + k * (b * ck - a * sk), r2 - k * k * (a * ck + b * sk)
    return s.r0 * r, s.r0 * r1, s.r0 * r2


def _sh_radius(s, v):
    """r of the unit vectors along v [3][m]: real Schmidt semi-normalised harmonics, a polynomial of v."""
    x, y, z = v / (v * v).sum(0).sqrt()
    total = torch.ones_like(x)
    cr, ci = torch.ones_like(x), torch.zeros_like(x)  # (x + i y)^m
    for m in range(5):
        p0, p1 = torch.zeros_like(x), torch.full_like(x, float(math.prod(range(1, 2 * m, 2))))  # P_m^m / sin^m
        for l in range(m, 5):
            if l > m:
                p0, p1 = p1, ((2 * l - 1) * z * p1 - (l + m - 1) * p0) / (l - m)
            norm = 1.0 if m == 0 else math.sqrt(2.0 * math.factorial(l - m) / math.factorial(l + m))
            total = total + float(s.coef[l * l + l + m]) * norm * p1 * cr
            if m:
                total = total + float(s.coef[l * l + l - m]) * norm * p1 * ci
        cr, ci = cr * x - ci * y, cr * y + ci * x
    return s.r0 * total


def _sh_grad(s, v):
    v = v.detach().requires_grad_()
    with torch.enable_grad():
        r = _sh_radius(s, v)
        g, = torch.autograd.grad(r.sum(), v)
    return r.detach(), g


def _surface_points(s, dim, nq):
    """Points, outward normals and weights of the body's surface."""
    t = (torch.arange(nq, dtype=F64, device="cuda") + 0.5) / nq
    c = torch.tensor(s.center[:dim], dtype=F64, device="cuda")[:, None]
    if dim == 3:  # a spiral of equal steps in z
        z, ph = 1 - 2 * t, math.pi * (3 - math.sqrt(5)) * torch.arange(nq, dtype=F64, device="cuda")
        w = torch.stack([(1 - z * z).sqrt() * torch.cos(ph), (1 - z * z).sqrt() * torch.sin(ph), z])
        r, g = _sh_grad(s, w) if s.kind == gcr.SHSTAR else (torch.full_like(z, s.r0), torch.zeros_like(w))
        m = w - g / r
        area = r * r * (m * m).sum(0).sqrt() * (4 * math.pi / nq)
        return c + r * w, m / (m * m).sum(0).sqrt(), area
    if s.kind == gcr.AIRFOIL:
        a = 2 * t - 1
        X, D, _ = _airfoil_curve(s, a)
        T = _airfoil_world(s, D)
        ds = (T * T).sum(0).sqrt()
        return c + _airfoil_world(s, X), torch.stack([-T[1], T[0]]) / ds, ds * (2.0 / nq)
    th = 2 * math.pi * t
    r, r1, _ = _star_radius(s, th) if s.kind == gcr.STAR2D else (torch.full_like(t, s.r0),) + (torch.zeros_like(t),) * 2
    T = torch.stack([r1 * torch.cos(th) - r * torch.sin(th), r1 * torch.sin(th) + r * torch.cos(th)])
    ds = (T * T).sum(0).sqrt()
    return c + r * torch.stack([torch.cos(th), torch.sin(th)]), torch.stack([T[1], -T[0]]) / ds, ds * (2 * math.pi / nq)


def _bodies(case, seed):
    rng = random.Random(seed * 1000003 + 17)
    return [_body(case["body"], n, case.get("stretch", 1.0), rng) for n in _sizes(case)]


def _fields(case, seed):
    """The fields and their mixed data's angles, and the sample of every field on a grid."""
    rng = random.Random(seed * 1000003 + 29)
    dim = 3 if case["body"] in THREE_D else 2
    return [Field(dim, rng) for _ in range(case["nf"])], [rng.uniform(0, 2 * math.pi) for _ in range(case["nf"])]


# ----------------------------------------------------------------------------------------------------------
# prepare and run
# ----------------------------------------------------------------------------------------------------------

def prepare(case, seed):
    do, scheme = case["do"], SCHEMES[case["scheme"]]
    bodies = _bodies(case, seed)
    st = {"do": do, "scheme": scheme, "grid": bodies[0][0], "shape": bodies[0][1]}
    dim, cap = bodies[0][0].dim, _room(case)
    if do == "build":
        st["spec"] = gcr.BatchSpec([g for g, _ in bodies], [s for _, s in bodies], [scheme] * len(bodies))
        st["S"], st["n"] = (torch.zeros(dim * cap, dtype=F64, device="cuda") for _ in range(2))
        return st
    fields, beta = _fields(case, seed)
    kinds, nf = _kinds(case), case["nf"]
    st.update({"kinds": kinds, "mu": 0.7})
    if do in ("plan", "move"):  # walls at a constant value or with a constant flux
        st["wall"] = [torch.full((cap,), b, dtype=F64, device="cuda") for b in beta]
    if do == "move":  # around a small square, 0.4 of a cell a move
        st["orbit"] = _orbit(*bodies[0])
        st["plans"] = [gcr.Plan(st["grid"], st["orbit"][k], scheme) for k in (0, 1)]
        u = fields[0].value(st["grid"].mesh()).reshape(-1)
        st["u"], st["fresh"] = [u.clone() for _ in range(4)], max(64, cap // 4)
        st["at"] = torch.arange(st["fresh"], device="cuda")
        return st
    pts = [_surface_points(s, dim, case["nq"]) for _, s in bodies]
    if do == "forward":
        ninst = len(bodies)
        B = gcr.Batch([g for g, _ in bodies], [s for _, s in bodies], [scheme] * ninst)
        S, n = B.foot_points()
        u = torch.empty(nf * sum(g.n[0] * g.n[1] * g.n[2] for g, _ in bodies), dtype=F64, device="cuda")
        views, bcv, bct, at, off = [], [], [], 0, 0
        for (g, s), ng in zip(bodies, B.counts()):
            cells = g.n[0] * g.n[1] * g.n[2]
            for f in fields:
                u[at:at + cells] = f.value(g.mesh()).reshape(-1)
                views.append(u[at:at + cells])
                at += cells
            v, t = _boundary(fields, kinds, s.center, beta, S[:, off:off + ng], n[:, off:off + ng])
            bcv, bct, off = bcv + v, bct + t, off + ng
        nq, k = case["nq"], ninst * nf
        st.update({"batch": B, "u": u, "F": torch.zeros((ninst, 3), dtype=F64, device="cuda"),
                   "val": torch.empty((k, nq), dtype=F64, device="cuda"),
                   "grad": torch.empty((k, dim, nq), dtype=F64, device="cuda")})
        st["args"] = gcr.ForwardArgs(nf, views, kinds, bcv, bc_type=bct if case["bc"] == "mixed" else None,
                                     nq=[nq] * ninst, xq=[p[0] for p in pts], nrm=[p[1] for p in pts],
                                     wq=[p[2] for p in pts], p_field=nf - 1, u_first=0, mu=st["mu"], F=st["F"],
                                     sval=list(st["val"]), sgrad=list(st["grad"]))
        return st
    st.update({"pts": pts[0], "u": [f.value(st["grid"].mesh()).reshape(-1).contiguous() for f in fields]})
    if do == "plan":
        return st
    st["plan"] = plan = gcr.Plan(st["grid"], st["shape"], scheme)
    S, n = plan.foot_points()
    bcv, bct = _boundary(fields, kinds, st["shape"].center, beta, S, n)
    st.update({"bcv": bcv, "bct": bct if case["bc"] == "mixed" else None})
    if do == "grad":
        st["gF"], st["ng"] = _weights_of_force(dim), plan.n_ghost
        st["bcv"] = [torch.nn.functional.pad(b, (0, cap - plan.n_ghost)) for b in bcv]
        for t in st["u"] + st["bcv"]:
            t.requires_grad_()
    return st


def _room(case):
    """Room for the ghosts of a case's bodies, whatever the seed: what a program that places them over and over
    allocates once."""
    return int(1.6 * sum(_ghosts(case, n) for n in _sizes(case))) + 256


def _orbit(g, s):
    d = 0.4 * g.h[0]
    v, w = (0.8 * d, 0.48 * d, 0.36 * d), (-0.6 * d, 0.64 * d, 0.48 * d)
    steps = [(0, 0), (1, 0), (1, 1), (0, 1)]
    return [Shape(s.kind, tuple(c + i * a + j * b for c, a, b in zip(s.center, v, w)), s.r0) for i, j in steps]


def _weights_of_force(dim):
    return torch.tensor([1.0, 0.5, -0.25][:dim], dtype=F64, device="cuda")


def run(st):
    do = st["do"]
    if do == "plan":
        plan = gcr.Plan(st["grid"], st["shape"], st["scheme"])
        tags = plan.export(("tags",))["tags"]
        plan.fill(st["u"], st["kinds"], [b[:plan.n_ghost] for b in st["wall"]])
        val, grad, anchor = plan.surface(st["pts"][0], st["u"])
        return {"tags": tags, "u": st["u"], "val": val, "grad": grad, "anchor": anchor}
    if do == "move":  # two plans in turn, each from two positions back; at the end both are where they were
        out = []
        for k in (2, 3, 0, 1):
            before, plan = st["plans"][(k + 1) % 2], st["plans"][k % 2]
            plan.update(st["orbit"][k])
            fresh, counts = before.fresh_cells(plan, cap=st["fresh"])
            plan.fill([st["u"][k]], st["kinds"], [b[:plan.n_ghost] for b in st["wall"]])
            out.append({"counts": counts, "fresh": torch.where(st["at"] < counts[0], fresh, -1)})
        return {"u": st["u"], "moves": out}
    if do == "build":
        B = gcr.Batch(spec=st["spec"])
        counts, dim = np.array(B.counts()), st["grid"].dim
        ng = int(counts.sum())
        B.foot_points(out=(st["S"][:dim * ng].view(dim, ng), st["n"][:dim * ng].view(dim, ng)))
        return {"S": st["S"], "n": st["n"], "counts": counts}
    if do == "forward":
        st["batch"].forward(args=st["args"])
        return {"u": st["u"], "F": st["F"], "val": st["val"], "grad": st["grad"]}
    x, nrm, w = st["pts"]
    if do == "step":
        st["plan"].fill(st["u"], st["kinds"], st["bcv"], st["bct"])
        val, grad, anchor = st["plan"].surface(x, st["u"])
        F = st["plan"].forces(x, nrm, w, st["u"][-1], st["u"][:-1], st["mu"])
        return {"u": st["u"], "val": val, "grad": grad, "anchor": anchor, "F": F}
    u = gcr_autograd.ghost_fill(st["plan"], st["u"], st["kinds"], [b[:st["ng"]] for b in st["bcv"]], st["bct"])
    F = gcr_autograd.forces(st["plan"], x, nrm, w, u[-1], u[:-1], st["mu"])
    g = torch.autograd.grad(F, st["u"] + st["bcv"], st["gF"])
    return {"u": [t.detach() for t in u], "F": F.detach(), "du": list(g[:len(u)]), "db": list(g[len(u):])}


# ----------------------------------------------------------------------------------------------------------
# the same in plain torch
# ----------------------------------------------------------------------------------------------------------

def _airfoil_half(t, x):
    return 5 * t * (0.2969 * x.sqrt() - 0.1260 * x - 0.3516 * x ** 2 + 0.2843 * x ** 3 - 0.1036 * x ** 4)


def _airfoil_curve(s, a):
    """The contour of a unit chord at x = a^2 (a > 0 the upper side), its first and second derivative by a."""
    sg, t = torch.where(a < 0, -1.0, 1.0).to(F64), 5 * s.thick
    b = (0.1260, 0.3516, -0.2843, 0.1036)
    y = t * (0.2969 * a - sg * sum(c * a ** (2 * k + 2) for k, c in enumerate(b)))
    y1 = t * (0.2969 - sg * sum((2 * k + 2) * c * a ** (2 * k + 1) for k, c in enumerate(b)))
    y2 = -t * sg * sum((2 * k + 2) * (2 * k + 1) * c * a ** (2 * k) for k, c in enumerate(b))
    return torch.stack([a * a, y]), torch.stack([2 * a, y1]), torch.stack([torch.full_like(a, 2.0), y2])


def _airfoil_world(s, b):
    ca, sa = math.cos(s.incidence), math.sin(s.incidence)
    return torch.stack([ca * b[0] + sa * b[1], -sa * b[0] + ca * b[1]])


def _airfoil_body(s, v):
    ca, sa = math.cos(s.incidence), math.sin(s.incidence)
    return torch.stack([ca * v[0] - sa * v[1], sa * v[0] + ca * v[1]])


def _solid(g, s):
    """Whether each cell's centre lies in the body, flat."""
    v = [x - c for x, c in zip(g.mesh(), s.center)]
    if s.kind == gcr.AIRFOIL:
        b = _airfoil_body(s, torch.stack(torch.broadcast_tensors(*v)).reshape(2, -1))
        return (b[0] >= 0) & (b[0] <= 1) & (b[1].abs() <= _airfoil_half(s.thick, b[0].clamp(0, 1)))
    rho = sum(x * x for x in v).sqrt().reshape(-1)
    if s.kind == gcr.SPHERE:
        return s.r0 - rho >= 0
    if s.kind == gcr.STAR2D:
        th = torch.atan2(v[1].expand(g.n[1], g.n[0]), v[0].expand(g.n[1], g.n[0])).reshape(-1)
        return _star_radius(s, th)[0] - rho >= 0
    much = float(np.abs(s.coef).sum())
    solid = rho < s.r0 * (1 - much)
    near = torch.nonzero((rho >= s.r0 * (1 - much)) & (rho <= s.r0 * (1 + much))).reshape(-1)
    w = torch.stack([x.expand(g.n[2], g.n[1], g.n[0]).reshape(-1)[near] for x in v])
    solid[near] = _sh_radius(s, w) - rho[near] >= 0
    return solid


def _project(s, x, solid):
    """psi and the unit outward normal at the closest point of the boundary, for points x [dim][m]."""
    c = torch.tensor(s.center[:x.shape[0]], dtype=F64, device="cuda")[:, None]
    v = x - c
    rho = (v * v).sum(0).sqrt()
    if s.kind == gcr.SPHERE:
        return s.r0 - rho, v / rho
    if s.kind == gcr.SHSTAR:
        w = v / rho
        for _ in range(80):  # Gauss-Newton on the sphere of directions
            r, gr = _sh_grad(s, w)
            i = w.abs().argmin(0)
            e = torch.zeros_like(w).scatter_(0, i[None], 1.0)
            t1 = e - (e * w).sum(0) * w
            t1 = t1 / (t1 * t1).sum(0).sqrt()
            t2 = torch.linalg.cross(w, t1, dim=0)
            J1, J2 = (gr * t1).sum(0) * w + r * t1, (gr * t2).sum(0) * w + r * t2
            R = r * w - v
            a11, a12, a22 = (J1 * J1).sum(0), (J1 * J2).sum(0), (J2 * J2).sum(0)
            b1, b2 = -(J1 * R).sum(0), -(J2 * R).sum(0)
            det = a11 * a22 - a12 * a12
            w = w + (b1 * a22 - b2 * a12) / det * t1 + (a11 * b2 - a12 * b1) / det * t2
            w = w / (w * w).sum(0).sqrt()
        r, gr = _sh_grad(s, w)
        S, n = r * w, w - gr / r
    elif s.kind == gcr.STAR2D:
        th = torch.atan2(v[1], v[0])
        for k in range(61):
            r, r1, r2 = _star_radius(s, th)
            ct, st = torch.cos(th), torch.sin(th)
            S, D = torch.stack([r * ct, r * st]), torch.stack([r1 * ct - r * st, r1 * st + r * ct])
            E = torch.stack([(r2 - r) * ct - 2 * r1 * st, (r2 - r) * st + 2 * r1 * ct])
            g1, g0 = ((S - v) * D).sum(0), (D * D).sum(0)
            g2 = g0 + ((S - v) * E).sum(0)
            if k < 60:
                th = th - g1 / torch.where(g2 > 0, g2, g0)
        n = torch.stack([D[1], -D[0]])
    else:
        b = _airfoil_body(s, v)
        best = None
        for sign in (1.0, -1.0):
            a = sign * b[0].clamp(0, 1).sqrt()
            a = torch.where(a == 0, sign * 1e-3, a)
            for _ in range(60):
                X, D, E = _airfoil_curve(s, a)
                g1, g0 = ((X - b) * D).sum(0), (D * D).sum(0)
                g2 = g0 + ((X - b) * E).sum(0)
                a = a - g1 / torch.where(g2 > 0, g2, g0)
                a = a.clamp(0, 1) if sign > 0 else a.clamp(-1, 0)
            X, D, _ = _airfoil_curve(s, a)
            d2 = ((X - b) ** 2).sum(0)
            corner = torch.where(solid, -1.0, 1.0) * (b - X)
            nb = torch.where(a.abs() >= 1, corner, torch.stack([-D[1], D[0]]))
            best = (d2, X, nb) if best is None else tuple(torch.where(d2 < best[0], p, q)
                                                          for p, q in zip((d2, X, nb), best))
        S, n = _airfoil_world(s, best[1]), _airfoil_world(s, best[2])
    psi = ((v - S) ** 2).sum(0).sqrt()
    return torch.where(solid, psi, -psi), n / (n * n).sum(0).sqrt()


class Reference:
    """The plan of one body: ghosts in canonical order, their geometry and stencils."""

    def __init__(self, g, s, scheme):
        self.g, dim = g, g.dim
        self.dim = dim
        dims = [g.n[a] for a in reversed(range(dim))]
        self.stride = [1, g.n[0], g.n[0] * g.n[1]][:dim]
        base, second = scheme & 3, bool(scheme & LAYER2)
        solid = _solid(g, s).view(dims)
        face = torch.zeros_like(solid)
        for a in range(dim):
            m = solid.shape[a]
            diff = solid.narrow(a, 0, m - 1) != solid.narrow(a, 1, m - 1)
            face.narrow(a, 0, m - 1).logical_or_(diff)
            face.narrow(a, 1, m - 1).logical_or_(diff)
        solid, face = solid.reshape(-1), face.reshape(-1)
        cell = torch.nonzero(solid | face if second else face).reshape(-1)
        if second:  # round bodies: solid cells within a few cells of the boundary
            x = self._centre(self._split(cell))
            wide = max(float(g.widths(a).max()) for a in range(dim))
            c = torch.tensor(s.center[:dim], dtype=F64, device="cuda")[:, None]
            cell = cell[face[cell] | (s.r0 - ((x - c) ** 2).sum(0).sqrt() <= 2 * wide)]
        ijk = self._split(cell)
        x, sol = self._centre(ijk), solid[cell]
        psi, n = _project(s, x, sol)
        w = torch.stack([g.widths(a)[ijk[a]] for a in range(dim)])
        dn = 1.0 / ((n / w) ** 2).sum(0).sqrt()
        own = face[cell] & (torch.where(sol, psi <= dn / 2, -psi < dn / 2) if base == HGC else sol)
        extra = sol & ~own & (psi <= 1.5 * dn) if second else torch.zeros_like(sol)
        keep = own | extra
        cell, ijk, n, psi, w, x, extra = cell[keep], ijk[:, keep], n[:, keep], psi[keep], w[:, keep], x[:, keep], extra[keep]
        delta = psi * n
        e = torch.where(n >= 0, 1, -1)
        r = torch.where((base == CGC_ES) | extra, (2 * delta.abs() / w).ceil().clamp(min=1).long(), 1)
        far = ijk + e * r
        X = torch.empty_like(delta)
        corner = []
        for a in range(dim):
            cs = g.centres(a)
            ok = (far[a] >= 0) & (far[a] < g.n[a])
            X[a] = torch.where(ok, cs[far[a].clamp(0, g.n[a] - 1)] - cs[ijk[a]], (e * r)[a] * w[a])
        for bits in itertools.product((0, 1), repeat=dim):
            if any(bits):
                skip = torch.zeros_like(extra)
                for a in range(dim):
                    if bits[a]:
                        skip |= n[a] == 0
                at = cell + sum(bits[a] * (e * r)[a] * self.stride[a] for a in range(dim))
                corner.append(torch.where(skip, cell, at))
        corner = torch.stack(corner)
        ng = cell.numel()
        pos = torch.searchsorted(cell, corner).clamp(max=ng - 1)
        dep = torch.where((cell[pos] == corner) & (corner != cell), pos, -1)
        level, unit = self._levels(dep, ng)
        order = torch.sort(level, stable=True).indices
        self.cell, self.level, self.unit = cell[order], level[order], unit[order]
        self.n, self.psi, self.delta, self.X, self.x = n[:, order], psi[order], delta[:, order], X[:, order], x[:, order]
        self.corner, self.ijk, self.S = corner[:, order], ijk[:, order], (x + delta)[:, order]

    def _split(self, c):
        n = self.g.n
        return torch.stack([c % n[0], c // n[0] % n[1], c // (n[0] * n[1])][:self.dim])

    def _centre(self, ijk):
        return torch.stack([self.g.centres(a)[ijk[a]] for a in range(self.dim)])

    @staticmethod
    def _levels(dep, ng):
        """Level of every ghost, and of ghosts that read each other in a circle the first of them (else -1)."""
        level = torch.zeros(ng + 1, dtype=torch.long, device="cuda")
        level[ng] = 1  # stands for "no ghost"
        unit = torch.full((ng,), -1, dtype=torch.long, device="cuda")
        d = torch.where(dep < 0, ng, dep)
        k = 0
        while True:
            k += 1
            ready = (level[:ng] == 0) & (level[d] > 0).all(0)
            if not bool(ready.any()):
                break
            level[:ng][ready] = k
        left = torch.nonzero(level[:ng] == 0).reshape(-1)
        if left.numel():
            m = left.numel()
            where = torch.full((ng + 1,), m, dtype=torch.long, device="cuda")
            where[left] = torch.arange(m, device="cuda")
            A = torch.zeros((m, m + 1), device="cuda")
            A[torch.arange(m, device="cuda").expand(d.shape[0], m), where[d[:, left]]] = 1
            reach = torch.clamp(A[:, :m] + torch.eye(m, device="cuda"), max=1)
            for _ in range(max(1, math.ceil(math.log2(m + 1)))):
                reach = torch.clamp(reach @ reach, max=1)
            first = (reach * reach.T).argmax(1)
            together = torch.bincount(first, minlength=m)[first] > 1
            unit[left] = torch.where(together, left[first], -1)
            owner = torch.cat([first, torch.tensor([m], device="cuda")])
            dl = where[d[:, left]]
            outer = torch.where(owner[dl] == first, 0, 1)
            lev = torch.ones(m + 1, dtype=torch.long, device="cuda")
            known = torch.where(dl == m, level[d[:, left]] * (d[:, left] != ng), 0)
            while True:
                need = 1 + torch.maximum(known, torch.where(dl == m, 0, lev[dl] * outer)).max(0).values
                group = torch.zeros(m, dtype=torch.long, device="cuda").scatter_reduce(0, first, need, "amax")
                if bool((group[first] == lev[:m]).all()):
                    break
                lev[:m] = group[first]
            level[left] = lev[:m]
        return level[:ng], unit

    def basis(self, at, rel, grad):
        """Values [corner][m] of the stencils' Lagrange functions at points rel [dim][m], or their gradients
        [dim][corner][m]; the ghost itself is the first corner."""
        X = self.X[:, at]
        a = rel / X
        one = [[(1 - a[i], -1 / X[i]), (a[i], 1 / X[i])] for i in range(self.dim)]
        bits = list(itertools.product((0, 1), repeat=self.dim))
        if not grad:
            return torch.stack([math.prod(one[i][b[i]][0] for i in range(self.dim)) for b in bits])
        return torch.stack([torch.stack([math.prod(one[i][b[i]][int(i == j)] for i in range(self.dim)) for b in bits])
                            for j in range(self.dim)])

    def fill(self, u, bcv, bct):
        """The filled fields [nf][cells], differentiable."""
        every = torch.arange(self.cell.numel(), device="cuda")
        L, G = self.basis(every, self.delta, False), (self.basis(every, self.delta, True) * self.n[:, None]).sum(0)
        W = torch.stack([torch.where(t.bool(), G, L) for t in bct])  # [nf][corner][ng]
        ws, W = 1 / W[:, 0], -W[:, 1:] / W[:, :1]
        b = torch.stack(bcv) * ws
        for k in range(1, int(self.level.max()) + 1):
            at = torch.nonzero(self.level == k).reshape(-1)
            alone = at[self.unit[at] < 0]
            new = (W[:, :, alone] * u[:, self.corner[:, alone]]).sum(1) + b[:, alone]
            cells = [self.cell[alone]]
            news = [new]
            for q in torch.unique(self.unit[at]).tolist():
                if q >= 0:
                    mem = at[self.unit[at] == q]
                    inside = self.corner[:, mem][:, :, None] == self.cell[mem]  # [corner][member][member]
                    M = torch.eye(mem.numel(), dtype=F64, device="cuda") - (W[:, :, mem, None] * inside).sum(1)
                    known = torch.where(inside.any(2), 0.0, u[:, self.corner[:, mem]])
                    news.append(torch.linalg.solve(M, (W[:, :, mem] * known).sum(1) + b[:, mem]))
                    cells.append(self.cell[mem])
            new, c = torch.cat(news, 1), torch.cat(cells)
            if u.requires_grad or new.requires_grad:
                u = u.index_put((torch.arange(u.shape[0], device="cuda")[:, None], c[None]), new)
            else:
                u[:, c] = new
        return u

    def surface(self, x, u):
        """Values [nf][nq] and gradients [nf][dim][nq] at points x, each from its nearest ghost's stencil."""
        g, got = self.g, []
        for part in x.split(128, 1):
            q = []
            for a in range(self.dim):
                if g.faces is not None:
                    q.append(torch.bucketize(part[a], torch.tensor(g.faces[a], dtype=F64, device="cuda"), right=True) - 1)
                else:
                    q.append(((part[a] - g.lo[a]) / g.h[a]).floor().long())
            near = torch.ones((part.shape[1], self.cell.numel()), dtype=torch.bool, device="cuda")
            d2 = torch.zeros(near.shape, dtype=F64, device="cuda")
            for a in range(self.dim):
                near &= (q[a][:, None] - self.ijk[a]).abs() <= 2
                d2 += (part[a][:, None] - self.S[a]) ** 2
            got.append(torch.where(near, d2, math.inf).argmin(1))
        at = torch.cat(got)
        rel = x - self.x[:, at]
        box = torch.cat([self.cell[at][None], self.corner[:, at]])
        v = u[:, box]  # [nf][corner][nq]
        return (self.basis(at, rel, False) * v).sum(1), (self.basis(at, rel, True)[None] * v[:, None]).sum(2)


def _force(val, grad, n, w, mu):
    """The force from the last field's values and the other fields' gradients."""
    J = grad[:-1]
    t = -val[-1] * n + mu * ((J + J.transpose(0, 1)) * n).sum(1)
    return (t * w).sum(1)


def _padded(t, room):
    return torch.nn.functional.pad(t.reshape(-1), (0, room - t.numel()))


def exact(case, seed):
    do, scheme, room = case["do"], SCHEMES[case["scheme"]], _room(case)
    bodies = _bodies(case, seed)
    if do == "build":
        plans = [Reference(g, s, scheme) for g, s in bodies]
        dim = bodies[0][0].dim
        return {"S": _padded(torch.cat([p.S for p in plans], 1), dim * room),
                "n": _padded(torch.cat([p.n for p in plans], 1), dim * room), "counts": None}
    fields, beta = _fields(case, seed)
    kinds, mu = _kinds(case), 0.7
    flux = [torch.tensor(k == NEUMANN, device="cuda") for k in kinds]
    if do == "move":
        us = []
        for shape in _orbit(*bodies[0]):
            p = Reference(bodies[0][0], shape, scheme)
            u = fields[0].value(p.g.mesh()).reshape(1, -1)
            us.append(p.fill(u, [torch.full_like(p.psi, beta[0])], flux)[0])
        return {"u": us, "moves": None}
    got = {"u": [], "val": [], "grad": [], "F": []}
    for g, s in bodies:
        p = Reference(g, s, scheme)
        x, n, w = _surface_points(s, g.dim, case["nq"])
        u = torch.stack([f.value(g.mesh()).reshape(-1) for f in fields])
        if do == "plan":
            bcv, bct = [torch.full_like(p.psi, b) for b in beta], flux
        else:
            bcv, bct = _boundary(fields, kinds, s.center, beta, p.S, p.n)
        if do == "grad":
            for t in [u] + bcv:
                t.requires_grad_()
            full = p.fill(u, bcv, bct)
            val, grad = p.surface(x, full)
            F = _force(val, grad, n, w, mu)
            du, *db = torch.autograd.grad(F, [u] + bcv, _weights_of_force(g.dim))
            return {"u": list(full.detach()), "F": F.detach(), "du": list(du), "db": [_padded(b, room) for b in db]}
        u = p.fill(u, bcv, bct)
        val, grad = p.surface(x, u)
        for k, v in (("u", u), ("val", val), ("grad", grad)):
            got[k].append(v)
        if do != "plan":
            got["F"].append(_force(val, grad, n, w, mu))
    if do in ("plan", "step"):
        out = {"u": list(got["u"][0]), "val": got["val"][0], "grad": got["grad"][0], "anchor": None}
        out.update({"tags": None} if do == "plan" else {"F": got["F"][0]})
        return out
    F = torch.zeros((len(bodies), 3), dtype=F64, device="cuda")
    F[:, :bodies[0][0].dim] = torch.stack(got["F"])
    return {"u": torch.cat([v.reshape(-1) for v in got["u"]]), "F": F, "val": torch.cat(got["val"]),
            "grad": torch.cat(got["grad"])}
