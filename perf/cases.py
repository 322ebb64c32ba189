"""Timed cases of the extension library, with inputs, work counts and 64-bit results.

A case is one call (or one time step, or one burst of requests) as a user's
program makes it: the level-set function and the field are on the GPU, the
handle or the serving engine is kept for the life of the program, and the
extended field is what comes back.  Tolerances are tight (1e-10 to 1e-12), so
that a result is a property of the problem and not of the path the conjugate
gradients took to it.
"""
import math

import numpy as np
import torch

from paper_1704_08897_amd import bhx
from paper_1704_08897_amd.server import Request, Server, serve_stream

NEUMANN, PERIODIC, DIRICHLET = 0, 1, 2
DEV = "cuda:0"


def listed():
    N, P, D = NEUMANN, PERIODIC, DIRICHLET
    return [
        # the smallest call in use: one small field, where launches and waits count
        dict(name="circle_64", kind="solve", nx=64, ny=64, bcx=N, bcy=N, shape="disc",
             known="inside", tol=1e-10),
        # a field extended into an interior region on a power-of-two grid
        dict(name="star_inward_1024", kind="solve", nx=1024, ny=1024, bcx=N, bcy=N, shape="star",
             known="outside", tol=1e-12),
        # the largest plane grid, both axes periodic
        dict(name="star_periodic_2048", kind="solve", nx=2048, ny=2048, bcx=P, bcy=P,
             shape="star", known="outside", tol=1e-12),
        # an ordinary request of arbitrary (prime, odd) sides
        dict(name="request_1231x877", kind="solve", nx=1231, ny=877, bcx=N, bcy=P, shape="star",
             known="inside", tol=2e-12),
        # many separate known regions, periodic, sides without a fast transform
        dict(name="circles_450", kind="solve", nx=450, ny=450, bcx=P, bcy=P, shape="circles",
             known="inside", tol=1e-12),
        # a Dirichlet axis long enough for its own transform path, and a Neumann one
        dict(name="dirichlet_1100x600", kind="solve", nx=1100, ny=600, bcx=D, bcy=N, shape="star",
             known="inside", tol=2e-12),
        # the FP32 preconditioner inside FP64 defect correction
        dict(name="fp32_precond_300x256", kind="solve", nx=300, ny=256, bcx=N, bcy=N,
             shape="star", known="inside", tol=1e-12, precision=1, accurate=1),
        # one batched call over instances of mixed sizes and rules
        dict(name="batch_40", kind="batch", count=40, lo=64, hi=512, mix=4, tol=2e-12),
        # a burst of requests through the serving engine
        dict(name="serve_8", kind="serve", count=8, lo=128, hi=800, mix=5, tol=2e-12),
        # a time step: three fields known on one region, started from the last step's
        dict(name="fields_warm_512", kind="fields", nx=512, ny=512, bcx=N, bcy=N, shape="star",
             known="outside", count=3, tol=2e-12),
        # three dimensions: two balls in a periodic box
        dict(name="balls_128_3d", kind="solve3", nx=128, ny=128, nz=128, bcx=P, bcy=P, bcz=P,
             tol=2e-11),
        # the sparse direct route
        dict(name="direct_star_512", kind="solve", nx=512, ny=512, bcx=N, bcy=N, shape="star",
             known="outside", tol=1e-10, solver=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plane", "plane", "plane", "plane", "circles", "fp32", "batch", "serve",
                       "fields", "space", "direct"])
    rules = (NEUMANN, PERIODIC, DIRICHLET)
    if kind == "space":
        nx, ny, nz = (_log(rng, 24, 128) for _ in range(3))
        return dict(kind="solve3", nx=nx, ny=ny, nz=nz, bcx=rng.choice(rules),
                    bcy=rng.choice(rules), bcz=rng.choice(rules), tol=2e-11)
    if kind in ("batch", "serve"):
        count = rng.randint(6, 24) if kind == "batch" else rng.randint(4, 10)
        hi = rng.randint(256, 512) if kind == "batch" else rng.randint(300, 800)
        return dict(kind=kind, count=count, lo=64 if kind == "batch" else 128, hi=hi,
                    mix=rng.randrange(1 << 16), tol=2e-12)
    hi = {"plane": 1000, "circles": 450, "fp32": 300, "fields": 640, "direct": 300}[kind]
    nx = _log(rng, 64, hi)
    # sides within a factor of two of each other; every third draw a power of two
    ny = max(64, min(hi, int(nx * math.exp(rng.uniform(-0.7, 0.7)))))
    if rng.randrange(3) == 0:
        nx = 1 << int(round(math.log2(nx)))
        ny = 1 << int(round(math.log2(ny)))
    c = dict(kind="solve", nx=nx, ny=ny, bcx=rng.choice(rules), bcy=rng.choice(rules),
             shape="star", known=rng.choice(["inside", "outside"]), tol=2e-12)
    if kind == "circles":
        c.update(shape="circles", known="inside", bcx=PERIODIC, bcy=PERIODIC, tol=1e-12)
    elif kind == "fp32":
        c.update(tol=1e-12, precision=1, accurate=1)
    elif kind == "fields":
        c.update(kind="fields", count=rng.randint(2, 4))
    elif kind == "direct":
        c.update(bcx=NEUMANN, shape="front", known="inside", solver=1, tol=1e-10,
                 bcy=rng.choice((NEUMANN, PERIODIC)))
    return c


# ---------------------------------------------------------------------------
# Inputs: closed-form level sets and smooth fields, evaluated on the GPU
# ---------------------------------------------------------------------------

def _axis(n, half, rule):
    """Node coordinates on [-half, half]: cell-centred, or from the left end where periodic."""
    i = torch.arange(n, dtype=torch.float64, device=DEV)
    return -half + (i + (0.0 if rule == PERIODIC else 0.5)) * (2.0 * half / n)


def _plane(nx, ny, bcx, bcy):
    h = 2.0 / min(nx, ny)
    Y, X = torch.meshgrid(_axis(ny, ny * h / 2, bcy), _axis(nx, nx * h / 2, bcx), indexing="ij")
    return X, Y, h


def _level_set(c, X, Y, h, rng):
    """phi of one instance (negative on the known side)."""
    if c["shape"] == "disc":
        phi = torch.sqrt(X * X + Y * Y) - rng.uniform(0.45, 0.55)
    elif c["shape"] == "star":
        a, w = rng.uniform(0, 0.05, 8), rng.uniform(0, 2 * np.pi, 8)
        th, r = torch.atan2(Y, X), torch.ones_like(X)
        for k in range(8):
            r = r + float(a[k]) * torch.cos((k + 1) * th + float(w[k]))
        phi = torch.sqrt(X * X + Y * Y) - (0.5 if c["known"] == "inside" else 0.4) * r
    elif c["shape"] == "circles":
        # twelve circles in the periodic cell of side `L`
        phi = None
        Lx, Ly = X.shape[1] * h, X.shape[0] * h
        for cx, cy, r in zip(rng.uniform(0, Lx, 12), rng.uniform(0, Ly, 12),
                             rng.uniform(0.1, 0.3, 12)):
            dx, dy = X - float(cx), Y - float(cy)
            dx, dy = dx - Lx * torch.round(dx / Lx), dy - Ly * torch.round(dy / Ly)
            d = torch.sqrt(dx * dx + dy * dy) - float(r)
            phi = d if phi is None else torch.minimum(phi, d)
    else:
        # a front across the channel, known to its left
        a, w = rng.uniform(-0.05, 0.05, 10), rng.uniform(0, 2 * np.pi, 10)
        Ly = X.shape[0] * h
        phi = X.clone()
        for k in range(10):
            phi = phi - float(a[k]) * torch.sin(2 * np.pi * (k + 1) / Ly * Y + float(w[k]))
    return (phi if c["known"] == "inside" else -phi).contiguous()


def _modes(X, Y, h, rng):
    """A smooth field: eight Fourier modes of the box."""
    F = torch.zeros_like(X)
    Lx, Ly = X.shape[1] * h, X.shape[0] * h
    for _ in range(8):
        kx, ky = (int(k) for k in rng.randint(-3, 4, 2))
        a, w = float(rng.normal()), float(rng.uniform(0, 2 * np.pi))
        F += a * torch.cos(2 * np.pi * (kx / Lx * X + ky / Ly * Y) + w)
    return F


def _instance(c, rng):
    X, Y, h = _plane(c["nx"], c["ny"], c["bcx"], c["bcy"])
    return {"phi": _level_set(c, X, Y, h, rng), "F": _modes(X, Y, h, rng), "h": h,
            "rules": (c["bcx"], c["bcy"])}


def _mix(c):
    """Sizes and rules of a batch or a burst: the case's own, whatever the seed."""
    g = np.random.RandomState(c["mix"])
    out = []
    for _ in range(c["count"]):
        nx, ny = (int(round(math.exp(g.uniform(math.log(c["lo"]), math.log(c["hi"])))))
                  for _ in range(2))
        bcx, bcy = (int(b) for b in g.randint(0, 2, 2))
        known = "inside" if g.randint(0, 2) else "outside"
        if c["kind"] == "serve":
            ny, bcy, known = nx, bcx, "inside"       # square, one rule, as requests come
        else:
            ny = max(c["lo"], min(ny, 2 * nx))       # elongation as boxes around one region have
            nx = min(nx, 2 * ny)
        out.append(dict(nx=nx, ny=ny, bcx=bcx, bcy=bcy, shape="star", known=known))
    return out


def _instances(c, seed):
    rng = np.random.RandomState(seed % (1 << 32))
    if c["kind"] in ("batch", "serve"):
        return [_instance(m, rng) for m in _mix(c)]
    if c["kind"] == "fields":
        X, Y, h = _plane(c["nx"], c["ny"], c["bcx"], c["bcy"])
        phi = _level_set(c, X, Y, h, rng)
        out = []
        for _ in range(c["count"]):
            F, dF = _modes(X, Y, h, rng), _modes(X, Y, h, rng)
            out.append({"phi": phi, "old": F, "F": F + 0.01 * dF, "h": h,
                        "rules": (c["bcx"], c["bcy"])})
        return out
    if c["kind"] == "solve3":
        n, rules = (c["nx"], c["ny"], c["nz"]), (c["bcx"], c["bcy"], c["bcz"])
        h = 2.0 / max(n)
        Z, Y, X = torch.meshgrid(*(_axis(m, m * h / 2, b) for m, b in zip(n[::-1], rules[::-1])),
                                 indexing="ij")
        s, r, a = rng.uniform(0.2, 0.3), rng.uniform(0.25, 0.35, 2), rng.normal(size=4)
        box = [m * h / 2 for m in n]
        phi = torch.minimum(
            torch.sqrt((X - s * box[0]) ** 2 + Y ** 2 + Z ** 2) - float(r[0]) * min(box),
            torch.sqrt((X + s * box[0]) ** 2 + Y ** 2 + Z ** 2) - float(r[1]) * min(box))
        F = (float(a[0]) * torch.cos(2 * X) * torch.sin(2 * Y) + float(a[1]) * torch.sin(3 * Z)
             + float(a[2]) * X * Z + float(a[3]) * torch.cos(Y) * Z)
        return [{"phi": phi.contiguous(), "F": F.contiguous(), "h": h, "rules": rules}]
    return [_instance(c, rng)]


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

_kept = {}


def _handle():
    """The handle that a program keeps for all its calls."""
    if "handle" not in _kept:
        _kept["handle"] = bhx.Handle(0)
    return _kept["handle"]


def _server(tol):
    """The serving engine that a program keeps for all its requests."""
    if "server" not in _kept:
        _kept["server"] = Server(0, hbm_budget=16 << 30, max_slots=32)
    return _kept["server"]


def _bc(rules):
    return bhx.BC(*rules) if len(rules) == 2 else bhx.BC3(*rules)


def prepare(case, seed):
    c = dict(case)
    ins = _instances(c, seed)
    st = {"case": c, "ins": ins, "out": [i["F"].clone() for i in ins],
          "opts": bhx.default_opts(**{k: c[k] for k in ("precision", "accurate", "solver")
                                      if k in c})}
    if c["kind"] == "serve":
        st["server"] = _server(c["tol"])
    else:
        st["handle"] = _handle()
    if c["kind"] == "fields":
        # the extension of the step before, which the program holds
        st["opts"].warm_start = 1
        for i in ins:
            bhx.extend_ex(st["handle"], i["phi"], i["old"], h=i["h"], bc=_bc(i["rules"]), tol=1e-8)
            i["F"] = torch.where(i["phi"] < 0, i["F"], i["old"])
    return st


def _ok(status):
    if status != bhx.OK:
        raise bhx.BhxError(status)


def run(st):
    c, ins, out = st["case"], st["ins"], st["out"]
    if c["kind"] == "serve":
        reqs = [Request(i["phi"], F, _bc(i["rules"]), i["h"], c["tol"]) for i, F in zip(ins, out)]
        for r in serve_stream(st["server"], reqs):
            _ok(r.stats["status"])
    elif c["kind"] == "batch":
        _ok(bhx.extend_batched(st["handle"], [i["phi"] for i in ins], out, [i["h"] for i in ins],
                               [_bc(i["rules"]) for i in ins], [c["tol"]] * len(ins),
                               opts=st["opts"])[0])
    elif c["kind"] == "fields":
        for i, F in zip(ins, out):
            F.copy_(i["F"])              # the step's known values, the last step's extension
        i = ins[0]
        _ok(bhx.extend_fields(st["handle"], i["phi"], out, h=i["h"], bc=_bc(i["rules"]),
                              tol=c["tol"], opts=st["opts"])[0])
    else:
        f = bhx.extend3d if c["kind"] == "solve3" else bhx.extend_ex
        i = ins[0]
        _ok(f(st["handle"], i["phi"], out[0], h=i["h"], bc=_bc(i["rules"]), tol=c["tol"],
              opts=st["opts"])[0])
    return out


def work(case):
    """phi and the field in, the field out; and an iteration count that grows with the side (about
    half of it), each iteration a stencil, the vector updates and two fast transforms per axis."""
    c = dict(case)
    if c["kind"] in ("batch", "serve"):
        sizes = [(m["nx"], m["ny"]) for m in _mix(c)]
    elif c["kind"] == "fields":
        sizes = [(c["nx"], c["ny"])] * c["count"]
    else:
        sizes = [tuple(c[k] for k in ("nx", "ny", "nz") if k in c)]
    total = {"bytes": 0.0, "flops": 0.0}
    for n in sizes:
        nodes = float(np.prod(n))
        total["bytes"] += 24.0 * nodes
        total["flops"] += nodes * 0.5 * max(n) * (
            40.0 + sum(4 * 2.5 * math.log2(k) for k in n))
    return total


# ---------------------------------------------------------------------------
# The same extension in plain 64-bit arithmetic
# ---------------------------------------------------------------------------

def _lap(f, rules):
    """Sum over the axes (x last) of the negative second difference with the axis' rule."""
    out = 0
    for d, rule in enumerate(rules):
        g = f.swapaxes(0, f.ndim - 1 - d)
        t = 2 * g
        t[1:] -= g[:-1]
        t[:-1] -= g[1:]
        if rule == NEUMANN:
            t[0] -= g[0]
            t[-1] -= g[-1]
        elif rule == PERIODIC:
            t[0] -= g[-1]
            t[-1] -= g[0]
        out = out + t.swapaxes(0, f.ndim - 1 - d)
    return out


def _basis(n, rule):
    """Orthonormal eigenvectors (rows) and eigenvalues of the second difference."""
    k = torch.arange(n, dtype=torch.float64, device=DEV)[:, None]
    i = torch.arange(n, dtype=torch.float64, device=DEV)[None, :]
    if rule == NEUMANN:
        q, lam = torch.cos(np.pi * torch.remainder(k * (2 * i + 1), 4 * n) / (2 * n)), k / (2 * n)
    elif rule == PERIODIC:
        a = 2 * np.pi * torch.remainder(k * i, n) / n
        q, lam = torch.cos(a) + torch.sin(a), k / n
    else:
        q = torch.sin(np.pi * torch.remainder((k + 1) * (i + 1), 2 * n + 2) / (n + 1))
        lam = (k + 1) / (2 * n + 2)
    return q / q.norm(dim=1, keepdim=True), 4 * torch.sin(np.pi * lam[:, 0]) ** 2


def _along(q, v, axis):
    """Product of matrix q with v along an axis (0: the first)."""
    w = v.swapaxes(0, axis)
    return (q @ w.reshape(w.shape[0], -1)).reshape(w.shape).swapaxes(0, axis)


def _extend64(ins):
    """Preconditioned conjugate gradients with corrections from a longer-precision residual."""
    rules, F = ins["rules"], ins["F"].clone()
    U = ~(ins["phi"] < 0)
    if not bool(U.any()):
        return F
    m = U.double()
    dims = range(F.ndim)
    q = [_basis(F.shape[F.ndim - 1 - d], rules[d]) for d in dims]
    lam = sum(q[d][1].reshape([-1 if a == F.ndim - 1 - d else 1 for a in dims]) for d in dims)
    w = torch.where(lam > 1e-12, 1.0 / lam.clamp_min(1e-12) ** 2, torch.zeros_like(lam))

    def precondition(r):
        for d in dims:
            r = _along(q[d][0], r, F.ndim - 1 - d)
        r = r * w
        for d in dims:
            r = _along(q[d][0].T.contiguous(), r, F.ndim - 1 - d)
        return r * m

    def residual(f):
        g = f.cpu().numpy().astype(np.longdouble)
        r = -_lap(_lap(g, rules), rules)
        return torch.from_numpy(r.astype(np.float64)).to(DEV) * m

    F = torch.where(U, torch.zeros_like(F), F)
    first = None
    for _ in range(5):
        r = residual(F)
        size = float(r.norm())
        first = size if first is None else first
        if size <= 1e-15 * first:
            break
        x, p, rz = torch.zeros_like(r), None, None
        for it in range(40 * max(F.shape)):
            z = precondition(r)
            new = (r * z).sum()
            p = z if p is None else z + (new / rz) * p
            rz = new
            ap = _lap(_lap(p, rules), rules) * m
            a = rz / (p * ap).sum()
            x += a * p
            r = r - a * ap
            if it % 8 == 7 and float(r.norm()) <= 1e-9 * size:
                break
        F = F + x * m
    return F


def exact(case, seed):
    c = dict(case)
    ins = _instances(c, seed)
    # three corrections of up to three iterations per node of the longer side
    cost = sum(9 * max(i["F"].shape) * (3e-4 + i["F"].numel() * sum(i["F"].shape) * 2e-13)
               for i in ins)
    if cost > 20:
        return None
    return [_extend64(i) for i in ins]
