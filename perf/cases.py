"""The workloads by which the speed of the projection library is judged.

Every case is a call that a flow solver makes: a whole projection step, a
pressure solve on fixed coefficients, a differentiable solve with its backward
pass, an implicit viscous step or a projection around solids.  `prepare` builds
what such a program holds before the call (fields on the GPU, the solver
context), `run` makes the call, `exact` solves the same system in FP64 with
plain torch (Jacobi-preconditioned conjugate gradients on the face-wise
operator) and `work` counts the bytes and operations no method can avoid.

The fields follow the five seeded configurations of workloads.py (a drop, gas
bubbles in liquid, a wavy layer with droplets, a jet), drawn on the GPU with
volume fractions from the signed distance to the interface, u* uniform in
[-1, 1].
"""
import math
import random

import torch

from paper_2012_11744_amd import solver as S

DT = 1e-3
DEVICE = "cuda"


def _case(name, kind, n, bc, geom, ratio, prec, tol=1e-8, cycle="v"):
    c = {"kind": kind, "nx": n[0], "ny": n[1], "nz": n[2], "bc": bc, "geom": geom,
         "ratio": float(ratio), "prec": prec, "tol": float(tol), "cycle": cycle}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a small periodic box in full FP64: kernel launches and host waits are the cost
        _case("step-32-fp64", "step", (32, 32, 32), "ppp", "drop", 10, "fp64", 1e-10),
        # a short channel whose sides are no powers of two (coarsest level 18 x 10 x 4)
        _case("step-144x80x32", "step", (144, 80, 32), "pww", "drops", 1000, "fp32"),
        # the same step as four library calls, on a ragged box
        _case("calls-96x80x112", "calls", (96, 80, 112), "wpw", "drops", 100, "fp32", 1e-10),
        # training through the solve: forward and backward at 64^3, density ratio 100
        _case("grad-64", "grad", (64, 64, 64), "ppp", "drop", 100, "fp32"),
        # implicit viscous step of the three velocity components, started from the old velocity
        _case("viscous-160x128x96", "viscous", (160, 128, 96), "pwp", "drops", 100, "fp32", 1e-10),
        # projection around solids: closed links, excluded cells, full FP64
        _case("solids-96", "solids", (96, 96, 96), "pww", "drops", 10, "fp64", 1e-10),
        # 20 gas bubbles in liquid, density ratio 1000, walled 128^3 box: mixed and full FP64
        _case("step-128-bubbles", "step", (128, 128, 128), "www", "bubbles", 1000, "fp32"),
        _case("solve-128-bubbles-fp64", "solve", (128, 128, 128), "www", "bubbles", 1000, "fp64"),
        # wavy liquid layer with 200 droplets at 256^3, density ratio 833: every precision
        _case("step-256-layer", "step", (256, 256, 256), "ppw", "layer", 1000 / 1.2, "fp32"),
        _case("step-256-layer-fp16", "step", (256, 256, 256), "ppw", "layer", 1000 / 1.2, "fp16"),
        _case("solve-256-layer-fp64", "solve", (256, 256, 256), "ppw", "layer", 1000 / 1.2, "fp64"),
        # the largest: forward and backward around a liquid jet in a walled 512^3 box
        _case("grad-512-jet", "grad", (512, 512, 512), "www", "jet", 800, "fp32"),
    ]


def draw(rng):
    """Boxes of 16^3 to 320^3 cells, of any shape that coarsens (m 2^k cells a side)."""
    target = math.exp(rng.uniform(math.log(16.0 ** 3), math.log(320.0 ** 3)))
    while True:
        k = rng.randint(1, 7)
        per = (target / 8.0 ** k) ** (1.0 / 3.0)
        m = [int(round(per * math.exp(rng.uniform(-0.45, 0.45)))) for _ in range(3)]
        if min(m) < 4 or max(m) > 20 or m[0] * m[1] * m[2] > 800:
            continue
        n = [v << k for v in m]
        if n[0] * n[1] * n[2] <= 330 ** 3 and max(n) <= 512:
            break
    bc = "".join(rng.choice("pw") for _ in range(3))
    kind = rng.choice(["step", "step", "calls", "solve", "solve", "grad", "viscous", "solids"])
    general = kind in ("viscous", "solids")
    geom = "drops" if general else rng.choice(["drop", "drops", "layer", "jet", "bubbles"])
    ratio = rng.choice([10, 100, 1000])
    if kind == "solids":
        ratio = 10
    prec = rng.choice(["fp32", "fp32", "fp64"]) if general else rng.choice(["fp32", "fp32", "fp64", "fp16"])
    tol = rng.choice([1e-8, 1e-8, 1e-10])
    cycle = rng.choice(["v", "v", "v", "f"]) if geom == "bubbles" else "v"
    return _case(None, kind, n, bc, geom, ratio, prec, tol, cycle)


# -- fields ---------------------------------------------------------------------

def _bc(case):
    return tuple(1 if b == "w" else 0 for b in case["bc"])


def _grid(case):
    n = (case["nx"], case["ny"], case["nz"])
    h = 1.0 / max(n)
    return n, h


def _axes(n, h):
    ax = [(torch.arange(v, dtype=torch.float64, device=DEVICE) + 0.5) * h for v in n]
    return ax[0].view(1, 1, -1), ax[1].view(1, -1, 1), ax[2].view(-1, 1, 1)


def _balls(dist, n, h, bc, centres, radii):
    """dist = min(dist, signed distance to each ball), near the ball only."""
    for c, r in zip(centres, radii):
        idx = []
        for m in range(3):
            lo = math.floor((c[m] - r) / h) - 2
            hi = math.floor((c[m] + r) / h) + 3
            if hi - lo >= n[m]:
                lo, hi = 0, n[m]
            i = torch.arange(lo, hi, device=DEVICE)
            idx.append(i % n[m] if not bc[m] else i[(i >= 0) & (i < n[m])])
        d = []
        for m in range(3):
            x = (idx[m].double() + 0.5) * h - c[m]
            if not bc[m]:
                x = x - n[m] * h * torch.round(x / (n[m] * h))
            d.append(x)
        phi = (d[0].view(1, 1, -1) ** 2 + d[1].view(1, -1, 1) ** 2
               + d[2].view(-1, 1, 1) ** 2).sqrt() - r
        at = (idx[2].view(-1, 1, 1), idx[1].view(1, -1, 1), idx[0].view(1, 1, -1))
        dist[at] = torch.minimum(dist[at], phi)


def _fraction(case, seed):
    """Volume fraction of the heavy phase, from the signed distance to the interface."""
    rng = random.Random(seed)
    n, h = _grid(case)
    bc = _bc(case)
    box = [v * h for v in n]
    size = min(box)
    shape = (n[2], n[1], n[0])
    x, y, z = _axes(n, h)
    geom = case["geom"]
    far = torch.full(shape, 1.0, dtype=torch.float64, device=DEVICE)

    def anywhere(lo, hi):
        return [(lo + (hi - lo) * rng.random()) * b for b in box]

    if geom == "drop":
        _balls(far, n, h, bc, [anywhere(0.4, 0.6)], [0.25 * size])
    elif geom == "drops":
        k = 8
        _balls(far, n, h, bc, [anywhere(0.0, 1.0) for _ in range(k)],
               [rng.uniform(0.08, 0.25) * size for _ in range(k)])
    elif geom == "bubbles":
        _balls(far, n, h, bc, [anywhere(0.15, 0.85) for _ in range(20)],
               [rng.uniform(0.05, 0.15) * size for _ in range(20)])
    elif geom == "layer":
        lip = math.sqrt(1.0 + (0.05 * 2.0 * math.pi / 0.25) ** 2)
        ph = rng.uniform(0.0, 2.0 * math.pi)
        surf = 0.5 + 0.05 * torch.sin(2.0 * math.pi * x / (0.25 * box[0]) + ph)
        far = ((z / box[2] - surf) * box[2] / lip).expand(shape).contiguous()
        centres = [anywhere(0.0, 1.0)[:2] + [(0.58 + 0.39 * rng.random()) * box[2]]
                   for _ in range(200)]
        _balls(far, n, h, bc, centres, [rng.uniform(0.01, 0.03) * size for _ in range(200)])
    elif geom == "jet":
        dy, dz = (y - 0.5 * box[1]) / size, (z - 0.5 * box[2]) / size
        th = torch.atan2(dz, dy)
        radius = torch.full((1, 1, 1), 0.1, dtype=torch.float64, device=DEVICE)
        for _ in range(5):
            k, q, ph = rng.randint(1, 8), rng.randint(0, 2), rng.uniform(0.0, 2.0 * math.pi)
            radius = radius + 0.01 * torch.cos(2.0 * math.pi * k * x / box[0] + q * th + ph)
        far = (((dy * dy + dz * dz).sqrt() - radius) * size).expand(shape).contiguous()
    frac = far.div_(-h).add_(0.5).clamp_(0.0, 1.0)
    return 1.0 - frac if geom == "bubbles" else frac


def _inputs(case, seed):
    """rho, u* (and the generator, for what else a case draws)."""
    n, h = _grid(case)
    rho_g = 1.2 if case["geom"] == "layer" else 1.0
    rho = _fraction(case, seed).mul_(rho_g * (case["ratio"] - 1.0)).add_(rho_g)
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    us = []
    for m in range(3):
        u = torch.rand(rho.shape, generator=gen, device=DEVICE, dtype=torch.float64)
        u.mul_(2.0).sub_(1.0)
        if m == 2 and case["geom"] == "bubbles":
            u.sub_(9.81 * DT)
        if _bc(case)[m]:
            u.select(2 - m, 0).zero_()
        us.append(u)
    return rho, us, gen


def _solid(case, gen, shape):
    """A solid post through the box and a block on its floor, placed by the seed."""
    nz, ny, nx = shape
    at = torch.rand(2, generator=gen, device=DEVICE).cpu().tolist()
    solid = torch.zeros(shape, dtype=torch.bool, device=DEVICE)
    i, j = int(at[0] * nx * 0.6), int((0.1 + 0.5 * at[1]) * ny)
    solid[:, j:j + max(2, ny // 6), i:i + max(2, nx // 6)] = True
    solid[:max(1, nz // 8), : max(2, ny // 3), max(1, nx // 4):max(3, nx // 2)] = True
    return solid


def _general(case, seed):
    """Coefficients, diagonal term and right-hand sides of the general operator."""
    rho, us, gen = _inputs(case, seed)
    n, h = _grid(case)
    if case["kind"] == "viscous":
        beta = tuple(torch.ones_like(rho) for _ in range(3))
        mu = rho * 1e-2                       # tau mu: the heavy phase is the more viscous
        sigma = 1.0 / (DT * mu)
        return rho, us, beta, sigma
    beta = S.face_coeffs(rho, h, _bc(case))
    solid = _solid(case, gen, rho.shape)
    for m in range(3):
        beta[m][solid | solid.roll(1, 2 - m)] = 0.0
    return rho, us, beta, None


def _solver(case, beta, **kw):
    return S.Solver(beta, _grid(case)[1], _bc(case), precision=case["prec"], cycle=case["cycle"],
                    **kw)


def prepare(case, seed):
    n, h = _grid(case)
    kind = case["kind"]
    st = {"kind": kind, "tol": case["tol"]}
    if kind in ("viscous", "solids"):
        rho, us, beta, sigma = _general(case, seed)
        st["us"] = us
        st["solver"] = _solver(case, beta, sigma=sigma, general=True,
                               warm_start=kind == "viscous")
        if kind == "viscous":
            st["rhs"] = [-sigma * u for u in us]
        st["out"] = [torch.empty_like(rho) for _ in range(3)]
        st["p"], st["b"] = torch.empty_like(rho), torch.empty_like(rho)
        return st
    rho, us, gen = _inputs(case, seed)
    beta = S.face_coeffs(rho, h, _bc(case))
    st["solver"] = _solver(case, beta)
    if kind in ("step", "calls"):
        st["rho"], st["us"] = rho, us
        st["p"], st["b"] = torch.empty_like(rho), torch.empty_like(rho)
        st["out"] = [torch.empty_like(rho) for _ in range(3)]
        return st
    st["rhs"] = st["solver"].divergence(us, 1.0 / DT)
    if kind == "solve":
        st["p"] = torch.empty_like(rho)
        return st
    st["beta"] = [b.requires_grad_(True) for b in beta]
    st["rhs"].requires_grad_(True)
    st["w"] = torch.rand(rho.shape, generator=gen, device=DEVICE, dtype=torch.float64)
    st["w"].mul_(2.0).sub_(1.0)
    return st


def run(st):
    sol, tol, kind = st["solver"], st["tol"], st["kind"]
    if kind == "step":
        p, u = sol.step(st["rho"], st["us"], DT, tol=tol, p=st["p"], rhs=st["b"], out=st["out"])
        return {"b": st["b"], "p": p, "u": list(u)}
    if kind == "calls":
        sol.update_density(st["rho"])
        b = sol.divergence(st["us"], 1.0 / DT, out=st["b"])
        p = sol.solve(b, tol=tol, p=st["p"])
        return {"b": b, "p": p, "u": list(sol.project(st["us"], p, DT, out=st["out"]))}
    if kind == "solve":
        return {"p": sol.solve(st["rhs"], tol=tol, p=st["p"])}
    if kind == "grad":
        p = S.pressure_solve(st["rhs"], st["beta"], sol, tol=tol)
        g = torch.autograd.grad(p, [st["rhs"], *st["beta"]], grad_outputs=st["w"])
        return {"p": p.detach(), "g_rhs": g[0], "g_beta": list(g[1:])}
    if kind == "viscous":
        for u, b, x in zip(st["us"], st["rhs"], st["out"]):
            x.copy_(u)                        # the old velocity is the first guess
            sol.solve(b, tol=tol, p=x)
        return {"u": list(st["out"])}
    b = sol.divergence(st["us"], 1.0 / DT, out=st["b"])
    p = sol.solve(b, tol=tol, p=st["p"])
    return {"b": b, "p": p, "u": list(sol.project(st["us"], p, DT, out=st["out"]))}


def work(case):
    """Each input read once and each output written once, 8 bytes a value; the
    operations of one application of the operator and of what goes around it."""
    n = case["nx"] * case["ny"] * case["nz"]
    words, ops = {"step": (4 + 5, 40), "calls": (4 + 5, 40), "solve": (4 + 1, 20),
                  "grad": (5 + 5, 55), "viscous": (4 + 3 + 3, 66),
                  "solids": (3 + 3 + 5, 40)}[case["kind"]]
    return {"bytes": 8.0 * words * n, "flops": float(ops) * n}


# -- the same results in plain torch, FP64 ----------------------------------------

EXACT_CELLS = 256 ** 3


def _down(x, m):
    return x.roll(1, 2 - m)


def _up(x, m):
    return x.roll(-1, 2 - m)


def _faces(rho, bc):
    out = []
    for m in range(3):
        b = 2.0 / (rho + _down(rho, m))
        if bc[m]:
            b.select(2 - m, 0).zero_()
        out.append(b)
    return out


def _exact_solve(beta, sigma, h, rhs):
    """x with A x - sigma x = rhs (mean-free over the active cells when sigma
    is None); cells without an open face are 0."""
    ih2 = 1.0 / (h * h)
    hi = [_up(b, m) for m, b in enumerate(beta)]
    diag = sum(beta) + sum(hi)
    diag *= ih2
    if sigma is not None:
        diag = diag + sigma
    act = diag > 0
    inv = torch.where(act, 1.0 / diag, torch.zeros_like(diag))
    na = act.sum()

    def apply(x):                             # -(A - sigma) x
        y = diag * x
        for m in range(3):
            y -= ih2 * (beta[m] * _down(x, m) + hi[m] * _up(x, m))
        return y

    def centre(v):
        return torch.where(act, v - (v * act).sum() / na, torch.zeros_like(v)) if sigma is None else v * act

    b = -centre(rhs)
    x = torch.zeros_like(b)
    for restart in range(3):                  # a second run on the residual of the first
        r = centre(b - apply(x))
        bb = (b * b).sum().item()
        z = inv * r
        d = z.clone()
        rz = (r * z).sum()
        e = torch.zeros_like(b)
        for it in range(30000):
            q = apply(d)
            a = rz / (d * q).sum()
            e.addcmul_(d, a)
            r.addcmul_(q, -a)
            z = inv * r
            new = (r * z).sum()
            d.mul_(new / rz).add_(z)
            rz = new
            if it % 50 == 49 and (r * r).sum().item() <= 1e-26 * bb:
                break
        x = centre(x + e)
        if (centre(b - apply(x)) ** 2).sum().item() <= 1e-25 * bb:
            break
    return x


def _exact_divergence(us, beta, bc, h, closed):
    out = torch.zeros_like(us[0])
    for m in range(3):
        u = us[m].clone()
        if bc[m]:
            u.select(2 - m, 0).zero_()
        if closed:
            u[beta[m] == 0] = 0.0
        out += (_up(u, m) - u) / h
    return out / DT


def _exact_project(us, beta, p, h):
    return [torch.where(beta[m] > 0, us[m] - DT * beta[m] * (p - _down(p, m)) / h,
                        torch.zeros_like(p)) for m in range(3)]


def exact(case, seed):
    n, h = _grid(case)
    if n[0] * n[1] * n[2] > EXACT_CELLS:
        return None
    bc, kind = _bc(case), case["kind"]
    if kind in ("viscous", "solids"):
        rho, us, beta, sigma = _general(case, seed)
        for m in range(3):
            if bc[m]:
                beta[m].select(2 - m, 0).zero_()
        if kind == "viscous":
            return {"u": [_exact_solve(beta, sigma, h, -sigma * u) for u in us]}
        b = _exact_divergence(us, beta, bc, h, True)
        p = _exact_solve(beta, None, h, b)
        return {"b": b, "p": p, "u": _exact_project(us, beta, p, h)}
    rho, us, gen = _inputs(case, seed)
    beta = _faces(rho, bc)
    b = _exact_divergence(us, beta, bc, h, False)
    p = _exact_solve(beta, None, h, b)
    if kind == "solve":
        return {"p": p}
    if kind in ("step", "calls"):
        return {"b": b, "p": p, "u": _exact_project(us, beta, p, h)}
    w = torch.rand(rho.shape, generator=gen, device=DEVICE, dtype=torch.float64).mul_(2.0).sub_(1.0)
    lam = _exact_solve(beta, None, h, w)
    g = [torch.where(beta[m] > 0, (lam - _down(lam, m)) * (p - _down(p, m)) / (h * h),
                     torch.zeros_like(p)) for m in range(3)]
    return {"p": p, "g_rhs": lam, "g_beta": g}
