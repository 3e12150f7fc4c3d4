"""Performance cases of the pressure-Poisson tree-code.

Each case is work that a user of the library has it do, through its Python
entry points: the full-field and the surface pressure solve on grids from 64^2
to 4096^2, solves of several bodies at once, the time step on a kept tree,
scattered sources, the paper's tree-code evaluation, and the whole step from a
velocity field to the forces on a body.  Inputs are synthetic: the pressure
source of seeded Lamb-Oseen vortices (f = 2 (u_x v_y - u_y v_x)), whole, masked
to a band around a swimmer's midline, or times a Gaussian envelope; targets are
all grid nodes, an ellipse, or a fish body's surface points and their copies
lifted 2h along the normal.

    listed()            the cases, from the smallest call to the largest
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs on the GPU, and the solver a program keeps
    run(state)          one pass; its outputs
    work(case)          bytes and flops of a pass that it cannot do without
    exact(case, seed)   the outputs in 64 bits by direct summation (torch only)
"""

import math

import numpy as np
import torch

import paper_1610_04398_amd as pp

DEVICE = "cuda"
F64 = torch.float64
KAPPA = 1.5 - math.pi / 4.0 + math.log(2.0) / 2.0  # the cell average of ln r over an h x h cell is ln h - KAPPA


# ---------------------------------------------------------------- the cases

def _grid(name, nx, ny, source, targets, m, p=12, theta=0.5, precision="mixed", self_mode="skip", method="fmm",
          vortices=64, call="solve", nreq=1):
    return dict(name=name, call=call, nx=nx, ny=ny, source=source, vortices=vortices, targets=targets, m=m, p=p,
                theta=theta, precision=precision, self_mode=self_mode, method=method, nreq=nreq)


def listed():
    return [
        # the smallest call: a coarse field at all its nodes in FP64 (latency and launches count)
        _grid("nodes_64_fp64", 64, 64, "gauss", "nodes", 0, p=8, precision="fp64"),
        # the smallest serving request: the pressure on one ellipse in a 128^2 flow
        _grid("ellipse_128", 128, 128, "vortex", "ellipse", 1237, vortices=24),
        # the largest serving request: a fish in a 1024^2 flow
        _grid("fish_1024", 1024, 1024, "vortex", "fish", 8192),
        # an odd rectangular domain, both FP64 and the cell-average self rule: the reference-accuracy field
        _grid("nodes_301x243_fp64", 301, 243, "vortex", "nodes", 0, precision="fp64", self_mode="cellavg"),
        # queued requests of one shape solved together, as the server does
        _grid("batch_6x256", 256, 256, "vortex", "ellipse", 2050, vortices=32, call="batch", nreq=6),
        # the full-field evaluation plus a body surface
        _grid("nodes_512", 512, 512, "vortex", "nodes+ellipse", 2048),
        # the same field by the paper's own tree-code evaluation
        _grid("treecode_512", 512, 512, "vortex", "nodes+ellipse", 2048, method="treecode"),
        # a swimmer in a large, mostly empty domain at high order
        _grid("band_2048_p16", 2048, 2048, "band", "fish", 16384, p=16, theta=0.4),
        # the largest domain: two wakes in 4096^2, surface and lifted targets
        _grid("envelope_4096", 4096, 4096, "envelope", "fish2", 32768),
        # the same domain's next time step on the kept tree
        _grid("resident_4096", 4096, 4096, "envelope", "fish2", 32768, call="resident"),
        # scattered sources with their own cell areas (a grid stretched towards the body), some targets on them
        dict(name="points_256", call="points", nx=256, ny=256, vortices=64, targets="coincident+ellipse", m=2048,
             p=12, theta=0.5, precision="mixed", method="fmm"),
        # one whole step: velocity -> source -> pressure on the body -> pressure and viscous forces
        dict(name="step_1024", call="step", nx=1024, ny=1024, vortices=32, m=4096, p=12, theta=0.5,
             precision="mixed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["solve", "solve", "nodes", "nodes", "treecode", "batch", "resident", "points", "points",
                       "step"])
    prec = rng.choice(["mixed", "mixed", "fp64"])
    p = rng.choice([8, 12, 12, 16])
    nv = rng.randint(16, 64)
    if call == "solve":
        n = _log_int(rng, 96, 4096)
        nx, ny = rng.choice([(n, n), (n, max(64, n * 2 // 3)), (max(64, n // 2 + 1), n)])
        source = rng.choice(["vortex", "envelope"]) if n <= 2048 else "envelope"
        return dict(call="solve", nx=nx, ny=ny, source=source, vortices=nv,
                    targets=rng.choice(["ellipse", "fish"]) if nx == ny else "ellipse",
                    m=_log_int(rng, 512, 32768), p=p, theta=0.5, precision=prec, self_mode="skip", method="fmm",
                    nreq=1)
    if call in ("nodes", "treecode"):
        n = _log_int(rng, 64, 512 if prec == "mixed" else 320)
        nx, ny = rng.choice([(n, n), (n, max(48, n * 3 // 4))])
        return dict(call="solve", nx=nx, ny=ny, source="vortex", vortices=nv, targets="nodes+ellipse",
                    m=_log_int(rng, 256, 2048), p=p, theta=rng.choice([0.5, 0.5, 0.4]), precision=prec,
                    self_mode=rng.choice(["skip", "cellavg"]), method="fmm" if call == "nodes" else "treecode", nreq=1)
    if call == "batch":
        n = _log_int(rng, 128, 512)
        return dict(call="batch", nx=n, ny=n, source="vortex", vortices=nv, targets="ellipse",
                    m=_log_int(rng, 1024, 8192), p=12, theta=0.5, precision=prec, self_mode="skip", method="fmm",
                    nreq=rng.randint(2, 8))
    if call == "resident":
        n = _log_int(rng, 256, 4096)
        return dict(call="resident", nx=n, ny=n, source="envelope", vortices=nv, targets="fish2",
                    m=4 * _log_int(rng, 512, 8192), p=12, theta=0.5, precision="mixed", self_mode="skip",
                    method="fmm", nreq=1)
    if call == "points":
        n = _log_int(rng, 64, 512)
        return dict(call="points", nx=n, ny=_log_int(rng, 64, 512), vortices=nv,
                    targets=rng.choice(["coincident+ellipse", "ellipse"]), m=_log_int(rng, 512, 8192), p=p, theta=0.5,
                    precision=prec, method=rng.choice(["fmm", "fmm", "treecode"]))
    n = _log_int(rng, 128, 2048)
    return dict(call="step", nx=n, ny=n, vortices=nv, m=_log_int(rng, 512, 8192), p=12, theta=0.5, precision=prec)


# ---------------------------------------------------------------- inputs

def _rng(seed, *more):
    return np.random.Generator(np.random.PCG64((int(seed), *more)))


def _dev(a):
    return torch.as_tensor(a, dtype=F64, device=DEVICE)


def _frame(case, rng):
    """(h, x0, y0) of the grid: unit width, an anchor away from the origin for rectangular domains."""
    nx, ny = case["nx"], case["ny"]
    h = 1.0 / max(nx, ny)
    return (h, 0.0, 0.0) if nx == ny else (h, float(rng.uniform(-1.0, 1.0)), float(rng.uniform(-1.0, 1.0)))


def _axes(nx, ny, h, x0, y0):
    """Node coordinates x0 + (i + 1/2) h along each axis, every operation rounded."""
    x = (torch.arange(nx, dtype=F64, device=DEVICE) + 0.5) * h
    y = (torch.arange(ny, dtype=F64, device=DEVICE) + 0.5) * h
    return x + x0, y + y0


def _vortices(rng, n, x0=0.0, y0=0.0, w=1.0, hgt=1.0):
    c = rng.uniform(0.0, 1.0, size=(n, 2))
    return x0 + w * c[:, 0], y0 + hgt * c[:, 1], rng.standard_normal(n), rng.uniform(0.01, 0.05, size=n)


def _vortex_source(X, Y, vort):
    """2 (u_x v_y - u_y v_x) of Lamb-Oseen vortices at (X, Y), broadcast together."""
    shape = torch.broadcast_shapes(X.shape, Y.shape)
    ux, uy, vx, vy = (torch.zeros(shape, dtype=F64, device=DEVICE) for _ in range(4))
    for xc, yc, gm, rc in zip(*vort):
        K, a = float(gm) / (2.0 * math.pi), float(rc) ** 2
        dx, dy = X - float(xc), Y - float(yc)
        s = (dx * dx + dy * dy).clamp_min_(1e-6 * a)
        e = torch.exp(-s / a)
        g = -torch.expm1(-s / a) / s
        gp = (s * e / a - g * s) / (s * s)
        ux -= (2.0 * K) * dx * dy * gp
        vy += (2.0 * K) * dx * dy * gp
        uy -= K * (g + 2.0 * dy * dy * gp)
        vx += K * (g + 2.0 * dx * dx * gp)
    return 2.0 * (ux * vy - uy * vx)


def _velocity(X, Y, vort):
    shape = torch.broadcast_shapes(X.shape, Y.shape)
    u, v = torch.zeros(shape, dtype=F64, device=DEVICE), torch.zeros(shape, dtype=F64, device=DEVICE)
    for xc, yc, gm, rc in zip(*vort):
        K, a = float(gm) / (2.0 * math.pi), float(rc) ** 2
        dx, dy = X - float(xc), Y - float(yc)
        s = (dx * dx + dy * dy).clamp_min_(1e-6 * a)
        g = -torch.expm1(-s / a) / s
        u -= K * g * dy
        v += K * g * dx
    return u, v


def _midline(x, yc, phase):
    return yc + 0.1 * torch.sin(2.0 * math.pi * ((x - 0.2) / 0.6 - phase))


def _bodies(case, rng):
    """(yc, phase) of the midline of each swimmer of the case."""
    two = case["source"] == "envelope"
    return [(yc, float(rng.uniform())) for yc in ((0.35, 0.65) if two else (0.5,))]


def _source(case, rng, bodies, h, x0, y0):
    nx, ny = case["nx"], case["ny"]
    x, y = _axes(nx, ny, h, x0, y0)
    X, Y = x[None, :], y[:, None]
    if case["source"] == "gauss":
        cx, cy = rng.uniform(0.4, 0.6, size=2)
        return torch.exp(-((X - float(cx)) ** 2 + (Y - float(cy)) ** 2) / 0.01).contiguous()
    f = _vortex_source(X, Y, _vortices(rng, case["vortices"], x0, y0, nx * h, ny * h))
    xs, ys = (X - x0) / (nx * h), (Y - y0) / (ny * h)
    if case["source"] == "band":
        yc, phase = bodies[0]
        f *= (xs >= 0.2) & (xs <= 0.8) & ((ys - _midline(xs, yc, phase)).abs() <= 0.05)
    elif case["source"] == "envelope":
        out_x = torch.clamp_min(torch.maximum(0.2 - xs, xs - 0.8), 0.0)
        e = torch.zeros_like(f)
        for yc, phase in bodies:
            e += torch.exp(-((ys - _midline(xs, yc, phase)) ** 2 + out_x * out_x) / 0.02 ** 2)
        f *= torch.where(e >= 1e-16, e, torch.zeros_like(e))
    return f


def _ellipse(m, rng, x0=0.0, y0=0.0, w=1.0, hgt=1.0):
    cx, cy = rng.uniform(0.45, 0.55, size=2)
    th = float(rng.uniform(-0.3, 0.3))
    t = (2.0 * math.pi / m) * torch.arange(m, dtype=F64, device=DEVICE)
    s = min(w, hgt)
    ex, ey = 0.2 * s * torch.cos(t), 0.05 * s * torch.sin(t)
    return (x0 + w * float(cx) + math.cos(th) * ex - math.sin(th) * ey,
            y0 + hgt * float(cy) + math.sin(th) * ex + math.cos(th) * ey)


def _fish(m, h, yc, phase):
    """m points: a fish body's surface (both sides) and the same points lifted 2h along the normal."""
    n = max(1, m // 4)
    x = 0.2 + 0.6 * (torch.arange(n, dtype=F64, device=DEVICE) + 0.5) / n
    y = _midline(x, yc, phase)
    dy = (0.1 * 2.0 * math.pi / 0.6) * torch.cos(2.0 * math.pi * ((x - 0.2) / 0.6 - phase))
    q = torch.sqrt(1.0 + dy * dy)
    nx, ny = -dy / q, 1.0 / q
    s, L = (x - 0.2) / 0.6 * 0.8, 0.8
    wh, st, wt = 0.04 * L, 0.95 * L, 0.01 * L
    head = torch.sqrt(torch.clamp_min(2.0 * wh * s - s * s, 0.0))
    mid = wh - (wh - wt) * (s - wh) / (st - wh)
    w = torch.where(s < wh, head, torch.where(s < st, mid, wt * (L - s) / (L - st)))
    parts = [(x + d * nx, y + d * ny) for d in (w, -w, w + 2 * h, -(w + 2 * h))]
    return torch.cat([a for a, _ in parts]), torch.cat([b for _, b in parts])


def _targets(case, rng, bodies, h, x0, y0):
    kind, m, nx, ny = case["targets"], case["m"], case["nx"], case["ny"]
    if kind == "fish":
        return _fish(m, h, *bodies[0])
    if kind == "fish2":
        a = [_fish(m // 2, h, *b) for b in bodies]
        return torch.cat([q[0] for q in a]), torch.cat([q[1] for q in a])
    tx, ty = [], []
    if kind.startswith("nodes"):
        x, y = _axes(nx, ny, h, x0, y0)
        tx.append(x[None, :].expand(ny, nx).reshape(-1))
        ty.append(y[:, None].expand(ny, nx).reshape(-1))
    if kind.endswith("ellipse"):
        a, b = _ellipse(m, rng, x0, y0, nx * h, ny * h)
        tx.append(a)
        ty.append(b)
    return torch.cat(tx).contiguous(), torch.cat(ty).contiguous()


def _grid_inputs(case, seed, request=0):
    rng = _rng(seed, 1, request)
    h, x0, y0 = _frame(case, rng)
    bodies = _bodies(case, rng)
    f = _source(case, rng, bodies, h, x0, y0).contiguous()
    tx, ty = _targets(case, rng, bodies, h, x0, y0)
    return dict(f=f, h=h, x0=x0, y0=y0, tx=tx, ty=ty)


def _stretched(n):
    """Cell centres and widths of [0, 1] cut into n cells refined towards the middle."""
    e = torch.sinh(2.0 * (torch.arange(n + 1, dtype=F64, device=DEVICE) / n - 0.5))
    e = (e - e[0]) / (e[-1] - e[0])
    return 0.5 * (e[1:] + e[:-1]), e[1:] - e[:-1]


def _points_inputs(case, seed):
    rng = _rng(seed, 2)
    cx, wx = _stretched(case["nx"])
    cy, wy = _stretched(case["ny"])
    f = _vortex_source(cx[None, :], cy[:, None], _vortices(rng, case["vortices"]))
    sx = cx[None, :].expand_as(f).reshape(-1).contiguous()
    sy = cy[:, None].expand_as(f).reshape(-1).contiguous()
    w = (f * wx[None, :] * wy[:, None]).reshape(-1).contiguous()
    tx, ty = _ellipse(case["m"], rng)
    if case["targets"].startswith("coincident"):
        tx, ty = torch.cat([sx[::7], tx]), torch.cat([sy[::7], ty])
    return dict(sx=sx, sy=sy, w=w, tx=tx, ty=ty)


def _step_inputs(case, seed):
    rng = _rng(seed, 3)
    n, m = case["nx"], case["m"]
    h = 1.0 / n
    x, y = _axes(n, n, h, 0.0, 0.0)
    X, Y = x[None, :], y[:, None]
    u, v = _velocity(X, Y, _vortices(rng, case["vortices"]))
    cx, cy = (float(c) for c in rng.uniform(0.45, 0.55, size=2))
    re = torch.sqrt(((X - cx) / 0.2) ** 2 + ((Y - cy) / 0.05) ** 2)
    d, eps = 0.05 * (1.0 - re), 2.0 * h
    chi = torch.where(d <= -eps, 0.0, torch.where(d >= eps, 1.0, 0.5 * (1 + d / eps + torch.sin(math.pi * d / eps) / math.pi)))
    om = float(rng.uniform(0.5, 1.5))
    us = (-om * (Y - cy)).expand(n, n).contiguous()
    vs = (om * (X - cx)).expand(n, n).contiguous()
    t = (2.0 * math.pi / m) * torch.arange(m + 1, dtype=F64, device=DEVICE)
    px, py = cx + 0.2 * torch.cos(t), cy + 0.05 * torch.sin(t)  # the body's polygon, counter-clockwise
    ex, ey = px[1:] - px[:-1], py[1:] - py[:-1]
    ds = torch.sqrt(ex * ex + ey * ey)
    nx_, ny_ = ey / ds, -ex / ds
    tx, ty = 0.5 * (px[1:] + px[:-1]), 0.5 * (py[1:] + py[:-1])
    return dict(u=u, v=v, chi=chi.contiguous(), us=us, vs=vs, h=h, lam=50.0, tx=tx, ty=ty, nx=nx_, ny=ny_, ds=ds,
                lx=tx + 2 * h * nx_, ly=ty + 2 * h * ny_, seg=np.array([0, m], dtype=np.int64), mu=1e-3)


# ---------------------------------------------------------------- one pass

def _options(case):
    o = dict(p=case["p"], theta=case["theta"], precision=case["precision"])
    if "self_mode" in case:
        o["self_mode"] = case["self_mode"]
    return o


def prepare(case, seed):
    call = case["call"]
    st = dict(call=call, solver=pp.Solver(0), opt=_options(case))
    if call == "points":
        st.update(_points_inputs(case, seed))
        st["opt"]["method"] = case["method"]
        st["out"] = torch.empty_like(st["tx"])
        return st
    if call == "step":
        st.update(_step_inputs(case, seed))
        st["f"] = torch.empty_like(st["u"])
        st["out"] = torch.empty_like(st["tx"])
        return st
    if call == "batch":
        reqs = [_grid_inputs(case, seed, r) for r in range(case["nreq"])]
        st.update(h=reqs[0]["h"], x0=reqs[0]["x0"], y0=reqs[0]["y0"])
        for k in ("f", "tx", "ty"):
            st[k] = [q[k] for q in reqs]
        st["out"] = [torch.empty_like(t) for t in st["tx"]]
        return st
    st.update(_grid_inputs(case, seed))
    st["out"] = torch.empty_like(st["tx"])
    if call == "resident":
        # the first time step builds the tree that the later ones keep
        torch.cuda.synchronize()
        st["solver"].solve_grid(st["f"], st["h"], st["tx"], st["ty"], st["x0"], st["y0"], out=st["out"], **st["opt"])
        st["f"] = _next_step(st["f"], seed)
    else:
        st["opt"]["method"] = case["method"]
    return st


def _next_step(f, seed):
    """The source of a later time step: the same nonzero nodes, other values."""
    amp = _rng(seed, 4).uniform(0.2, 0.8)
    j = torch.arange(f.shape[0], dtype=F64, device=DEVICE)[:, None] / f.shape[0]
    return f * (1.0 + float(amp) * torch.sin(6.0 * j))


def run(st):
    call, s, opt = st["call"], st["solver"], st["opt"]
    if call == "solve":
        return s.solve_grid(st["f"], st["h"], st["tx"], st["ty"], st["x0"], st["y0"], out=st["out"], **opt)
    if call == "resident":
        return s.solve_grid_resident(st["f"], st["tx"], st["ty"], out=st["out"])
    if call == "batch":
        return s.solve_grid_batch(st["f"], st["h"], st["tx"], st["ty"], st["x0"], st["y0"], outs=st["out"], **opt)
    if call == "points":
        return s.solve_points(st["sx"], st["sy"], st["w"], st["tx"], st["ty"], out=st["out"], **opt)
    f = s.pressure_source(st["u"], st["v"], st["h"], lam=st["lam"], chi=st["chi"], us=st["us"], vs=st["vs"],
                          out=st["f"])
    p = s.solve_grid(f, st["h"], st["tx"], st["ty"], out=st["out"], **opt)
    fp, px, py = s.surface_forces(p, st["nx"], st["ny"], st["ds"], st["seg"], pointwise=True)
    fv, vx, vy = s.viscous_forces(st["u"], st["v"], st["h"], st["lx"], st["ly"], st["nx"], st["ny"], st["ds"],
                                  st["seg"], mu=st["mu"], pointwise=True)
    return dict(f=f, p=p, px=px, py=py, vx=vx, vy=vy, pressure=fp, viscous=fv)


# ---------------------------------------------------------------- necessary work

def work(case):
    """Inputs read once, outputs written once; per source its leaf's p + 1 complex multipole terms, per
    target its leaf's p + 1 local terms and the pairs with the nearest leaves (nine half-full leaves of 64;
    6 operations a pair)."""
    nx, ny, p = case["nx"], case["ny"], case["p"]
    nodes = nx * ny
    if case["call"] == "points":
        m = case["m"] + (-(-nodes // 7) if case["targets"].startswith("coincident") else 0)
        bytes_ = 24 * nodes + 24 * m
        n = nodes
    elif case["call"] == "step":
        m, n = case["m"], nodes
        bytes_ = 48 * nodes + 24 * m + (5 + 2 + 7 + 2) * 8 * m
    else:
        m = case["m"] + (nodes if case["targets"].startswith("nodes") else 0)
        if case["targets"] == "nodes":
            m = nodes
        # the masked sources keep this share of the nodes
        n = nodes * {"gauss": 1.0, "vortex": 1.0, "band": 0.06, "envelope": 0.37}[case["source"]]
        m, n, bytes_ = m * case["nreq"], n * case["nreq"], (8 * nodes + 24 * m) * case["nreq"]
    return {"bytes": float(bytes_), "flops": float(8 * (p + 1) * (n + m) + 6 * m * min(n, 9 * 32))}


# ---------------------------------------------------------------- the sum itself, in 64 bits

def _direct(sx, sy, w, tx, ty, self_term=0.0):
    """(1/2pi) sum_i w_i ln|t_j - s_i| by direct summation; a coincident pair adds w self_term."""
    keep = w != 0
    sx, sy, w = sx[keep], sy[keep], w[keep]
    out = torch.zeros_like(tx)
    if not sx.numel():
        return out
    rows = 512
    cols = 1 << 15
    for a in range(0, tx.numel(), rows):
        x, y = tx[a:a + rows, None], ty[a:a + rows, None]
        acc = torch.zeros(x.shape[0], dtype=F64, device=tx.device)
        for b in range(0, sx.numel(), cols):
            dx = x - sx[None, b:b + cols]
            dy = y - sy[None, b:b + cols]
            r2 = dx.mul_(dx).addcmul_(dy, dy)
            hit = r2 == 0.0
            lg = r2.masked_fill_(hit, 1.0).log_().mul_(0.5)
            if self_term:
                lg.masked_fill_(hit, self_term)
            acc += lg @ w[b:b + cols]
        out[a:a + rows] = acc
    return out / (2.0 * math.pi)


def _direct_grid(g, f, self_mode):
    x, y = _axes(f.shape[1], f.shape[0], g["h"], g["x0"], g["y0"])
    sx = x[None, :].expand_as(f).reshape(-1)
    sy = y[:, None].expand_as(f).reshape(-1)
    term = math.log(g["h"]) - KAPPA if self_mode == "cellavg" else 0.0
    return _direct(sx, sy, (f * g["h"] ** 2).reshape(-1), g["tx"], g["ty"], term)


def _pairs(case):
    nodes = case["nx"] * case["ny"]
    m = case["m"] + (nodes if case.get("targets", "").startswith("nodes") else 0)
    m += nodes // 7 if case.get("targets", "").startswith("coincident") else 0
    share = {"band": 0.06, "envelope": 0.37}.get(case.get("source"), 1.0)
    return nodes * share * m * case.get("nreq", 1)


def _diff(a, axis, h):
    """Central differences inside, second-order one-sided ones on the first and last node."""
    return torch.gradient(a, spacing=h, dim=axis, edge_order=2)[0]


def exact(case, seed):
    if _pairs(case) > 6e11:  # over about 15 seconds of direct summation
        return None
    call = case["call"]
    if call == "points":
        q = _points_inputs(case, seed)
        return _direct(q["sx"], q["sy"], q["w"], q["tx"], q["ty"])
    if call == "batch":
        qs = [_grid_inputs(case, seed, r) for r in range(case["nreq"])]
        return [_direct_grid(q, q["f"], case["self_mode"]) for q in qs]
    if call != "step":
        q = _grid_inputs(case, seed)
        return _direct_grid(q, _next_step(q["f"], seed) if call == "resident" else q["f"], case["self_mode"])
    q = _step_inputs(case, seed)
    h = q["h"]
    ux, uy, vx, vy = _diff(q["u"], 1, h), _diff(q["u"], 0, h), _diff(q["v"], 1, h), _diff(q["v"], 0, h)
    pen = _diff(q["chi"] * (q["us"] - q["u"]), 1, h) + _diff(q["chi"] * (q["vs"] - q["v"]), 0, h)
    f = -(ux * ux + 2.0 * uy * vx + vy * vy) + q["lam"] * pen
    p = _direct_grid(dict(q, x0=0.0, y0=0.0), f, "skip")
    px, py = -p * q["nx"] * q["ds"], -p * q["ny"] * q["ds"]
    n = case["nx"]
    i = torch.floor(q["lx"] / h).long().clamp_(0, n - 1)
    j = torch.floor(q["ly"] / h).long().clamp_(0, n - 1)
    at = lambda a: a[j, i]  # noqa: E731
    off = 0.5 * (at(uy) + at(vx))
    tx = 2.0 * q["mu"] * (at(ux) * q["nx"] + off * q["ny"]) * q["ds"]
    ty = 2.0 * q["mu"] * (off * q["nx"] + at(vy) * q["ny"]) * q["ds"]
    force = lambda a, b: [dict(fx=float(a.sum()), fy=float(b.sum()), drag=float(a.sum()),  # noqa: E731
                               cd=2.0 * float(a.sum()))]
    return dict(f=f, p=p, px=px, py=py, vx=tx, vy=ty, pressure=force(px, py), viscous=force(tx, ty))
