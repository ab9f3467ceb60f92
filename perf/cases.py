"""Workloads that the solver's performance is measured on.

Each case is a plain dict.  Three kinds cover what a program does with the
library through its Python binding:

  run    one mesh: a device-resident initial state is handed over
         (Hydro.set_primitive_device), advanced some steps, and the conserved
         state is read where it lies (Hydro.state_view).  dt "device" uses
         Hydro.step_auto; dt "host" is the loop of a program that asks for each
         time step itself (cfl_dt, step) and for the totals at the end.
         blocks > 1 splits every axis; refine > 0 refines the central half of
         the root blocks.
  batch  many ragged 2-D shear layers stepped together from a captured graph.
  serve  one iteration of a server over freshly admitted 2-D and 3-D requests
         of either precision: batched steps launched directly, then the status.

exact() advances the same inputs with a plain FP64 torch evaluation of the
published scheme (minmod PLM on primitive variables, HLLC, Heun or van Leer).
"""
import math
import random

import torch

from paper_2501_02317_amd import hydro as H

DEV = "cuda"
PREC = {"fp64": H.FP64, "mixed": H.MIXED}
INTEG = {"heun": H.HEUN, "vl2": H.VL2}
BC = {"periodic": H.BC_PERIODIC, "free": H.BC_FREE, "outflow": H.BC_OUTFLOW, "reflect": H.BC_REFLECT}

# the most cells x steps, weighted by cost, that a drawn case may ask for
MOST = 256 ** 3 * 6


def run_case(name, n, prec, steps, integ="heun", bc="periodic", init="random", mach=1.0, gamma=5.0 / 3.0,
             dt="device", blocks=1, refine=0):
    n = tuple(n) + (0,) * (3 - len(n))
    c = {"kind": "run", "nx": n[0], "ny": n[1], "nz": n[2], "prec": prec, "integ": integ, "bc": bc, "init": init,
         "mach": mach, "gamma": gamma, "steps": steps, "dt": dt, "blocks": blocks, "refine": refine}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a shock tube of 256 cells, where launches are all there is
        run_case("tube_1d_256_fp64", (256,), "fp64", 100, bc="free", init="tube", gamma=1.4),
        # a small 2-D run whose program takes every time step itself
        run_case("host_dt_2d_160x96_mixed", (160, 96), "mixed", 16, gamma=1.4, dt="host"),
        # the implosion in a reflecting box at its usual size
        run_case("implosion_2d_256_fp64", (256, 256), "fp64", 40, bc="reflect", init="diagonal", gamma=1.4),
        # the paper's Table 1 grid
        run_case("grid_2d_4096x1024_mixed", (4096, 1024), "mixed", 10, gamma=1.4),
        # a small 3-D run, as the serving mix has many
        run_case("box_3d_48_mixed", (48, 48, 48), "mixed", 40, mach=2.0),
        # an odd box with open sides, no extent a multiple of a tile
        run_case("open_3d_101x75x50_fp64", (101, 75, 50), "fp64", 20, bc="outflow", init="blast", gamma=1.4),
        # the headline workload in both precisions: 256^3, Mach 2
        run_case("box_3d_256_mixed", (256, 256, 256), "mixed", 8, mach=2.0),
        run_case("box_3d_256_fp64", (256, 256, 256), "fp64", 6, mach=2.0),
        # the memory-optimised van Leer integrator, on a mesh split into blocks
        run_case("vl2_3d_192_blocks_mixed", (192, 192, 192), "mixed", 10, integ="vl2", blocks=2),
        # the refined mesh: 4^3 root blocks of 32^3, the central eight refined
        run_case("refined_3d_128_mixed", (128, 128, 128), "mixed", 10, blocks=4, refine=1),
        # a batch of ragged 2-D meshes replayed from a graph
        {"name": "batch_2d_48_mixed", "kind": "batch", "count": 48, "lo": 64, "hi": 512, "prec": "mixed",
         "integ": "heun", "steps": 50, "sizes": 401},
        # a server's iteration over requests that have just arrived
        {"name": "serve_12_requests", "kind": "serve", "count": 12, "steps": 16, "sizes": 505},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run1", "run2", "run2", "run3", "run3", "run3", "run3", "split", "refined", "batch", "serve"])
    prec = rng.choice(["fp64", "mixed"])
    integ = rng.choice(["heun", "heun", "heun", "vl2"])
    gamma = rng.choice([1.4, 5.0 / 3.0])
    bc = rng.choice(["periodic", "periodic", "free", "outflow", "reflect"])
    mach = round(rng.uniform(0.5, 2.0), 3)
    if kind == "batch":
        return {"kind": "batch", "count": rng.randint(12, 60), "lo": 64, "hi": rng.choice([192, 256, 384]),
                "prec": prec, "integ": integ, "steps": rng.randint(10, 50), "sizes": rng.randrange(1 << 20)}
    if kind == "serve":
        return {"kind": "serve", "count": rng.randint(4, 12), "steps": 16, "sizes": rng.randrange(1 << 20)}
    blocks, refine = 1, 0
    if kind == "run1":
        n = (_log(rng, 64, 65536),)
    elif kind == "run2":
        n = (_log(rng, 33, 4096), _log(rng, 33, 1024))
    elif kind == "run3":
        n = tuple(_log(rng, 17, 250) for _ in range(3))
    elif kind == "split":
        blocks = rng.choice([2, 2, 4])
        n = tuple(blocks * rng.randint(10, 128 // blocks) for _ in range(3))
    else:
        blocks, refine, bc = 4, 1, rng.choice(["periodic", "periodic", "outflow"])
        n = (4 * 2 * rng.randint(5, 16),) * 3 if rng.random() < 0.7 else (4 * 2 * rng.randint(8, 64),) * 2
    cells = math.prod(n) * (2 if refine else 1)
    steps = max(1, min(rng.randint(8, 60), MOST // (4 * max(cells, 1 << 17))))
    dt = "host" if kind != "refined" and rng.random() < 0.15 else "device"
    init = "random" if bc == "periodic" or refine else rng.choice(["blast", "random"])
    return run_case(None, n, prec, steps, integ, bc, init, mach, gamma, dt, blocks, refine)


# ------------------------------------------------------------------- inputs

def _dims(c):
    return tuple(v for v in (c["nx"], c["ny"], c["nz"]) if v > 0)


def _box(n):
    """Upper corner of a box of cubic cells whose longest side is 1."""
    return tuple(v / max(n) for v in n)


def _bcs(c, nd):
    return ((BC[c["bc"]],) * 2,) * nd


def _centres(n, hi):
    """Cell-centre coordinates, shaped to broadcast over (nz, ny, nx)."""
    out = []
    for d, v in enumerate(n):
        shape = [1, 1, 1]
        shape[2 - d] = v
        out.append(((torch.arange(v, device=DEV, dtype=torch.float64) + 0.5) * (hi[d] / v)).reshape(shape))
    return out


def _waves(g, x, periods, kmax, slope, count=20):
    """Sum of seeded plane waves with integer wavenumbers over the periods."""
    nd = len(x)
    shape = torch.broadcast_shapes(*[v.shape for v in x])
    out = torch.zeros(shape, device=DEV, dtype=torch.float64)
    k = torch.randint(-kmax, kmax + 1, (count, nd), generator=g, device=DEV)
    k[:, 0] += (k == 0).all(1).long()
    amp = torch.randn(count, generator=g, device=DEV, dtype=torch.float64) * k.double().norm(dim=1) ** slope
    ph = torch.rand(count, generator=g, device=DEV, dtype=torch.float64) * (2 * math.pi)
    for m in range(count):
        # cos(a + b) over the axes as the real part of a product of phases
        z = amp[m] * torch.exp(1j * ph[m])
        for d in range(nd):
            z = z * torch.exp(1j * (2 * math.pi / periods[d]) * k[m, d] * x[d])
        out += z.real
    return out / out.std().clamp_min(1e-30)


def _random(g, n, hi, mach, gamma, kmax=8, x=None):
    """Log-normal density, random velocity of the given rms, uniform pressure."""
    nd = len(n)
    x = _centres(n, hi) if x is None else x
    kmax = max(1, min(kmax, min(n) // 8))
    rho = torch.exp(0.1 * _waves(g, x, hi, kmax, 0.0))
    vel = [_waves(g, x, hi, kmax, -2.0 if nd == 3 else -1.5) * (mach / math.sqrt(nd)) for _ in range(nd)]
    return torch.stack([rho] + vel + [torch.full_like(rho, 1.0 / gamma)])


def _initial(c, n, hi, g):
    nd = len(n)
    x = _centres(n, hi)
    shape = (1,) * (3 - nd) + tuple(reversed(n))
    if c["init"] == "random":
        return _random(g, n, hi, c["mach"], c["gamma"])
    u = torch.rand(4, generator=g, device=DEV, dtype=torch.float64)
    if c["init"] == "tube":  # two states, as the Sod tube and its neighbours
        low = (x[0] < 0.5).expand(shape)
        rho = torch.where(low, 1.0 + 0.2 * u[0], 0.125 + 0.05 * u[1])
        p = torch.where(low, 1.0 + 0.2 * u[2], 0.1 + 0.05 * u[3])
    elif c["init"] == "diagonal":  # low-pressure triangle in a corner
        low = (x[0] + x[1] < 0.4 + 0.2 * u[0]).expand(shape)
        rho = torch.where(low, 0.125 + 0.02 * u[1], 1.0)
        p = torch.where(low, 0.14 + 0.02 * u[2], 1.0)
    else:  # a hot ball in a gas at rest
        r2 = sum((x[d] - hi[d] * (0.4 + 0.2 * u[d])) ** 2 for d in range(nd)).expand(shape)
        hot = torch.exp(-r2 / (0.15 * min(hi)) ** 2)
        rho, p = 1.0 + 0.5 * hot, 0.1 + (3.0 + u[3]) * hot
    zero = torch.zeros(shape, device=DEV, dtype=torch.float64)
    return torch.stack([rho] + [zero] * nd + [p])


def _shear(g, nx, ny):
    """Double shear layer on a periodic unit square, density ratio 1:2."""
    x, y = _centres((nx, ny), (1.0, 1.0))
    th = torch.tanh(((y - 0.5).abs() - 0.25) / 0.02) + 0.0 * x
    k = torch.arange(1, 9, device=DEV, dtype=torch.float64).reshape(8, 1, 1, 1)
    ph = torch.rand(8, 1, 1, 1, generator=g, device=DEV, dtype=torch.float64)
    w = torch.sin(2 * math.pi * (k * x + ph)).sum(0)
    env = torch.exp(-((y - 0.25) ** 2) / 0.08) + torch.exp(-((y - 0.75) ** 2) / 0.08)
    return torch.stack([1.5 + 0.5 * th, 0.5 * th, 0.01 * (w / w.abs().max()) * env, torch.full_like(th, 2.5)])


def _members(c):
    """(n, precision, gamma, cfl, mach) of every member of a batch."""
    r = random.Random(c["sizes"])
    out = []
    for _ in range(c["count"]):
        if c["kind"] == "batch":
            widths = [w for w in (64, 96, 128, 192, 256, 384, 512) if c["lo"] <= w <= c["hi"]]
            out.append(((r.choice(widths), r.choice(widths)), c["prec"], 1.4, 0.4, 0.5))
        else:
            nd = r.choice([2, 3])
            lo, hi, q = (64, 1024, 32) if nd == 2 else (32, 160, 16)
            v = max(lo, min(hi, round(math.exp(r.uniform(math.log(lo), math.log(hi))) / q) * q))
            out.append(((v,) * nd, r.choice(["fp64", "mixed"]), r.choice([1.4, 5.0 / 3.0]), 0.3 if nd == 3 else 0.4,
                        r.uniform(0.5, 2.0)))
    return out


def _member_inputs(c, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    out = []
    for n, prec, gamma, cfl, mach in _members(c):
        out.append(_shear(g, *n) if c["kind"] == "batch" else _random(g, n, (1.0,) * len(n), mach, gamma))
    return out


def _refined(c):
    """The central half of the root blocks along every axis."""
    b, nd = c["blocks"], len(_dims(c))
    mid = range(b // 4, b - b // 4)
    ids = [0]
    for d in reversed(range(nd)):
        ids = [i * b + m for i in ids for m in mid]
    return ids


def _inputs(c, seed, leaves=None):
    g = torch.Generator(device=DEV).manual_seed(seed)
    n = _dims(c)
    hi = _box(n)
    if leaves is None:
        return _initial(c, n, hi, g).contiguous()
    # block layout of a refined mesh: a leaf's cells are the root blocks' cells
    # halved per level, each leaf with the coordinates of its own corner
    nd, b = len(n), c["blocks"]
    x = []
    lev = torch.tensor(leaves[:, 0], device=DEV, dtype=torch.float64)
    for d in range(nd):
        m = n[d] // b
        dx = (hi[d] / n[d]) * 2.0 ** -lev
        at = torch.tensor(leaves[:, 1 + d], device=DEV, dtype=torch.float64) * m * dx
        shape = [1, 1, 1, 1]
        shape[3 - d] = m
        i = torch.arange(m, device=DEV, dtype=torch.float64).reshape(shape) + 0.5
        x.append(at.reshape(-1, 1, 1, 1) + i * dx.reshape(-1, 1, 1, 1))
    W = _random(g, n, hi, min(c["mach"], 1.0), c["gamma"], kmax=4, x=x)
    return W.transpose(0, 1).contiguous()


# ------------------------------------------------------------ prepare and run

def prepare(case, seed):
    if case["kind"] != "run":
        stream = torch.cuda.Stream()
        fields = _member_inputs(case, seed)
        torch.cuda.current_stream().synchronize()
        meshes = [H.Hydro(n, gamma, cfl, precision=PREC[prec], device=DEV, stream=stream,
                          integrator=INTEG[case.get("integ", "heun")])
                  for n, prec, gamma, cfl, _ in _members(case)]
        batch = H.Batch(meshes, use_graph=case["kind"] == "batch")
        stream.synchronize()
        return {"case": case, "W": fields, "meshes": meshes, "batch": batch}
    n = _dims(case)
    nd = len(n)
    refined = _refined(case) if case["refine"] else None
    h = H.Hydro(n, case["gamma"], 0.3 if nd == 3 else 0.4, precision=PREC[case["prec"]], hi=_box(n),
                bc=_bcs(case, nd), device=DEV, integrator=INTEG[case["integ"]],
                blocks=(case["blocks"],) * nd if case["blocks"] > 1 else None, refined=refined)
    W = _inputs(case, seed, h.leaves if refined is not None else None)
    return {"case": case, "W": W, "mesh": h}


def run(state):
    c = state["case"]
    if c["kind"] != "run":
        for h, W in zip(state["meshes"], state["W"]):
            h.set_primitive_device(W)
        state["batch"].step(c["steps"])
        if c["kind"] == "batch":
            return [h.state_view() for h in state["meshes"]]
        done, steps, flags = state["batch"].status()
        return {"state": [h.state_view() for h in state["meshes"]], "steps": steps, "flags": flags}
    h = state["mesh"]
    h.set_primitive_device(state["W"])
    if c["dt"] == "host":
        for _ in range(c["steps"]):
            h.step(h.cfl_dt())
        return {"state": h.state_view(), "totals": h.totals()}
    h.step_auto(c["steps"])
    return h.state_view()


def _cells(case):
    """(cells, ndim, precision) of every mesh of a case."""
    if case["kind"] != "run":
        return [(math.prod(n), len(n), prec) for n, prec, *_ in _members(case)]
    n = _dims(case)
    cells = math.prod(n)
    if case["refine"]:
        r = len(_refined(case)) / case["blocks"] ** len(n)
        cells *= 1 - r + r * 2 ** len(n)
    return [(cells, len(n), case["prec"])]


def work(case):
    """Per pass: the initial state read, then per step the state read and
    written once, and the scheme's arithmetic (per stage: conversion, one
    reconstruction and Riemann solve per cell and axis, the update)."""
    b = f = 0.0
    for cells, nd, _ in _cells(case):
        nc = nd + 2
        b += cells * nc * 8 * (2 * case["steps"] + 2)
        f += cells * case["steps"] * 2 * (nd * (7 * nc + 75) + 6 * nc + 25)
    return {"bytes": b, "flops": f}


# ------------------------------------------------- plain FP64 evaluation

def _pad(W, bc, ax):
    """Two ghost layers on physical axis ax (array axis 3 - ax)."""
    d = 3 - ax
    N = W.shape[d]

    def at(i):
        return W.narrow(d, i, 1).clone()

    if bc == "periodic":
        lo, hi = [at(N - 2), at(N - 1)], [at(0), at(1)]
    elif bc == "reflect":
        lo, hi = [at(1), at(0)], [at(N - 1), at(N - 2)]
        for t in lo + hi:
            t[1 + ax].neg_()
    else:
        lo, hi = [at(0), at(0)], [at(N - 1), at(N - 1)]
        if bc == "outflow":
            for t in lo:
                t[1 + ax].clamp_(max=0.0)
            for t in hi:
                t[1 + ax].clamp_(min=0.0)
    return torch.cat(lo + [W] + hi, d)


def _minmod(a, b):
    return torch.where(a * b > 0, torch.where(a.abs() < b.abs(), a, b), torch.zeros((), device=DEV, dtype=a.dtype))


def _hllc(L, R, ax, gamma):
    """Flux of conserved variables along axis ax from primitive face states."""
    rl, ul, pl = L[0], L[1 + ax], L[-1]
    rr, ur, pr = R[0], R[1 + ax], R[-1]
    cl, cr = (gamma * pl / rl).sqrt(), (gamma * pr / rr).sqrt()
    ps = (0.5 * (pl + pr) - 0.125 * (ur - ul) * (rl + rr) * (cl + cr)).clamp_min(0.0)
    z = (gamma + 1) / (2 * gamma)
    dl = -cl * (1 + z * ((ps / pl).clamp_min(1.0) - 1)).sqrt()
    dr = cr * (1 + z * ((ps / pr).clamp_min(1.0) - 1)).sqrt()
    sl, sr = ul + dl, ur + dr
    ss = (pr - pl + rl * ul * dl - rr * ur * dr) / (rl * dl - rr * dr)
    left = (sl >= 0) | (ss >= 0)
    K = torch.where(left, L, R)
    s, ds = torch.where(left, sl, sr), torch.where(left, dl, dr)
    star = torch.where(left, sl < 0, sr > 0)
    rho, u, p = K[0], K[1 + ax], K[-1]
    E = p / (gamma - 1) + 0.5 * rho * (K[1:-1] ** 2).sum(0)
    F = torch.cat([(rho * u)[None], rho * u * K[1:-1], ((E + p) * u)[None]])
    F[1 + ax] += p
    chi = torch.where(star, rho * ds / torch.where(star, s - ss, torch.ones_like(s)), rho)
    Us = torch.cat([chi[None], chi * K[1:-1], (chi * (E / rho + (ss - u) * (ss + p / (rho * ds))))[None]])
    Us[1 + ax] = chi * ss
    U = torch.cat([rho[None], rho * K[1:-1], E[None]])
    return torch.where(star, F + s * (Us - U), F)


def _prim(U, gamma):
    v = U[1:-1] / U[0]
    return torch.cat([U[:1], v, ((gamma - 1) * (U[-1] - 0.5 * (U[1:-1] * v).sum(0)))[None]])


def _rhs(W, dx, bc, gamma, first=False):
    """-div F of the primitive state W."""
    out = torch.zeros_like(W)
    for ax in range(len(dx)):
        d = 3 - ax
        P = _pad(W, bc, ax)
        n = W.shape[d]
        if first:
            L, R = P.narrow(d, 1, n + 1), P.narrow(d, 2, n + 1)
        else:
            D = P.narrow(d, 1, n + 3) - P.narrow(d, 0, n + 3)
            S = _minmod(D.narrow(d, 0, n + 2), D.narrow(d, 1, n + 2))
            C = P.narrow(d, 1, n + 2)
            L, R = (C + 0.5 * S).narrow(d, 0, n + 1), (C - 0.5 * S).narrow(d, 1, n + 1)
        F = _hllc(L, R, ax, gamma)
        out += (F.narrow(d, 0, n) - F.narrow(d, 1, n)) / dx[ax]
    return out


def _advance(W, dx, bc, gamma, cfl, steps, vl2):
    U = torch.cat([W[:1], W[:1] * W[1:-1],
                   (W[-1] / (gamma - 1) + 0.5 * W[0] * (W[1:-1] ** 2).sum(0))[None]])
    nd = len(dx)
    for _ in range(steps):
        W = _prim(U, gamma)
        c = (gamma * W[-1] / W[0]).sqrt()
        dt = cfl / max(float(((W[1 + d].abs() + c) / dx[d]).max()) for d in range(nd))
        if vl2:
            U = U + dt * _rhs(_prim(U + 0.5 * dt * _rhs(W, dx, bc, gamma, True), gamma), dx, bc, gamma)
        else:
            U1 = U + dt * _rhs(W, dx, bc, gamma)
            U = 0.5 * U + 0.5 * (U1 + dt * _rhs(_prim(U1, gamma), dx, bc, gamma))
    return U


def exact(case, seed):
    if case["kind"] != "run":
        vl2 = case.get("integ", "heun") == "vl2"
        every = 4 if case["kind"] == "batch" else 1  # a quarter of a batch, in the interest of time
        out = []
        for i, (W, (n, _, gamma, cfl, _)) in enumerate(zip(_member_inputs(case, seed), _members(case))):
            out.append(_advance(W, [1.0 / v for v in n], "periodic", gamma, cfl, case["steps"], vl2)
                       if i % every == 0 else None)
        return out if case["kind"] == "batch" else {"state": out, "steps": None, "flags": None}
    if case["refine"]:
        return None
    n = _dims(case)
    nd, hi = len(n), _box(n)
    dx = [hi[d] / n[d] for d in range(nd)]
    U = _advance(_inputs(case, seed), dx, case["bc"], case["gamma"], 0.3 if nd == 3 else 0.4, case["steps"],
                 case["integ"] == "vl2")
    totals = U.reshape(nd + 2, -1).sum(1).cpu().numpy() * math.prod(dx)
    b = case["blocks"]
    if b > 1:
        s = U.shape
        parts = [b if d < nd else 1 for d in (2, 1, 0)]
        U = U.reshape(nd + 2, parts[0], s[1] // parts[0], parts[1], s[2] // parts[1], parts[2], s[3] // parts[2])
        U = U.permute(1, 3, 5, 0, 2, 4, 6).reshape(-1, nd + 2, *U.shape[2:7:2])
    return {"state": U, "totals": totals} if case["dt"] == "host" else U
