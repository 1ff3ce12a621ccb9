"""Performance cases: calls that a program using this framework makes, through
the public entry points of ``paper_2101_05886_amd.fp``.

Every case is a dict of plain values.  ``prepare`` makes what a program holds
before the call (grid, metrics, state, workspace, batch handle) on the GPU from
a seed; ``run`` is one pass; ``work`` its compulsory bytes and operations;
``exact`` the same result from plain torch in 64 bits.

Kinds of call:
  solve     fp.solve: RK3 steps replayed from the captured step graph
  step      fp.rk3_step: one step, for a program with its own time loop
  residual  fp.residual: dQ/dt alone, for a program with its own integrator
  ns        fp.solve_ns: Navier-Stokes steps
  bcs       fp.solve_bcs: the double Mach reflection with its boundary faces
  batch     fp.Batch.solve: blocks of uneven sizes advanced together
  setup     fp.metrics, fp.max_dt and fp.check_state of a new block, which
            every run and every serving request starts with
"""
import math
import random

import numpy as np
import torch

from paper_2101_05886_amd import fp

GAMMA = 1.4
DEV = "cuda"
F64 = torch.float64


def _case(name, kind, n, recon="weno5", Y=6, prec="fp64", grid="wavy", steps=1, blocks=0, jitter=0.05, mach=0.8):
    n = list(n) + [1] * (3 - len(n))
    return {"name": name, "kind": kind, "n0": n[0], "n1": n[1], "n2": n[2], "recon": recon, "Y": Y, "prec": prec,
            "grid": grid, "steps": steps, "blocks": blocks, "jitter": jitter, "mach": mach}


def listed():
    return [
        # the smallest runs: a 2D grid of 64^2, ten steps per call (4096 nodes: launches and latency)
        _case("solve-2d-64x64-m2", "solve", (64, 64), Y=2, steps=10, mach=0.5),
        # a small odd-sized 3D body-fitted block in a program with its own integrator
        _case("residual-3d-45x33x29-m4", "residual", (45, 33, 29), Y=4, grid="ogrid", mach=2.0),
        # accuracy studies with the linear upwind scheme: 128^3 vortex, sixth-order metrics
        _case("solve-128-linup5", "solve", (128, 128, 128), recon="linup5", steps=2, jitter=0.0, mach=0.5),
        # the standard single-block production run, 64-bit
        _case("solve-256-weno5", "solve", (256, 256, 256)),
        # the same with the 32-bit reconstruction
        _case("solve-256-weno5-mixed", "solve", (256, 256, 256), prec="mixed"),
        # the wide-stencil scheme (ghost 4, eighth-order metrics), odd extents, own time loop
        _case("step-191x161x133-weno7-m8-mixed", "step", (191, 161, 133), recon="weno7", Y=8, prec="mixed"),
        # the adaptive central-upwind scheme on a body-fitted block with odd extents, 64-bit
        _case("step-145x113x97-wenocu6", "step", (145, 113, 97), recon="wenocu6", grid="ogrid", mach=2.0),
        # a shock problem in 2D with global Lax-Friedrichs speeds and boundary faces
        _case("dmr-961x241", "bcs", (961, 241), steps=5, grid="dmr"),
        # a viscous run
        _case("ns-160", "ns", (160, 160, 160)),
        # a multi-block grid around a body, 48 uneven blocks of 20 million nodes
        _case("batch-48-ogrid-mixed", "batch", (0, 0, 0), prec="mixed", grid="ogrid", steps=2, blocks=48, mach=3.0),
        # one round of a serving loop: 24 requests, 2D and 3D, five steps each
        _case("batch-24-serving-mixed", "batch", (0, 0, 0), prec="mixed", grid="serving", steps=5, blocks=24),
        # the start of a run or a serving request
        _case("setup-160x144x150", "setup", (160, 144, 150)),
    ]


def _extents(rng, ndim, lo, hi):
    """extents of a block of about 10^U(lo, hi) nodes, each axis off the cube by up to 1.5x"""
    side = (10.0 ** rng.uniform(lo, hi)) ** (1.0 / ndim)
    return [max(12, int(round(side * 1.5 ** rng.uniform(-1, 1)))) for _ in range(ndim)]


def draw(rng: random.Random):
    kind = rng.choice(["solve", "solve", "step", "step", "residual", "ns", "bcs", "batch", "setup"])
    recon = rng.choice(["weno5", "weno5", "linup5", "weno7", "wenocu6"])
    Y = rng.choice([2, 4, 6, 6, 6, 8])
    prec = rng.choice(["fp64", "mixed"])
    grid = rng.choice(["wavy", "ogrid"])
    mach = round(rng.uniform(0.3, 2.0), 2)
    ndim = rng.choice([2, 3, 3])
    if kind == "bcs":
        ny = int(round(10 ** rng.uniform(math.log10(60), math.log10(241))))
        c = _case("", "bcs", (4 * (ny - 1) + 1, ny), Y=rng.choice([4, 6]), steps=rng.randint(1, 5), grid="dmr")
    elif kind == "batch":
        blocks = rng.randint(3, 40)
        c = _case("", "batch", (0, 0, 0), prec=prec, grid=rng.choice(["ogrid", "serving"]), blocks=blocks,
                  steps=1 if blocks > 20 else 2, mach=mach)
    elif kind == "ns":
        n = _extents(rng, ndim, 3.6, 6.6)
        c = _case("", "ns", n, recon=rng.choice(["weno5", "linup5"]), Y=rng.choice([4, 6]), mach=mach)
    elif kind == "setup":
        c = _case("", "setup", _extents(rng, ndim, 3.6, 6.5 if ndim == 3 else 6.0), Y=Y, grid=grid, mach=mach)
    elif kind == "residual":
        # a 32-bit reconstruction goes through the steps: a lone residual is asked for in 64 bits
        c = _case("", "residual", _extents(rng, ndim, 3.6, 6.8 if ndim == 3 else 6.0), recon=recon, Y=Y, grid=grid,
                  mach=mach)
    else:
        n = _extents(rng, ndim, 4.7 if ndim == 3 and prec == "mixed" else 4.0, 6.8 if ndim == 3 else 6.0)
        c = _case("", kind, n, recon=recon, Y=Y, prec=prec, grid=grid,
                  steps=rng.randint(1, 4) if kind == "solve" and prec == "fp64" else 1, mach=mach)
    del c["name"]
    return c


# --------------------------------------------------------------------------
# grids and states (torch, on the GPU, from a seed)
# --------------------------------------------------------------------------

def _ndim(c):
    return 2 if c["n2"] == 1 else 3


def _ghost(c):
    return 4 if c["recon"] == "weno7" or c["Y"] == 8 else 3


def _axes(n, gc):
    return [torch.arange(-gc, m + gc, dtype=F64, device=DEV) for m in n]


def _shape(v, d, ndim):
    """a vector along axis d of an array whose last axis is axis 0"""
    s = [1] * ndim
    s[ndim - 1 - d] = -1
    return v.reshape(s)


def _wavy(n, gc, L, jitter, gen):
    """periodic wavy grid (amplitude 0.1 of the shortest axis) with nodes jittered in random directions"""
    ndim = len(n)
    h = L / n[0]
    lens = [h * m for m in n]
    ax = [_shape(a * h - ln / 2, d, ndim) for d, (a, ln) in enumerate(zip(_axes(n, gc), lens))]
    P = 0.1 * min(lens)
    for x, ln in zip(ax, lens):
        P = P * torch.sin(2 * math.pi * (x + ln / 2) / ln)
    xyz = torch.stack([(x + P).expand(P.shape) for x in ax])
    if jitter:
        v = torch.randn((ndim, *reversed(n)), dtype=F64, device=DEV, generator=gen)
        v = v / v.norm(dim=0) * (jitter * h)
        for d, m in enumerate(n):
            v = v.index_select(ndim - d, torch.arange(-gc, m + gc, device=DEV) % m)
        xyz = xyz + v
    return xyz.contiguous(), lens


def _ogrid(n, gc, sector, skew, rot):
    """a sector of an O-grid around a cylinder of radius 1 (index 1 outward, first spacing 0.01 growing by 1.1)"""
    ndim = len(n)
    dth = sector / n[0]
    jj = np.arange(-gc, n[1] + gc)
    steps = np.concatenate([[0.0], np.cumsum(0.01 * 1.1 ** np.minimum(np.arange(n[1] + gc), 48))])
    r = torch.tensor(np.where(jj >= 0, 1.0 + steps[np.maximum(jj, 0)], 1.0 + jj * 0.01), dtype=F64, device=DEV)
    ax = _axes(n, gc)
    r = _shape(r, 1, ndim)
    th = 0.5 * sector - _shape(ax[0], 0, ndim) * dth + math.tan(skew) * (r - 1.0) / r + rot
    xyz = [r * torch.cos(th), r * torch.sin(th)]
    if ndim == 3:
        z = _shape(ax[2], 2, 3) * dth
        full = torch.broadcast_shapes(xyz[0].shape, z.shape)
        xyz = [x.expand(full) for x in xyz] + [z.expand(full)]
    return torch.stack(xyz).contiguous()


def _conserved(rho, vel, p):
    ke = sum(v * v for v in vel)
    return torch.stack([rho] + [rho * v for v in vel] + [p / (GAMMA - 1) + 0.5 * rho * ke]).contiguous()


def _nodes(xyz, Y):
    h = Y // 2
    return xyz[(slice(None),) + (slice(h, -h),) * (xyz.dim() - 1)]


def _vortex(x, lens, center, vel):
    """isentropic vortex column (strength 5, radius 1) on a uniform flow (rho 1.4, p 1), nearest periodic image"""
    eps, alpha = 5.0 / (2 * math.pi), 0.5
    dx, dy = x[0] - center[0], x[1] - center[1]
    dx, dy = dx - lens[0] * torch.round(dx / lens[0]), dy - lens[1] * torch.round(dy / lens[1])
    ex = torch.exp(alpha * (1.0 - dx * dx - dy * dy))
    T0 = 1.0 / GAMMA
    T = T0 - (GAMMA - 1) * eps ** 2 / (4 * alpha * GAMMA) * ex * ex
    rho = GAMMA * (T / T0) ** (1 / (GAMMA - 1))
    u = [vel[0] + eps * ex * dy, vel[1] - eps * ex * dx] + [torch.full_like(dx, w) for w in vel[2:len(x)]]
    return _conserved(rho, u, rho * T)


def _free_stream_bump(x, mach, gen):
    """uniform flow along x with a 5% density and energy bump near the body and 0.1% noise"""
    bump = 0.05 * torch.exp(-((x[0] - 1.2) ** 2 + (x[1] - 0.4) ** 2) / 0.25)
    noise = 1e-3 * (2 * torch.rand(x[0].shape, dtype=F64, device=DEV, generator=gen) - 1)
    f = 1 + bump + noise
    u = [torch.full_like(f, mach)] + [torch.zeros_like(f) for _ in range(len(x) - 1)]
    return _conserved(GAMMA * f, u, f)


def _block(n, c, rnd, gen):
    """(xyz, state) of one block of extents n"""
    g, Y, ndim = _ghost(c), c["Y"], len(n)
    gc = g + Y // 2
    if c["grid"] == "ogrid":
        xyz = _ogrid(n, gc, rnd.uniform(math.pi / 3, math.pi), math.radians(rnd.uniform(0, 30)), rnd.uniform(0, 6.28))
        return xyz, _free_stream_bump(_nodes(xyz, Y), c["mach"], gen)
    xyz, lens = _wavy(n, gc, 12.0 if ndim == 3 else 20.0, c["jitter"], gen)
    th, ph = math.radians(rnd.uniform(5, 30)), math.radians(rnd.uniform(5, 15)) if ndim == 3 else 0.0
    vel = [c["mach"] * v for v in (math.cos(th) * math.cos(ph), math.sin(th) * math.cos(ph), math.sin(ph))]
    center = [rnd.uniform(-0.3, 0.3) * ln for ln in lens[:2]]
    return xyz, _vortex(_nodes(xyz, Y), lens, center, vel)


# the double Mach reflection on [0, 4] x [0, 1]: Mach 10 shock at 60 degrees
DMR_PRE, DMR_POST = (1.4, 0.0, 0.0, 1.0), (8.0, 7.1447, -4.125, 116.5)
DMR_X0, DMR_SPEED = 1.0 / 6.0, 10.0
DMR_NORMAL = (math.cos(math.pi / 6), -math.sin(math.pi / 6))


def _prim_to_cons(s):
    rho, u, v, p = s
    return [rho, rho * u, rho * v, p / (GAMMA - 1) + 0.5 * rho * (u * u + v * v)]


def _dmr(c, gen):
    """grid (5% random), state and boundary faces of the double Mach reflection"""
    nx, ny, g, Y = c["n0"], c["n1"], _ghost(c), c["Y"]
    gc = g + Y // 2
    hx, hy = 4.0 / (nx - 1), 1.0 / (ny - 1)
    phi = torch.rand((ny, nx), dtype=F64, device=DEV, generator=gen)
    dx, dy = 0.05 * hx * phi, 0.05 * hy * torch.sqrt(1 - phi * phi)
    dx[:, [0, -1]] = 0.0
    dy[[0, -1], :] = 0.0
    X = torch.zeros((2, ny + 2 * gc, nx + 2 * gc), dtype=F64, device=DEV)
    X[0, gc:gc + ny, gc:gc + nx] = torch.arange(nx, dtype=F64, device=DEV)[None, :] * hx + dx
    X[1, gc:gc + ny, gc:gc + nx] = torch.arange(ny, dtype=F64, device=DEV)[:, None] * hy + dy
    r, t = gc + nx - 1, gc + ny - 1
    for m in range(1, gc + 1):  # sides: point reflection through the boundary nodes
        X[:, :, gc - m] = 2 * X[:, :, gc] - X[:, :, gc + m]
        X[:, :, r + m] = 2 * X[:, :, r] - X[:, :, r - m]
    for m in range(1, gc + 1):  # bottom: mirror image; top: point reflection
        X[0, gc - m], X[1, gc - m] = X[0, gc + m], -X[1, gc + m]
        X[:, t + m] = 2 * X[:, t] - X[:, t - m]
    x = _nodes(X, Y).contiguous()
    post = x[0] - x[1] * math.tan(math.pi / 6) < DMR_X0
    post[:g] = x[0, :g] < DMR_X0
    a, b = (torch.tensor(_prim_to_cons(s), dtype=F64, device=DEV)[:, None, None] for s in (DMR_POST, DMR_PRE))
    q = torch.where(post[None], a, b).contiguous()
    mask = (x[0, g, g:-g] >= DMR_X0).to(torch.uint8).contiguous()
    return X, x, q, mask


def _extents_of_batch(c, rnd):
    out = []
    for i in range(c["blocks"]):
        if c["grid"] == "ogrid":
            out.append([rnd.randint(32, 192), rnd.randint(32, 128), rnd.randint(16, 64)])
        else:  # serving: 2D from 64^2, 3D to about 64^3, log-uniform nodes
            ndim = 2 + i % 2
            out.append(_extents(rnd, ndim, 3.6, 5.4))
    return out


# --------------------------------------------------------------------------
# prepare and run
# --------------------------------------------------------------------------

def _grid_of(n, c, g):
    frozen = c["grid"] in ("ogrid", "dmr")
    return fp.Grid(len(n), n, g, bc=[fp.FP_BC_FROZEN if frozen else fp.FP_BC_PERIODIC] * 3)


def _scheme(c):
    return fp.Scheme(c["recon"], c["Y"], True, precision=c["prec"], splitting="glf" if c["kind"] == "bcs" else "llf",
                     mu=1e-3 if c["kind"] == "ns" else 0.0)


def _seeded(case, seed):
    return random.Random(seed), torch.Generator(device=DEV).manual_seed(seed)


def _inputs(case, seed):
    """[(n, xyz, q)] of the case's blocks (and the rest of the double Mach reflection)"""
    rnd, gen = _seeded(case, seed)
    if case["kind"] == "bcs":
        X, x, q, mask = _dmr(case, gen)
        return [([case["n0"], case["n1"]], X, q)], (x, mask)
    if case["kind"] == "batch":
        sizes = _extents_of_batch(case, random.Random(case["blocks"]))  # one block list, other grids and states by seed
        out = []
        for i, n in enumerate(sizes):
            c = dict(case, grid="ogrid" if case["grid"] == "ogrid" or i % 3 == 2 else "wavy")
            out.append((n, *_block(n, c, rnd, gen), c))
        return out, None
    n = [case["n0"], case["n1"], case["n2"]][:_ndim(case)]
    return [(n, *_block(n, case, rnd, gen))], None


def prepare(case, seed):
    blocks, more = _inputs(case, seed)
    sc, g, Y, kind = _scheme(case), _ghost(case), case["Y"], case["kind"]
    if kind == "setup":
        n, xyz, q = blocks[0]
        return {"kind": kind, "g": _grid_of(n, case, g), "sc": sc, "xyz": xyz, "q": q, "Y": Y,
                "met": torch.zeros(fp.Grid(len(n), n, g).metric_shape(), dtype=F64, device=DEV)}
    if kind == "batch":
        s = {"kind": kind, "steps": case["steps"], "batch": fp.Batch(sc, case["blocks"])}
        held = []
        for n, xyz, q, c in blocks:
            grid = _grid_of(n, c, g)
            met = fp.metrics(grid, Y, xyz)
            held.append([grid, met, q, torch.zeros(grid.work_shape(), dtype=F64, device=DEV),
                         fp.max_dt(grid, sc, met, q, 0.5)])
        dts = torch.cat([h[4] for h in held]).tolist()
        s["blocks"] = [(*h[:4], dt) for h, dt in zip(held, dts)]
        s["batch"].set(s["blocks"])
        s["batch"].autotune()
        s["q"] = [h[2] for h in held]
        return s
    n, xyz, q = blocks[0]
    grid = _grid_of(n, case, g)
    met = fp.metrics(grid, Y, xyz)
    s = {"kind": kind, "g": grid, "sc": sc, "met": met, "q": q, "steps": case["steps"]}
    if kind == "residual":
        s["dqdt"] = torch.zeros_like(q)
        return s
    s["work"] = torch.zeros(grid.work_shape(), dtype=F64, device=DEV)
    if kind == "bcs":
        x, mask = more
        s["bcs"] = fp.Bcs([[fp.FP_FACE_HOLD, fp.FP_FACE_EXTRAP], [fp.FP_FACE_WALL, fp.FP_FACE_SHOCK]],
                          mask={(1, 0): mask}, nodes=x, pre=_prim_to_cons(DMR_PRE), post=_prim_to_cons(DMR_POST),
                          normal=(*DMR_NORMAL, 0.0), offset=DMR_NORMAL[0] * DMR_X0, speed=DMR_SPEED)
        s["t"], s["q0"] = 0.0, q.clone()
        s["dt"] = float(fp.max_dt(grid, sc, met, q, 0.6).item())
        return s
    s["dt"] = float(fp.max_dt(grid, sc, met, q, 0.5).item())
    if kind == "ns":
        s["vwork"] = fp.viscous_work(grid)
    return s


def run(s):
    kind = s["kind"]
    if kind == "solve":
        return fp.solve(s["g"], s["sc"], s["met"], s["q"], s["work"], s["dt"], s["steps"])
    if kind == "step":
        return fp.rk3_step(s["g"], s["sc"], s["met"], s["q"], s["work"], s["dt"])
    if kind == "residual":
        return fp.residual(s["g"], s["sc"], s["met"], s["q"], s["dqdt"])
    if kind == "ns":
        return fp.solve_ns(s["g"], s["sc"], s["met"], s["q"], s["work"], s["vwork"], s["dt"], s["steps"])
    if kind == "bcs":
        if s["t"] >= 0.2:  # the problem's end time: start again
            s["q"].copy_(s["q0"])
            s["t"] = 0.0
        fp.solve_bcs(s["g"], s["sc"], s["bcs"], s["met"], s["q"], s["work"], s["t"], s["dt"], s["steps"])
        s["t"] += s["steps"] * s["dt"]
        return s["q"]
    if kind == "batch":
        s["batch"].solve(s["steps"])
        return s["q"]
    met = fp.metrics(s["g"], s["Y"], s["xyz"], s["met"])
    return {"met": met, "dt": fp.max_dt(s["g"], s["sc"], met, s["q"], 0.5), "bad": fp.check_state(s["g"], s["sc"], s["q"])}


def _face_flops(recon, D, Y):
    """operations of one face flux of the method (add, mul, div, sqrt = 1): reference state, subtraction,
    characteristic system, two projections per stencil node, splitting, reconstructions, back-projection"""
    nv, S = D + 2, 8 if recon == "weno7" else 6
    tang = 29 if D == 3 else 3
    ref = 2 * Y * (1 + D) + 3 * Y * nv + 9 * nv + 6
    node = (2 * nv + 12 * D + 10) * S
    eig = 14 * D + 22 + 2 * D - 1 + tang + (2 * D + 9) * S
    proj = 2 * (2 * D - 1) + (D - 1) * (2 * D - 1) + 12 + 2 * (D - 1)
    back = 35 if D == 3 else 24
    if recon == "linup5":
        return ref + node + eig + nv * 25 + proj + back + 2 * nv
    return ref + node + eig + 2 * S * proj + 4 * nv * S + 2 * nv * {"weno5": 60, "weno7": 150, "wenocu6": 155}[recon] + back


def work(case):
    """Bytes: per evaluation of the residual the state and the metrics read and a state written (a stage depends on
    the whole stage before it, so each stage is a pass of its own)."""
    sizes = (_extents_of_batch(case, random.Random(case["blocks"])) if case["kind"] == "batch"
             else [[case["n0"], case["n1"], case["n2"]][:_ndim(case)]])
    byts = flops = 0.0
    for n in sizes:
        D = len(n)
        nodes = float(math.prod(n))
        if case["kind"] == "setup":  # coordinates and state in, metrics out; the symmetric metrics' differences
            byts += 8 * nodes * (D + (D + 2) + (10 if D == 3 else 5))
            flops += nodes * ((18 * 3 + 9 * 2) * case["Y"] if D == 3 else 10 * case["Y"])
            continue
        evals = 1 if case["kind"] == "residual" else 3 * case["steps"]
        byts += evals * 8 * nodes * (2 * (D + 2) + (10 if D == 3 else 5))
        faces = sum(nodes / m * (m + 1) for m in n)
        flops += evals * faces * _face_flops(case["recon"], D, case["Y"])
        if case["kind"] == "ns":
            flops += evals * nodes * (12 * D * (D + 1) * 2 + 120)
    return {"bytes": byts, "flops": flops}


# --------------------------------------------------------------------------
# the same results from plain torch in 64 bits
# --------------------------------------------------------------------------

FACE = {2: [0, 0, 0, 1 / 2, 1 / 2, 0, 0, 0], 4: [0, 0, -1 / 12, 7 / 12, 7 / 12, -1 / 12, 0, 0],
        6: [0, 1 / 60, -8 / 60, 37 / 60, 37 / 60, -8 / 60, 1 / 60, 0],
        8: [v / 840 for v in (-3, 29, -139, 533, 533, -139, 29, -3)]}
DERIV = {2: [1 / 2], 4: [8 / 12, -1 / 12], 6: [45 / 60, -9 / 60, 1 / 60], 8: [672 / 840, -168 / 840, 32 / 840, -3 / 840]}


def _D(f, axis, Y):
    """central difference along the array axis (wrapping: outer layers are cut off by the caller)"""
    return sum(c * (torch.roll(f, -m, axis) - torch.roll(f, m, axis)) for m, c in enumerate(DERIV[Y], 1))


def _metrics_exact(xyz, Y):
    ndim, h = xyz.shape[0], Y // 2
    X = list(xyz)
    ax = [ndim - 1 - d for d in range(ndim)]
    if ndim == 2:
        xx, xe, yx, ye = (_D(X[c], ax[e], Y) for c in (0, 1) for e in (0, 1))
        J = 0.5 * (_D(X[0] * ye - X[1] * xe, ax[0], Y) + _D(X[1] * xx - X[0] * yx, ax[1], Y))
        out = [ye, -xe, -yx, xx, J]
    else:
        out = []
        for d in range(3):
            e, f = (d + 1) % 3, (d + 2) % 3
            for c in range(3):
                a, b = X[(c + 1) % 3], X[(c + 2) % 3]
                Pe = _D(a, ax[e], Y) * b - a * _D(b, ax[e], Y)
                Pf = _D(a, ax[f], Y) * b - a * _D(b, ax[f], Y)
                out.append(0.5 * (_D(Pe, ax[f], Y) - _D(Pf, ax[e], Y)))
        out.append(sum(_D(sum(X[c] * out[3 * d + c] for c in range(3)), ax[d], Y) for d in range(3)) / 3)
    cut = (slice(h, -h),) * ndim
    return torch.stack([o[cut] for o in out])


def _lines(a, d, g, n, periodic):
    """interior lines along axis d with their ghost layers, the line axis last"""
    ndim = a.dim() - 1
    for e in range(ndim):
        if e != d:
            a = a.narrow(ndim - e, g, n[e])
    if periodic:
        a = a.index_select(ndim - d, torch.arange(-g, n[d] + g, device=a.device) % n[d] + g)
    return a.movedim(ndim - d, -1)


def _weno5(a, b, c, d, e, eps):
    q = [(2 * a - 7 * b + 11 * c) / 6, (-b + 5 * c + 2 * d) / 6, (2 * c + 5 * d - e) / 6]
    s = [13 / 12 * (a - 2 * b + c) ** 2 + (a - 4 * b + 3 * c) ** 2 / 4, 13 / 12 * (b - 2 * c + d) ** 2 + (b - d) ** 2 / 4,
         13 / 12 * (c - 2 * d + e) ** 2 + (3 * c - 4 * d + e) ** 2 / 4]
    al = [w / (x + eps) ** 2 for w, x in zip((0.1, 0.6, 0.3), s)]
    return sum(w * x for w, x in zip(al, q)) / sum(al)


def _weno7(v, eps):
    a, b, c, d, e, f, g = v
    q = [(-3 * a + 13 * b - 23 * c + 25 * d) / 12, (b - 5 * c + 13 * d + 3 * e) / 12, (-c + 7 * d + 7 * e - f) / 12,
         (3 * d + 13 * e - 5 * f + g) / 12]
    s = [a * (547 * a - 3882 * b + 4642 * c - 1854 * d) + b * (7043 * b - 17246 * c + 7042 * d)
         + c * (11003 * c - 9402 * d) + 2107 * d * d,
         b * (267 * b - 1642 * c + 1602 * d - 494 * e) + c * (2843 * c - 5966 * d + 1922 * e)
         + d * (3443 * d - 2522 * e) + 547 * e * e,
         c * (547 * c - 2522 * d + 1922 * e - 494 * f) + d * (3443 * d - 5966 * e + 1602 * f)
         + e * (2843 * e - 1642 * f) + 267 * f * f,
         d * (2107 * d - 9402 * e + 7042 * f - 1854 * g) + e * (11003 * e - 17246 * f + 4642 * g)
         + f * (7043 * f - 3882 * g) + 547 * g * g]
    al = [w / (x + eps) ** 2 for w, x in zip((1, 12, 18, 4), s)]
    return sum(w * x for w, x in zip(al, q)) / sum(al)


def _beta6_factor():
    """rows l of B with sum_l (B v)_l^2 the Jiang-Shu measure of the quintic with cell averages v over cell 2"""
    A = np.array([[((j + 0.5) ** (k + 1) - (j - 0.5) ** (k + 1)) / (k + 1) for k in range(6)] for j in range(-2, 4)])
    M = np.zeros((6, 6))
    for order in range(1, 6):
        co = [math.prod(range(k - order + 1, k + 1)) if k >= order else 0 for k in range(6)]
        for k in range(order, 6):
            for m in range(order, 6):
                p = k + m - 2 * order
                M[k, m] += co[k] * co[m] * (2 * 0.5 ** (p + 1) / (p + 1) if p % 2 == 0 else 0.0)
    return np.linalg.cholesky(M[1:, 1:]).T @ np.linalg.inv(A)[1:]


def _wenocu6(v, eps):
    a, b, c, d, e, f = v
    q = [(2 * a - 7 * b + 11 * c) / 6, (-b + 5 * c + 2 * d) / 6, (2 * c + 5 * d - e) / 6, (11 * d - 7 * e + 2 * f) / 6]
    s = [13 / 12 * (a - 2 * b + c) ** 2 + (a - 4 * b + 3 * c) ** 2 / 4, 13 / 12 * (b - 2 * c + d) ** 2 + (b - d) ** 2 / 4,
         13 / 12 * (c - 2 * d + e) ** 2 + (3 * c - 4 * d + e) ** 2 / 4]
    s.append(sum(sum(float(w) * (x - c) for w, x in zip(row, v)) ** 2 for row in _beta6_factor()))
    tau = s[3] - (s[0] + 4 * s[1] + s[2]) / 6
    al = [w * (20 + tau / (x + eps)) ** 2 for w, x in zip((1, 9, 9, 1), s)]
    return sum(w * x for w, x in zip(al, q)) / sum(al)


def _speed(u, p, rho, n):
    un = sum(a * b for a, b in zip(n, u))
    return un, torch.sqrt(GAMMA * p / rho)


def _fluxes(q, s, V, g, n, recon, Y, glf, eps=1e-6):
    """face fluxes F'_{f+1/2}, f = -1 .. n - 1, of lines along the last axis"""
    D, E = len(s), len(s) + 1
    at = lambda x, r: x[..., g - 4 + r:g - 3 + r + n]  # noqa: E731
    wt = [(r, w) for r, w in enumerate(FACE[Y]) if w]
    Vf = sum(w * at(V, r) for r, w in wt)
    sf = [sum(w * at(x, r) for r, w in wt) for x in s]
    Qs = [sum(w * at(x, r) * at(V, r) for r, w in wt) / Vf for x in q]
    prim = lambda w: ([w[1 + c] / w[0] for c in range(D)],  # noqa: E731
                      (GAMMA - 1) * (w[E] - 0.5 * sum(w[1 + c] ** 2 for c in range(D)) / w[0]))

    def flux(w, u, p, sv):
        U = sum(a * b for a, b in zip(u, sv))
        return [w[0] * U] + [w[1 + c] * U + p * sv[c] for c in range(D)] + [(w[E] + p) * U]

    us, ps = prim(Qs)
    Fs = flux(Qs, us, ps, sf)
    sn = torch.sqrt(sum(x * x for x in sf))
    nv = [x / sn for x in sf]
    sig = sn / Vf
    L, R = [at(x, 3) for x in q], [at(x, 4) for x in q]
    (uL, pL), (uR, pR) = prim(L), prim(R)
    wL, wR = torch.sqrt(L[0]), torch.sqrt(R[0])
    mean = lambda x, y: (wL * x + wR * y) / (wL + wR)  # noqa: E731
    uh = [mean(x, y) for x, y in zip(uL, uR)]
    H = mean((L[E] + pL) / L[0], (R[E] + pR) / R[0])
    k2 = sum(x * x for x in uh)
    c2 = (GAMMA - 1) * (H - 0.5 * k2)
    ch, un = torch.sqrt(c2), sum(a * b for a, b in zip(nv, uh))
    if D == 2:
        T = [[-nv[1], nv[0]]]
    else:
        m = [x.abs() for x in nv]
        one = m[1] < m[0] - 1e-10
        two = m[2] < torch.where(one, m[1], m[0]) - 1e-10
        one = one & ~two
        z = torch.zeros_like(nv[0])
        pick = lambda a0, a1, a2: torch.where(two, a2, torch.where(one, a1, a0))  # noqa: E731
        t = [pick(z, -nv[2], nv[1]), pick(nv[2], z, -nv[0]), pick(-nv[1], nv[0], z)]
        ln = torch.sqrt(sum(x * x for x in t))
        t = [x / ln for x in t]
        T = [t, [nv[1] * t[2] - nv[2] * t[1], nv[2] * t[0] - nv[0] * t[2], nv[0] * t[1] - nv[1] * t[0]]]
    ut = [sum(a * b for a, b in zip(t, uh)) for t in T]

    def left(w):
        phi = (GAMMA - 1) / c2 * (0.5 * k2 * w[0] - sum(uh[c] * w[1 + c] for c in range(D)) + w[E])
        psi = (sum(nv[c] * w[1 + c] for c in range(D)) - un * w[0]) / ch
        return [0.5 * (phi - psi), w[0] - phi] + [sum(t[c] * w[1 + c] for c in range(D)) - x * w[0]
                                                  for t, x in zip(T, ut)] + [0.5 * (phi + psi)]

    slots = range(0, 8) if recon == "weno7" else range(1, 7)
    a, b, lam = [], [], [torch.zeros_like(un) for _ in range(3)]
    for r in slots:
        w, sv, Vr = [at(x, r) for x in q], [at(x, r) for x in s], at(V, r)
        u, p = prim(w)
        dF = [x - y for x, y in zip(flux(w, u, p, sv), flux(Qs, us, ps, sv))]
        a.append(left(dF))
        b.append(left([(x - y) * Vr for x, y in zip(w, Qs)]))
        vn, cs = _speed(u, p, w[0], nv)
        lam = [torch.maximum(x, (vn + k * cs).abs()) for x, k in zip(lam, (-1, 0, 1))]
    lam = [sig * x for x in lam]
    if glf:
        lam = [x.max() for x in lam]
    lam = [lam[0]] + [lam[1]] * D + [lam[2]]
    h = []
    for v in range(E + 1):
        plus = [0.5 * (x[v] + lam[v] * y[v]) for x, y in zip(a, b)]
        minus = [0.5 * (x[v] - lam[v] * y[v]) for x, y in zip(a, b)][::-1]
        if recon == "weno5":
            h.append(_weno5(*plus[:5], eps) + _weno5(*minus[:5], eps))
        elif recon == "weno7":
            h.append(_weno7(plus[:7], eps) + _weno7(minus[:7], eps))
        elif recon == "wenocu6":
            h.append(_wenocu6(plus, eps) + _wenocu6(minus, eps))
        else:
            up = (2 / 60, -13 / 60, 47 / 60, 27 / 60, -3 / 60)
            h.append(sum(k * x for k, x in zip(up, plus)) + sum(k * x for k, x in zip(up, minus)))
    h0, h1, hE, ht = h[0], h[1], h[E], h[2:E]
    o = [h0 + h1 + hE]
    o += [uh[c] * o[0] + ch * nv[c] * (hE - h0) + sum(t[c] * x for t, x in zip(T, ht)) for c in range(D)]
    o.append(H * (h0 + hE) + ch * un * (hE - h0) + 0.5 * k2 * h1 + sum(x * y for x, y in zip(ut, ht)))
    return [x + y for x, y in zip(Fs, o)]


def _viscous(q, met, mu, prandtl=0.72):
    """J sum_d D6_d(Fv_d) on the interior of a periodic block"""
    D = len(q) - 2
    ax = [D - 1 - d for d in range(D)]
    V = met[-1]
    u = [q[1 + c] / q[0] for c in range(D)]
    T = (GAMMA - 1) * (q[-1] - 0.5 * sum(q[1 + c] * u[c] for c in range(D))) / q[0]
    s = [[met[D * d + j] for j in range(D)] for d in range(D)]
    grad = []
    for f in u + [T]:
        df = [_D(f, ax[d], 6) for d in range(D)]
        grad.append([sum(s[d][j] * df[d] for d in range(D)) / V for j in range(D)])
    div = sum(grad[c][c] for c in range(D))
    kappa = mu * GAMMA / ((GAMMA - 1) * prandtl)
    F = []
    for j in range(D):
        tau = [mu * (grad[i][j] + grad[j][i] - (2 / 3 * div if i == j else 0.0)) for i in range(D)]
        F.append(tau + [sum(u[i] * tau[i] for i in range(D)) + kappa * grad[D][j]])
    out = [torch.zeros_like(V)]
    for v in range(D + 1):
        out.append(sum(_D(sum(s[d][j] * F[j][v] for j in range(D)), ax[d], 6) for d in range(D)) / V)
    return out


def _interior(a, g):
    return a[(slice(None),) + (slice(g, -g),) * (a.dim() - 1)]


def _rate(q, met, g, n, periodic, case):
    """dQ/dt on the interior"""
    D = len(n)
    total = [0.0] * (D + 2)
    for d in range(D):
        Q = _lines(q, d, g, n, periodic)
        s = _lines(met[D * d:D * d + D], d, g, n, False)
        V = _lines(met[-1:], d, g, n, False)[0]
        F = _fluxes(list(Q), list(s), V, g, n[d], case["recon"], case["Y"], case["kind"] == "bcs")
        for v in range(D + 2):
            total[v] = total[v] - (F[v][..., 1:] - F[v][..., :-1]).movedim(-1, D - 1 - d)
    inner = _interior(met, g)
    out = [t / inner[-1] for t in total]
    if case["kind"] == "ns":
        out = [x + y for x, y in zip(out, _viscous(list(_interior(q, g)), inner, 1e-3))]
    return torch.stack(out)


def _max_dt_exact(q, met, g, cfl):
    q, met = _interior(q, g), _interior(met, g)
    D = q.shape[0] - 2
    u = [q[1 + c] / q[0] for c in range(D)]
    c = torch.sqrt(GAMMA * (GAMMA - 1) * (q[-1] - 0.5 * sum(q[1 + i] * u[i] for i in range(D))) / q[0])
    rate = sum(sum(met[D * d + i] * u[i] for i in range(D)).abs()
               + c * torch.sqrt(sum(met[D * d + i] ** 2 for i in range(D))) for d in range(D)) / met[-1]
    return cfl / rate.max()


def _dmr_faces(q, met, x, mask, g, t):
    """ghost layers of the double Mach reflection at time t: outflow right, wall below (masked), shock above"""
    e = slice(g, -g)
    for m in range(1, g + 1):
        q[:, e, -g - 1 + m] = q[:, e, -g - 1]
    n = met[2:4, g, e]
    n = n / torch.sqrt((n * n).sum(0))
    keep = mask.bool()
    for m in range(1, g + 1):
        src = q[:, g + m, e].clone()
        src[1:3] -= 2 * (n * src[1:3]).sum(0) * n
        q[:, g - m, e] = torch.where(keep, src, q[:, g - m, e])
    post, pre = (torch.tensor(_prim_to_cons(w), dtype=F64, device=q.device)[:, None, None] for w in (DMR_POST, DMR_PRE))
    top = x[:, -g:, e]
    behind = DMR_NORMAL[0] * top[0] + DMR_NORMAL[1] * top[1] < DMR_NORMAL[0] * DMR_X0 + DMR_SPEED * t
    q[:, -g:, e] = torch.where(behind[None], post, pre)


def _steps_exact(q, met, g, n, periodic, case, dt, faces=None):
    q = q.clone()
    for i in range(case["steps"]):
        t = i * dt
        stage = q
        for a, b, ts in ((0.0, 1.0, t), (0.75, 0.25, t + dt), (1 / 3, 2 / 3, t + 0.5 * dt)):
            if faces:
                _dmr_faces(stage, met, *faces, g, ts)
            new = a * _interior(q, g) + b * (_interior(stage, g) + dt * _rate(stage, met, g, n, periodic, case))
            if stage is q:
                stage = q.clone()
            _interior(stage, g).copy_(new)
        _interior(q, g).copy_(_interior(stage, g))
    return q


def exact(case, seed):
    blocks, more = _inputs(case, seed)
    g, Y, kind = _ghost(case), case["Y"], case["kind"]
    if kind == "setup":
        n, xyz, q = blocks[0]
        met = _metrics_exact(xyz, Y)
        return {"met": met, "dt": _max_dt_exact(q, met, g, 0.5).reshape(1), "bad": None}
    out = []
    for blk in blocks:
        n, xyz, q = blk[:3]
        periodic = (blk[3] if len(blk) > 3 else case)["grid"] == "wavy"
        met = _metrics_exact(xyz, Y)
        if kind == "residual":
            dqdt = torch.zeros_like(q)
            _interior(dqdt, g).copy_(_rate(q, met, g, n, periodic, case))
            return dqdt
        dt = float(_max_dt_exact(q, met, g, 0.6 if kind == "bcs" else 0.5))
        out.append(_steps_exact(q, met, g, n, periodic, case, dt, more))
    return out if kind == "batch" else out[0]
