"""The global Lax-Friedrichs speeds against their definition in extended
precision, from the stage inputs that a step leaves in the workspace.

Bar: 32 roundings (2^-47).  A face's metric vector and 1/J are sums of at most
eight products whose weights add up to below 2 (16 roundings of the larger
one), sigma and n are a root and three quotients of them, n . u three products.
A node of negative pressure has no sound speed: it counts for the class u_n
alone."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2101_05886_amd import fp
from tests import gpu_cases as G

pytestmark = pytest.mark.gpu
W = {2: [0.5], 4: [7 / 12, -1 / 12], 6: [37 / 60, -8 / 60, 1 / 60], 8: [533 / 840, -139 / 840, 29 / 840, -3 / 840]}
LD = np.longdouble


def speeds(ndim, met, q, g, Y, lo):
    """[direction][class] of a periodic block; met with ghosts, q interior"""
    with np.errstate(invalid="ignore"):
        u = q[1:1 + ndim] / q[0]
        p = LD(1.4 - 1.0) * (q[-1] - (q[1:1 + ndim] * u).sum(0) / 2)
        c = np.sqrt(LD(1.4) * p / q[0])
    out = np.zeros((ndim, 3), LD)
    for d in range(ndim):
        ax = ndim - d  # of an array [component][..., j, i]

        def at(o):  # metrics of node f + o for every face f + 1/2 right of an interior node
            sl = [slice(None)] + [slice(g, -g)] * ndim
            n = met.shape[ax]
            sl[ax] = slice(g + o, n - g + o)
            return met[tuple(sl)]

        m = sum(LD(W[Y][k]) * (at(-k) + at(1 + k)) for k in range(Y // 2))
        s = m[d * ndim:(d + 1) * ndim]
        sn = np.sqrt((s * s).sum(0))
        for r in range(-lo, lo + 2):
            un = (s / sn * np.roll(u, -r, axis=ax)).sum(0)
            cs = np.roll(c, -r, axis=ax - 1)
            for k, v in enumerate((un - cs, un, un + cs)):
                out[d, k] = max(out[d, k], np.nanmax(np.abs(v) * sn / m[-1]))
    return out


@pytest.mark.parametrize("negative", [False, True])
@pytest.mark.parametrize("recon,Y,g", [("weno5", 2, 3), ("linup5", 6, 3), ("weno7", 8, 4)])
@pytest.mark.parametrize("ndim,n", [(3, (21, 18, 11)), (2, (67, 35))])
def test_speeds_of_the_stage_inputs(ndim, n, recon, Y, g, negative):
    case = G.periodic_case(ndim, n, Y, g=g, state="noisy", seed=31)
    og, fg = O.Grid(ndim, n, g), fp.Grid(ndim, n, g)
    met = O.metrics(og, Y, case["xyz"])
    q = case["q"].copy()
    q3 = q.reshape((ndim + 2,) + tuple(q.shape[-ndim:]))
    if negative:  # the fastest node of the block, at a slightly negative pressure
        at = (slice(None),) + (g + 2,) * ndim
        q3[at] = [1.4] + [1.4 * 10.0] * ndim + [-0.01 / 0.4 + 0.7 * ndim * 10.0 ** 2]
    work = torch.zeros(fg.work_shape(), dtype=torch.float64, device="cuda")
    qg = torch.from_numpy(q).cuda()
    # a step this short leaves the state as it is: every stage input is q
    fp.rk3_step(fg, fp.Scheme(recon, Y, True, splitting="glf"), torch.from_numpy(met).cuda(), qg, work, 1e-300)
    w = work.cpu().numpy().ravel()
    elems = q.size
    inner = (slice(None),) + (slice(g, -g),) * ndim
    mets = met.reshape((-1,) + q3.shape[1:]).astype(LD)
    for stage in (1, 2):  # the first stage's set is cleared by the last stage
        x = w[(stage - 1) * elems:stage * elems].reshape(q3.shape)[inner]
        ref = speeds(ndim, mets, x.astype(LD), g, Y, 3 if recon == "weno7" else 2)
        for d in range(ndim):
            got = w[3 * elems + 48 * stage + 16 * d:][:3]
            assert (np.abs(got - ref[d]) <= 2.0 ** -47 * ref[d]).all(), (stage, d, got, ref[d])
