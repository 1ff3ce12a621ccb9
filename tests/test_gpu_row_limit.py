"""2D blocks on both sides of the line between the one-launch stage (1024 pieces
of a row of at most 56 nodes) and the two sweeps, with local and global
Lax-Friedrichs speeds and with viscous terms in the accumulator: bitwise the
instrumented step, which launches the two sweeps in any case, and the oracle's
step to 1e-12 per variable."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2101_05886_amd import fp
from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("recon,Y,n", [("weno5", 6, (20, 1024)), ("weno5", 6, (20, 1025)), ("weno5", 6, (113, 341)),
                                       ("weno5", 6, (113, 342)), ("weno7", 8, (57, 512)), ("weno7", 8, (57, 513)),
                                       ("linup5", 4, (56, 1024)), ("linup5", 4, (56, 1025))])
@pytest.mark.parametrize("kind", ["llf", "glf", "viscous"])
def test_one_launch_stage_at_its_limit(recon, Y, n, kind):
    case = G.periodic_case(2, n, Y, g=4, state="noisy", seed=41)
    mu = 1e-2 if kind == "viscous" else 0.0
    split = "glf" if kind == "glf" else "llf"
    og, fg = O.Grid(2, n, 4), fp.Grid(2, n, 4)
    met = O.metrics(og, Y, case["xyz"])
    sc = fp.Scheme(recon, Y, True, splitting=split, mu=mu)
    mg = torch.from_numpy(met).cuda()
    q1, q2 = torch.from_numpy(case["q"]).cuda(), torch.from_numpy(case["q"]).cuda()
    w1, w2 = (torch.zeros(fg.work_shape(), dtype=torch.float64, device="cuda") for _ in range(2))
    vw = fp.viscous_work(fg) if mu else None
    dt = 1e-3
    if mu:
        fp.solve_ns(fg, sc, mg, q1, w1, vw, dt, 1)
    else:
        fp.rk3_step(fg, sc, mg, q1, w1, dt)
    fp.profile_step(fg, sc, mg, q2, w2, dt, vwork=vw)
    assert torch.equal(q1, q2)
    ref = O.rk3_step(og, O.Scheme(recon, Y, True, splitting=split, mu=mu), met, case["q"], dt)
    got = q1.cpu().numpy()
    for v in range(4):
        assert np.abs(got[v] - ref[v]).max() <= 1e-12 * np.abs(ref[v]).max()
