"""The small 2D block's stage, both sweeps in one launch, at the edges of its
tiles (56 nodes of a row, 256 workgroups) and beyond them: bitwise the two sweeps that
the instrumented step launches, and the FP64 oracle's step within the bar of
the other step tests (1e-12 per variable; FP32-mixed 1e-4 of the increment)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2101_05886_amd import fp
from paper_2101_05886_amd import inputs as I

pytestmark = pytest.mark.gpu

SIZES = [(3, 3), (55, 5), (56, 4), (57, 7), (64, 64), (112, 9), (113, 6), (20, 256), (20, 257)]


def case(n, g, Y, bc):
    xyz = I.wavy_grid(2, n, 10.0, g, Y, amp=0.05, jitter=0.03, seed=9)
    nodes = I.state_nodes(xyz, g, Y)
    per = I.wavy_periods(2, n, 10.0)
    s = np.sin(2 * np.pi * nodes[0] / per[0]) * np.cos(2 * np.pi * nodes[1] / per[1])
    rho = 1.4 * (1 + 0.1 * s)
    q = I.primitive_to_conserved(rho, [0.5 + 0.1 * s, -0.3 + 0.2 * s], 1.0 + 0.1 * s)
    og, fg = O.Grid(2, n, g, bc=bc), fp.Grid(2, n, g, bc=bc)
    return og, fg, O.metrics(og, Y, xyz), np.ascontiguousarray(q)


@pytest.mark.parametrize("bc", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("recon,Y,prec,g", [("weno5", 6, "fp64", 3), ("linup5", 4, "fp64", 3),
                                            ("weno7", 8, "mixed", 4), ("wenocu6", 2, "mixed", 3)])
def test_stage_matches_sweeps_and_oracle(recon, Y, prec, g, n, bc):
    if any(b == 0 and m < g for b, m in zip(bc, n)):
        pytest.skip("a periodic axis needs n >= ghost")
    og, fg, met, q = case(n, g, Y, list(bc) + [0])
    sc = fp.Scheme(recon, Y, True, precision=prec)
    mg = torch.from_numpy(met).cuda()
    q1, q2 = torch.from_numpy(q).cuda(), torch.from_numpy(q).cuda()
    w1 = torch.zeros(fg.work_shape(), dtype=torch.float64, device="cuda")
    w2 = torch.zeros_like(w1)
    dt = 1e-3
    fp.rk3_step(fg, sc, mg, q1, w1, dt)
    fp.profile_step(fg, sc, mg, q2, w2, dt)
    assert torch.equal(q1, q2)
    ref = O.rk3_step(og, O.Scheme(recon, Y, True), met, q, dt)
    got = q1.cpu().numpy()
    for v in range(4):
        scale = np.abs(ref[v] - q[v]).max() * 1e-4 if prec == "mixed" else np.abs(ref[v]).max() * 1e-12
        assert np.abs(got[v] - ref[v]).max() <= scale
