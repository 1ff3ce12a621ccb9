"""Balanced splits of the eta / zeta sweeps (workgroups whose nodes run across
the end of a line block): blocks that take one, with line blocks and quotas
that leave remainders, against the FP64 oracle's step (1e-12 per variable),
and bitwise against the batched sweeps, which never split that way."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2101_05886_amd import fp
from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(97, 90, 83), (95, 88, 88), (102, 67, 109)])
@pytest.mark.parametrize("recon", ["weno5", "linup5"])
def test_balanced_split_matches_oracle_and_batch(recon, n):
    case = G.periodic_case(3, n, 4, state="noisy", seed=81)
    og, fg = O.Grid(3, n, 3), fp.Grid(3, n, 3)
    met = O.metrics(og, 4, case["xyz"])
    sc = fp.Scheme(recon, 4, True)
    mg = torch.from_numpy(met).cuda()
    q1, q2 = torch.from_numpy(case["q"]).cuda(), torch.from_numpy(case["q"]).cuda()
    w1 = torch.zeros(fg.work_shape(), dtype=torch.float64, device="cuda")
    w2 = torch.zeros_like(w1)
    fp.rk3_step(fg, sc, mg, q1, w1, 1e-3)
    b = fp.Batch(sc, 1)
    b.set([(fg, mg, q2, w2, 1e-3)])
    b.rk3_step()
    torch.cuda.synchronize()
    assert torch.equal(q1, q2)
    b.close()
    ref = O.rk3_step(og, O.Scheme(recon, 4, True), met, case["q"], 1e-3)
    got = q1.cpu().numpy()
    for v in range(5):
        assert np.abs(got[v] - ref[v]).max() <= 1e-12 * np.abs(ref[v]).max()
