"""WENO7 and WENOCU6 in FP64 far from unit scale: the same flow in other units
of mass and length (powers of two, so that nothing rounds) and epsilon in the
units of the indicators gives the same weights.  Every operation of the path
scales exactly, so the residual is bitwise the scaled one, from indicators of
1e-120 to 1e123."""
import numpy as np
import pytest
import torch

from paper_2101_05886_amd import fp
from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


def residual(case, sc, a, c):
    grid = fp.Grid(case["ndim"], case["n"], case["g"])
    met = fp.metrics(grid, sc.metric_order, torch.from_numpy(case["xyz"] * 2.0 ** c).cuda())
    r = fp.residual(grid, sc, met, torch.from_numpy(case["q"] * 2.0 ** a).cuda())
    return G.I.interior(r.cpu().numpy(), case["g"])


@pytest.mark.parametrize("a,c", [(200, 3), (120, 0), (-120, 0), (-200, -3)])
@pytest.mark.parametrize("ndim,n", [(3, (19, 14, 11)), (2, (37, 23))])
@pytest.mark.parametrize("recon,Y", [("weno7", 8), ("wenocu6", 6)])
def test_residual_in_other_units(recon, Y, ndim, n, a, c):
    case = G.periodic_case(ndim, n, Y, g=4, state="noisy", seed=17)
    ref = residual(case, fp.Scheme(recon, Y, True), 0, 0)
    # fluxes carry mass times length^(ndim - 1), indicators its square
    eps = 1e-6 * 2.0 ** (2 * (a + c * (ndim - 1)))
    got = residual(case, fp.Scheme(recon, Y, True, weno_eps=eps), a, c)
    assert np.isfinite(ref).all() and np.array_equal(got, ref * 2.0 ** (a - c))
