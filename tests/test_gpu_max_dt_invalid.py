"""fp_max_dt on states with non-physical nodes, whose speeds are NaN.  The
interior nodes go in runs of 256; a run's value is the largest that is not NaN,
and NaN where none is (the last run's missing nodes count 0); the largest bit
pattern of the runs is the denominator of dt.  The same in numpy, to 1e-14
(some twenty operations per node)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2101_05886_amd import fp
from tests import gpu_cases as G

pytestmark = pytest.mark.gpu
GAMMA, CFL = 1.4, 0.5


def expected(ndim, met, q):
    with np.errstate(invalid="ignore"):
        u = q[1:1 + ndim] / q[0]
        c = np.sqrt(GAMMA * (GAMMA - 1) * (q[-1] - 0.5 * (q[1:1 + ndim] * u).sum(0)) / q[0])
        s = met[:ndim * ndim].reshape(ndim, ndim, *q.shape[1:])
        val = sum(np.abs((s[d] * u).sum(0)) + c * np.sqrt((s[d] ** 2).sum(0)) for d in range(ndim)) / met[-1]
    val = val.ravel()
    val = np.concatenate([val, np.zeros(-val.size % 256)]).reshape(-1, 256)
    runs = np.fmax.reduce(val, axis=1)
    with np.errstate(divide="ignore"):
        return CFL / runs[np.argmax(runs.view(np.uint64))]


@pytest.mark.parametrize("ndim,n", [(3, (40, 30, 20)), (2, (90, 70))])
@pytest.mark.parametrize("bad", ["none", "every", "a run", "a run but one", "the last run", "left-handed"])
def test_max_dt_of_invalid_states(ndim, n, bad):
    case = G.periodic_case(ndim, n, 4, state="noisy", seed=23)
    og, fg = O.Grid(ndim, n, 3), fp.Grid(ndim, n, 3)
    met = O.metrics(og, 4, case["xyz"])
    q = case["q"].copy()
    inner = (slice(None),) + (slice(3, -3),) * ndim
    qi = q.reshape((ndim + 2,) + tuple(q.shape[-ndim:]))[inner]
    tot = int(np.prod(n))
    where = {"none": [], "every": range(tot), "a run": range(512, 768), "a run but one": range(512, 767),
             "the last run": range(tot // 256 * 256, tot), "left-handed": []}[bad]
    e = qi[-1].ravel()
    e[list(where)] = -1.0
    qi[-1] = e.reshape(qi[-1].shape)
    if bad == "left-handed":
        met = met.copy()
        met[-1] *= -1.0
    want = expected(ndim, met.reshape((-1,) + q.shape[-ndim:])[inner], qi)
    got = float(fp.max_dt(fg, fp.Scheme("weno5", 4, True), torch.from_numpy(met).cuda(), torch.from_numpy(q).cuda(),
                          CFL).item())
    assert np.isnan(want) == (bad in ("every", "a run"))
    assert np.isnan(got) if np.isnan(want) else abs(got / want - 1) <= 1e-14 or got == want
