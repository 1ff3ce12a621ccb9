"""Rounding error of the FP64 residual: against the oracle evaluated in
extended precision (its source with long double for double), the GPU's rms
error is no larger than that of the oracle's plain double evaluation, from the
same metrics and state.  Noise of 2% on every conserved variable, so that the
roundings of neighbouring nodes are independent."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest
import torch

import oracle as O
from paper_2101_05886_amd import fp
from tests import gpu_cases as G

pytestmark = pytest.mark.gpu
LD = C.c_longdouble


class ExtendedScheme(C.Structure):
    _fields_ = [(n, LD if t is C.c_double else t) for n, t in O._Scheme._fields_]


@pytest.fixture(scope="module")
def extended(tmp_path_factory):
    """residual(grid, scheme, met, q) of the oracle in long double"""
    d = tmp_path_factory.mktemp("extended")
    src = os.path.dirname(O.__file__)
    for f in ("fpo.c", "fpo.h"):
        with open(os.path.join(src, f)) as h:
            text = re.sub(r"\bdouble\b", "long double", h.read()).replace("<math.h>", "<tgmath.h>")
        (d / f).write_text(text)
    so = str(d / "extended.so")
    subprocess.run(["gcc", *O.GCC_FLAGS, "-o", so, str(d / "fpo.c"), "-lm"], check=True)
    L = C.CDLL(so)

    def residual(grid, scheme, met, q):
        s = scheme.c()
        x = ExtendedScheme(*[getattr(s, n) for n, _ in s._fields_])
        m, v = met.astype(np.longdouble), q.astype(np.longdouble)
        r = np.zeros_like(v)
        p = [a.ctypes.data_as(C.POINTER(LD)) for a in (m, v, r)]
        assert L.fpo_residual(C.byref(grid.c()), C.byref(x), *p) == 0
        return r

    return residual


@pytest.mark.parametrize("recon,Y,g", [("weno5", 6, 3), ("weno5", 8, 4), ("linup5", 6, 3), ("linup5", 4, 3),
                                       ("linup5", 8, 4), ("weno7", 8, 4), ("wenocu6", 6, 3)])
@pytest.mark.parametrize("ndim,n", [(3, (31, 23, 17)), (2, (83, 61))])
def test_residual_rounding(extended, ndim, n, recon, Y, g):
    case = G.periodic_case(ndim, n, Y, g=g, state="noisy", seed=1)
    og, osc = O.Grid(ndim, n, g), O.Scheme(recon, Y, True)
    met = O.metrics(og, Y, case["xyz"])
    ref = G.I.interior(extended(og, osc, met, case["q"]), g)
    plain = G.I.interior(O.residual(og, osc, met, case["q"]), g)
    got = fp.residual(fp.Grid(ndim, n, g), fp.Scheme(recon, Y, True), torch.from_numpy(met).cuda(),
                      torch.from_numpy(case["q"]).cuda())
    got = G.I.interior(got.cpu().numpy(), g)

    def rms(x):  # relative to each variable's residual
        axes = tuple(range(1, ndim + 1))
        return float(np.sqrt(((x - ref) ** 2).mean(axes) / (ref ** 2).mean(axes)).mean())

    print(f"{recon} Y={Y} {ndim}D: GPU {rms(got):.3e}, plain double {rms(plain):.3e}")
    assert rms(got) <= rms(plain)
