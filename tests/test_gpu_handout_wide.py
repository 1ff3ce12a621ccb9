"""Handed-out eta / zeta work lists of wide 3D stencils, whose LDS holds the
ring and nothing beside it (the next item goes round through a word of it),
and the join of a mixed batch's 2D part: every block bitwise the block alone."""
import pytest
import torch

from paper_2101_05886_amd import fp
from tests import gpu_cases as G
from tests.test_gpu_batch import Block

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("recon,Y,prec", [("weno7", 8, "fp64"), ("weno7", 6, "mixed"), ("linup5", 8, "fp64")])
def test_long_work_lists_of_wide_stencils(recon, Y, prec):
    sc = fp.Scheme(recon, Y, True, precision=prec)
    shapes, count = [(192, 12, 192), (192, 192, 12)], 7
    # a workgroup takes 64 lines of an axis; at most two are resident on each of 256 CUs
    assert count * 192 * 192 // 64 > 6 * 512
    kinds = [Block(G.periodic_case(3, n, Y, g=4, state="noisy", seed=95 + i), sc) for i, n in enumerate(shapes)]
    refs = [[k.alone(sc, s) for s in (1, 3)] for k in kinds]
    qs = [[k.q0.clone() for _ in range(count)] for k in kinds]
    entries = [(k.grid, k.met, q, torch.zeros_like(k.work), k.dt) for k, kq in zip(kinds, qs) for q in kq]
    b = fp.Batch(sc, len(entries))
    b.set(entries)
    for step, advance in enumerate((b.rk3_step, lambda: b.solve(2))):
        advance()
        torch.cuda.synchronize()
        for ref, kq in zip(refs, qs):
            assert all(torch.equal(q, ref[step]) for q in kq)
    b.close()


def test_mixed_batch_is_joined_to_the_callers_stream():
    sc = fp.Scheme("weno5", 6, True)
    blocks = [Block(G.periodic_case(2, (200, 170), 6, state="noisy", seed=5), sc),
              Block(G.periodic_case(3, (20, 17, 13), 6, state="noisy", seed=6), sc),
              Block(G.periodic_case(2, (150, 190), 6, state="noisy", seed=7), sc)]
    refs = [k.alone(sc, 6) for k in blocks]
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    b = fp.Batch(sc, 4)
    with torch.cuda.stream(s):
        b.set([k.entry() for k in blocks])
        b.solve(4)
        b.solve(2)
        seen = [k.q.clone() for k in blocks]  # in stream order, nothing waited for
    s.synchronize()
    for got, ref in zip(seen, refs):
        assert torch.equal(got, ref)
    b.close()
