"""The xi sweep's division of its items over the XCDs: grids of a multiple of
eight workgroups, whose XCDs take an eighth of the items each (several items
per wave, one, and fewer items than waves), and others.  Bitwise the batched
sweep, which deals its items out in turn, and the accumulating variant bitwise
the sum."""
import pytest
import torch

from paper_2101_05886_amd import fp
from tests import gpu_cases as G
from tests.test_gpu_batch import Block

pytestmark = pytest.mark.gpu

# faces of a 62-node line: 63, one item; items, workgroups
SHAPES = [(62, 5, 6),      # 30, 8: fewer items than waves
          (62, 8, 8),      # 64, 16
          (62, 11, 9),     # 99, 25
          (62, 52, 40),    # 2080: 32 more than the waves of 512 workgroups
          (63, 50, 61),    # 3098 of 64 faces: an odd number per XCD
          (97, 90, 83),    # 11,620
          (30, 70, 90)]    # lines shorter than an item


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", SHAPES)
def test_items_of_every_xcd(n, prec):
    sc = fp.Scheme("weno5", 6, True, precision=prec)
    k = Block(G.periodic_case(3, n, 6, state="noisy", seed=61), sc)
    ref = k.alone(sc, 1)
    b = fp.Batch(sc, 1)
    b.set([k.entry()])
    b.rk3_step()
    torch.cuda.synchronize()
    assert torch.equal(k.q, ref)
    b.close()
    r = fp.residual_dir(k.grid, sc, k.met, k.q0, 0, torch.zeros_like(k.q0))
    acc = torch.rand_like(k.q0)
    got = fp.residual_dir(k.grid, sc, k.met, k.q0, 0, acc.clone(), accumulate=True)
    inner = (slice(None),) + (slice(3, -3),) * 3
    assert torch.equal(got[inner], acc[inner] + r[inner])
