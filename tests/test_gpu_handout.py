"""Batches whose eta / zeta work lists are long enough to be handed out item
by item (more than six per workgroup), step by step and through the step
graph, with a short list in between: every block bitwise equal to the block
advanced alone."""
import pytest
import torch

from paper_2101_05886_amd import fp
from tests import gpu_cases as G
from tests.test_gpu_batch import Block

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndim,shapes,count", [(3, [(192, 12, 192), (192, 192, 12)], 7), (2, [(60000, 12)], 4)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_long_work_lists_bitwise_equal_blocks_alone(ndim, shapes, count, prec):
    sc = fp.Scheme("weno5", 6, True, precision=prec)
    kinds = [Block(G.periodic_case(ndim, n, 6, state="noisy", seed=91 + i), sc) for i, n in enumerate(shapes)]
    refs = [[k.alone(sc, s) for s in (1, 2, 4)] for k in kinds]
    qs = [[k.q0.clone() for _ in range(count)] for k in kinds]
    entries = [(k.grid, k.met, q, torch.zeros_like(k.work), k.dt) for k, kq in zip(kinds, qs) for q in kq]
    # a workgroup takes 64 lines; at most 512 workgroups are resident
    assert count * shapes[0][0] * (shapes[0][2] if ndim == 3 else 1) // 64 > 6 * 512

    def check(step, blocks):
        torch.cuda.synchronize()
        for ref, kq in zip(refs, qs):
            for q in kq[:blocks]:
                assert torch.equal(q, ref[step])

    b = fp.Batch(sc, len(entries))
    b.set(entries)
    b.rk3_step()
    check(0, count)
    b.set(entries[:1])
    b.rk3_step()
    b.set(entries[1:])
    b.rk3_step()
    check(1, count)
    b.set(entries)
    b.solve(2)
    check(2, count)
    b.close()
