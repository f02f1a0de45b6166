"""The matrix-core products of an fp32 batch where the choice of the tile changes with the number of columns and of workgroups:
the residual against the oracle and G = X^T r through the l2 changes; and G's time where a grid is four rounds of the chip."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from workloads import random_batched

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("m,R,columns", [
    (70, 20, (1, 2, 3, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 65, 255, 256)),   # short chains: sets of 16
    (70, 20, (257, 287, 288, 289, 335, 336, 337, 384, 433)),                     # beyond: sets of 48
    (2048, 512, (16, 48, 50)),                                                   # the most workgroups of a short chain
    (2048, 513, (16, 48, 50)),                                                   # one more
])
def test_residual_at_the_edges_of_the_tiles(m, R, columns):
    from paper_2508_13437_amd import dmmv

    for n in columns:
        print("tiles", m, n, R, flush=True)
        inst = random_batched(7900 + n, m, n, R, 8)
        with dmmv.from_instance(inst, DEV, prune=True) as h:
            dmmv.dmmv_set_x(h, torch.from_numpy(inst.x0).to(DEV))
            r = dmmv.dmmv_residual(h).cpu().numpy()
            t = dmmv.dmmv_get_state(h)[2].cpu().numpy()
        assert np.array_equal(t, np.abs(r).max(1))
        for q in sorted({0, 17 % R, R // 2, R - 1}):
            want = orc.residual_dense(inst.A, inst.b[q], inst.D, inst.x0[q], scale=inst.scale[q])
            assert np.array_equal(r[q], want), (n, q)


@pytest.mark.parametrize("rows,n,R", [(256, 70, 20), (257, 70, 20), (17, 2048, 512), (17, 2048, 513), (60, 4000, 4000)])
def test_l2_changes_at_the_edges_of_the_tiles(rows, n, R):
    from paper_2508_13437_amd import dmmv

    print("tiles, l2", rows, n, R, flush=True)
    inst = random_batched(7950 + rows, rows, n, R, 2)
    with dmmv.from_instance(inst, DEV, l2_rule=3) as h:
        dmmv.dmmv_set_x(h, torch.from_numpy(inst.x0).to(DEV))
        r = dmmv.dmmv_residual(h).cpu().numpy()
        dq = dmmv.dmmv_l2_changes(h).cpu().numpy().reshape(R, n, 2)
    for q in sorted({0, R // 2, R - 1}):
        want = orc.l2_changes_dense(inst.A, inst.D, inst.x0[q], r[q], scale=float(inst.scale[q]))
        assert np.array_equal(dq[q], np.asarray(want).reshape(n, -1)), q


def test_l2_contraction_of_four_rounds_takes_twice_that_of_two():
    """G of 2048 x 4096: 4096 instances are 1024 workgroups of 128 x 128 on 256 compute units, 2048 are 512."""
    from paper_2508_13437_amd import dmmv

    def ms(R):
        g = torch.Generator(device=DEV).manual_seed(R)
        X = torch.randn(4096, 2048, generator=g, device=DEV)
        with dmmv.Handle(A=X.t(), b=torch.randn(R, 2048, generator=g, device=DEV), D=[-1.0, 0.0, 1.0],
                         scale=np.full(R, 0.01, dtype=np.float32), l2_rule=3) as h:
            dmmv.dmmv_set_x(h, torch.zeros(R, 4096, device=DEV))
            dmmv.dmmv_residual(h)
            return min(dmmv.dmmv_time_l2(h, 8) / 8 for _ in range(5))

    two, four = ms(2048), ms(4096)
    print(f"two rounds {two:.3f} ms, four {four:.3f} ms", flush=True)
    assert four < 2.25 * two
