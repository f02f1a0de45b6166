"""The matrix-core products of an fp32 batch over column counts around the two operand sets that take turns (one set, two,
three, a few columns more), in every tile: the residual against the oracle, and G = X^T r through the l2 changes."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from workloads import random_batched

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("m,R,columns", [
    (70, 20, (95, 96, 97, 143, 144, 145, 191, 192, 193, 290)),       # 64 x 16, one wavefront, sets of 48
    (1025, 513, (63, 64, 95, 96, 97, 128, 162)),                     # 64 x 16, four wavefronts, sets of 32
    (2049, 513, (31, 32, 47, 48, 49, 64, 82)),                       # 64 x 32, sets of 16
    (3999, 1990, (47, 48, 67)),                                      # 64 x 64, sets of 16
])
def test_residual_over_column_counts(m, R, columns):
    from paper_2508_13437_amd import dmmv

    for n in columns:
        print("columns", m, n, R, flush=True)
        inst = random_batched(7700 + n, m, n, R, 8)
        with dmmv.from_instance(inst, DEV, prune=True) as h:
            dmmv.dmmv_set_x(h, torch.from_numpy(inst.x0).to(DEV))
            r = dmmv.dmmv_residual(h).cpu().numpy()
            t = dmmv.dmmv_get_state(h)[2].cpu().numpy()
        assert np.array_equal(t, np.abs(r).max(1))
        for q in sorted({0, 17 % R, R // 2, R - 1}):
            want = orc.residual_dense(inst.A, inst.b[q], inst.D, inst.x0[q], scale=inst.scale[q])
            assert np.array_equal(r[q], want), (n, q)


@pytest.mark.parametrize("rows,n,R", [(145, 70, 20), (97, 1025, 513), (47, 2049, 513), (49, 3999, 1990)])
def test_l2_changes_in_every_tile(rows, n, R):
    from paper_2508_13437_amd import dmmv

    inst = random_batched(7800 + rows, rows, n, R, 3)
    with dmmv.from_instance(inst, DEV, l2_rule=3) as h:
        dmmv.dmmv_set_x(h, torch.from_numpy(inst.x0).to(DEV))
        r = dmmv.dmmv_residual(h).cpu().numpy()
        dq = dmmv.dmmv_l2_changes(h).cpu().numpy().reshape(R, n, 3)
    for q in sorted({0, R // 2, R - 1}):
        want = L2(inst, q, r[q])
        assert np.array_equal(dq[q], want), q


def L2(inst, q, r):
    return np.asarray(orc.l2_changes_dense(inst.A, inst.D, inst.x0[q], r, scale=float(inst.scale[q]))).reshape(inst.n, -1)
