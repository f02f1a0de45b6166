"""Residual of an fp32 batch on the matrix cores in the contract's order: bitwise against the oracle
at the edges of every tile shape the dispatch can take, and t = max |r| from the same launch."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from workloads import random_batched

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("m,n,R", [
    (1, 1, 1), (63, 24, 15), (64, 25, 16), (65, 47, 17), (130, 48, 33), (257, 97, 20),   # 64 x 16, one wavefront
    (1025, 49, 513),                                                                      # 64 x 16, four wavefronts
    (2049, 33, 513), (2050, 31, 520),                                                     # 64 x 32
    (3999, 13, 1990), (4000, 12, 1985), (3841, 5, 1921),                                  # 128 x 64
])
@pytest.mark.parametrize("integer", [False, True])
def test_batched_residual_in_order_on_matrix_cores(m, n, R, integer):
    from paper_2508_13437_amd import dmmv

    print("chain residual", m, n, R, integer, flush=True)
    inst = random_batched(7000 + m + n, m, n, R, 8, integer=integer)
    with dmmv.from_instance(inst, DEV) as h:
        dmmv.dmmv_set_x(h, torch.from_numpy(inst.x0).to(DEV))
        for _ in range(2):                                   # the maxima start again on every call
            r = dmmv.dmmv_residual(h).cpu().numpy()
            t = dmmv.dmmv_get_state(h)[2].cpu().numpy()
    assert np.array_equal(t, np.abs(r).max(1))
    for q in sorted({0, 1 % R, R // 2, max(R - 17, 0), R - 1}):
        want = orc.residual_dense(inst.A, inst.b[q], inst.D, inst.x0[q], scale=inst.scale[q])
        assert np.array_equal(r[q], want), q
