"""Arg-min of a given table of a single instance in two stages: sizes around a workgroup's pass and the stage limit,
equal scores in different workgroups (the lowest index wins), infinities."""
import numpy as np
import pytest
import torch

from workloads import random_dense

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,nd", [(64, 128), (91, 91), (1025, 8), (360, 100), (18001, 2), (5143, 7), (300, 999), (4000, 300)])
def test_argmin_of_a_given_table(n, nd, dtype):
    from paper_2508_13437_amd import dmmv
    inst = random_dense(8800 + n, 3, n, nd, dtype=dtype)
    rng = np.random.default_rng(n)
    table = rng.integers(5, 9, n * nd).astype(dtype)
    table[rng.integers(0, n * nd, 50)] = np.inf
    with dmmv.from_instance(inst, DEV) as h:
        for low in (None, 4.0):
            if low is not None:
                table[sorted(rng.integers(0, n * nd, 3))] = low
            best, score = dmmv.dmmv_argmin_move(h, torch.from_numpy(table).to(DEV))
            c = int(np.argmin(table))
            assert int(best[0, 0]) * nd + int(best[0, 1]) == c and float(score[0]) == table[c]
        table[:] = np.inf
        best, score = dmmv.dmmv_argmin_move(h, torch.from_numpy(table).to(DEV))
        assert best[0].tolist() == [0, 0] and float(score[0]) == np.inf
