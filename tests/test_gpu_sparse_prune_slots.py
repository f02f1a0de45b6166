"""Columns around the entries that the evaluation of the worst row's columns holds in registers (256, 512) and levels around those of
its shorter form (4), over one and several row partitions."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from test_gpu_sparse_prune import descent, structured
from workloads import random_sparse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("long_col", [250, 256, 260, 508, 512, 516])
@pytest.mark.parametrize("rows", [0, 300])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_columns_around_the_slots(long_col, rows, dtype):
    print("sparse prune slots", long_col, rows, dtype, flush=True)
    prob = structured(1200, 700, 5, long_col, dtype, long_col)
    opt = dict(sparse_partition_rows=rows) if rows else {}
    _, got = descent(prob, 30, prune=True, **opt)
    _, full = descent(prob, 30, sparse_eval=1, prune=False)
    for a, b in zip(got, full):
        assert np.array_equal(a, b)
    assert got[0][0] >= 5


@pytest.mark.parametrize("nd", [2, 4, 5, 8, 9])
def test_levels_around_the_short_form(nd):
    from paper_2508_13437_amd import dmmv
    inst = random_sparse(8600 + nd, 500, 200, nd, 0.04, dtype=np.float32)
    want = orc.solve_csr(inst.m, inst.n, inst.csr_rowptr, inst.csr_col, inst.csr_val, inst.b, inst.D, inst.x0, 40)
    with dmmv.from_instance(inst, "cuda:0", prune=True) as h:
        res = dmmv.dmmv_solve(h, torch.from_numpy(inst.x0).to("cuda:0"), 40, trace=True)
        assert np.array_equal(res.x.cpu().numpy(), want.x)
