"""Sparse repair with r in LDS: the largest r that is kept there and the first that is not, rows that do not fill an access
of four, picks around the portions that are fetched at once, two levels only; and the repair with tables in memory after an
iteration that leaves the reservoir to it."""
import numpy as np
import pytest

from test_gpu_alns import alns_check
from workloads import random_sparse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 3, 18, 127, 129, 1025])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_repair_of_few_rows(rows, dtype):
    alns_check(random_sparse(8100 + rows, rows, 40, 4, 0.3, dtype=dtype, integer=rows % 2 == 0), 12, ls_moves=2,
               destroy_count=6, seed=rows)


@pytest.mark.parametrize("extra", [0, 1])
@pytest.mark.parametrize("dtype,limit", [(np.float32, 28672), (np.float64, 14336)])
def test_repair_around_the_largest_r_in_lds(dtype, limit, extra):
    alns_check(random_sparse(8200 + extra, limit - extra, 60, 3, 0.004, dtype=dtype), 8, ls_moves=3, destroy_count=7, seed=5)
    alns_check(random_sparse(8210 + extra, limit + 1 + extra, 60, 3, 0.004, dtype=dtype), 8, ls_moves=3, destroy_count=7, seed=5)


@pytest.mark.parametrize("count", [1, 4, 15, 17, 255, 257, 515])
@pytest.mark.parametrize("levels", [2, 5])
def test_repair_portions_of_picks(count, levels):
    alns_check(random_sparse(8300 + count, 600, 530, levels, 0.03, dtype=np.float32), 8, ls_moves=1, destroy_count=count,
               seed=count, ls_swaps=count % 2)


@pytest.mark.parametrize("ls_moves", [0, 2])
def test_repair_with_tables_in_memory(ls_moves):
    alns_check(random_sparse(8400, 131073 + 16, 24, 4, 0.0008, dtype=np.float32), 6, ls_moves=ls_moves, destroy_count=5, seed=3)
