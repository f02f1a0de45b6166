"""The outer loop's launches for dense instances - prefix sums, draws and repair in one, the end of an iteration and the start of
the next in another - bitwise against the oracle where they can go wrong: rows around what a thread keeps in registers and past it,
variables around a tile of the prefix sums and around the marks that a draw looks up first, numbers of draws around one
wavefront's and around the picks prepared at a time, all variables drawn, two levels (no choice in a repair)."""
import numpy as np
import pytest

from test_gpu_alns import alns_check, batched_alns_check
from workloads import random_batched, random_dense

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n,nd,count", [(1, 1, 2, 1), (1023, 40, 4, 5), (2048, 33, 3, 32), (2049, 33, 3, 33), (8192, 9, 5, 3), (8193, 9, 5, 3),
                                          (60, 63, 2, 63), (30, 300, 3, 290), (30, 64, 4, 31), (12, 8191, 3, 10), (12, 8192, 3, 40), (12, 8193, 3, 6),
                                          (6, 16500, 2, 300)])
def test_single_instance(m, n, nd, count, dtype):
    alns_check(random_dense(12000 + m + n, m, n, nd, dtype=dtype), 8, ls_moves=1, destroy_count=count, seed=m + count)


@pytest.mark.parametrize("m,n,R,nd,count", [(2048, 12, 3, 4, 4), (2049, 12, 3, 4, 4), (8193, 6, 2, 4, 2), (40, 60, 513, 3, 6), (2049, 5, 513, 3, 2),
                                            (4097, 3, 513, 2, 2), (50, 150, 512, 4, 33), (20, 300, 5, 2, 280)])
def test_batch(m, n, R, nd, count):
    batched_alns_check(random_batched(12100 + m + n, m, n, R, nd), 4, ls_moves=1, destroy_count=count, seed=m + count)


def test_integer_ties_and_the_l2_guard():
    alns_check(random_dense(12200, 50, 40, 4, dtype=np.float32, integer=True), 30, ls_moves=2, destroy_count=6, seed=1, l2_guard=1)
    batched_alns_check(random_batched(12201, 40, 30, 300, 5, integer=True), 12, ls_moves=2, destroy_count=4, seed=2, l2_guard=1)


@pytest.mark.parametrize("m,n,R", [(5, 4, 256), (5, 4, 257), (40, 33, 1300), (700, 9, 600), (3, 2, 4097)])
def test_batch_of_several_strips(m, n, R):
    """The state of an instance turns with its strip of 256: the last of the workgroups that copy the strip's elements does it."""
    batched_alns_check(random_batched(12300 + R, m, n, R, 4), 7, ls_moves=1, destroy_count=max(1, n // 4), seed=R, l2_guard=R % 2)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n,R", [(2048, 7, 512), (2049, 7, 4), (4096, 7, 4), (4097, 7, 4), (8193, 2049, 2), (4097, 40, 513)])
def test_threads_of_an_instance(m, n, R, dtype):
    """Rows around those that 256 threads hold, and prefix sums around a tile of theirs where the launches are apart."""
    batched_alns_check(random_batched(12400 + m + n, m, n, R, 3, dtype=dtype), 3, ls_moves=0, destroy_count=2, seed=m)
