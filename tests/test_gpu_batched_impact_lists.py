"""Impact weights of a batch over the sorted rows of X: the outer loop, bitwise against the oracle, at the edges of the
kernel - variables around a wavefront's 64 list entries, around the smallest and the largest number that takes it; rows around a
workgroup's 8 and their multiples, for every number of rows (1, 2, 4, .. 32) that a wavefront takes at a time; prefixes that are empty,
whole, and ended by equal entries; zero columns."""
import numpy as np
import pytest

from test_gpu_alns import batched_alns_check
from workloads import random_batched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,R,alpha", [(1, 128, 3, 0.3), (1, 129, 3, 0.3), (15, 191, 4, 0.3), (17, 192, 2, 0.0), (64, 193, 5, 0.05),
                                         (127, 256, 9, 3.0), (129, 257, 6, 1e6), (513, 130, 3, 0.3), (1030, 140, 2, 0.02),
                                         (9, 1025, 1, 0.3), (4, 8192, 2, 0.3), (4, 8193, 2, 0.3)])
def test_batched_impact_weights_over_sorted_rows(m, n, R, alpha):
    inst = random_batched(9800 + m + n, m, n, R, 4)
    rng = np.random.default_rng(n)
    inst.A[:, rng.choice(n, max(1, n // 16), replace=False)] *= 20.0        # outlier channels
    inst.A[:, rng.choice(n, max(1, n // 16), replace=False)] = 0.0
    batched_alns_check(inst, 6, ls_moves=1, destroy_count=max(2, n // 20), seed=m, alpha=alpha)


@pytest.mark.parametrize("m,n,R,alpha", [(40, 150, 5, 0.3), (70, 300, 3, 0.0), (33, 200, 40, 0.1)])
def test_batched_impact_weights_of_equal_entries(m, n, R, alpha):
    inst = random_batched(9900 + m, m, n, R, 5, integer=True)
    batched_alns_check(inst, 6, ls_moves=1, destroy_count=n // 8, seed=m, alpha=alpha)


@pytest.mark.parametrize("alpha", [0.0, 1e-15, 1e-11, 1e-7])
@pytest.mark.parametrize("m,n,R", [(40, 150, 5), (70, 300, 3)])
def test_batched_impact_weights_where_the_limit_is_far_below_a_row(m, n, R, alpha):
    """Entries over 120 octaves, zeros among them: rows taken whole, most of whose terms are 0."""
    inst = random_batched(9950 + m, m, n, R, 4)
    rng = np.random.default_rng(m)
    inst.A[:] *= np.exp2(-np.round(120.0 * rng.random(inst.A.shape) ** 3)).astype(inst.A.dtype)
    inst.A[rng.random(inst.A.shape) < 0.1] = 0.0
    batched_alns_check(inst, 8, ls_moves=1, destroy_count=n // 10, seed=m, alpha=alpha)


# rows of the instances that are listed, about half of them, around 4096, 8192, .. 65536 in all
@pytest.mark.parametrize("m,n,R", [(63, 129, 130), (64, 129, 128), (129, 130, 65), (127, 130, 128), (128, 130, 128), (257, 131, 64), (255, 130, 128),
                                   (257, 130, 128), (255, 130, 256), (257, 130, 255), (255, 130, 512), (257, 131, 514)])
def test_batched_impact_weights_by_rows_a_wavefront_takes(m, n, R):
    batched_alns_check(random_batched(9970 + m + R, m, n, R, 4), 4, ls_moves=1, destroy_count=9, seed=m + R, alpha=0.3)
