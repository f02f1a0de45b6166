"""The pruned batched descent where an instance has few rows: fewer than the wavefronts, than the screening rows, than the threads,
and one more of each; the rows that screen are shared by the wavefronts below 256 and strided from there on."""
import numpy as np
import pytest

from workloads import random_batched, random_dense

from test_gpu_batched_pruned import dense_pruned_check
from test_gpu_parity import batched_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 7, 15, 16, 17, 63, 64, 65, 252, 253, 255, 256, 257, 300])
def test_pruned_rows(m, dtype):
    batched_check(random_batched(9900 + m, m, 40, 4, 6, dtype=dtype), 12, prune=True)
    batched_check(random_batched(9950 + m, m, 300, 3, 4, dtype=dtype, integer=True), 12, prune=True)
    dense_pruned_check(random_dense(9990 + m, m, 30, 5, dtype=dtype), 20)
