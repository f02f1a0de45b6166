"""options.prune on a batch, bitwise against the oracle: the screening rows listed anew from all rows, where |r| has a heavy tail, is
alike in more rows than the list holds or falls by a move; rows around the maxima of a workgroup's threads; and the forms of
the kernel by what a compute unit holds - instances around twice and five times the compute units, LDS for two of them."""
import numpy as np
import pytest

from test_gpu_batched_pruned_screening import _with_residual
from test_gpu_parity import batched_check
from workloads import random_batched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n,R,nd", [(64, 40, 4, 5), (127, 300, 3, 4), (257, 30, 3, 256), (511, 300, 2, 4), (513, 20, 3, 300), (2049, 300, 2, 3)])
def test_heavy_tails(m, n, R, nd, dtype):
    inst = random_batched(13100 + m, m, n, R, nd, dtype=dtype)
    rng = np.random.default_rng(m)
    batched_check(_with_residual(inst, rng.choice([-1.0, 1.0], size=(R, m)) * rng.pareto(0.7, size=(R, m))), 10, prune=True)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("alike", [9, 23, 64, 200])
def test_rows_alike(alike, dtype):
    """Integers, whose moves keep most rows on few values."""
    m, n, R = 300, 30, 3
    inst = random_batched(13200 + alike, m, n, R, 6, dtype=dtype, integer=True)
    rng = np.random.default_rng(alike)
    r = np.stack([rng.permutation(np.where(np.arange(m) < alike, 9.0, 2.0)) for _ in range(R)]) * rng.choice([-1.0, 1.0], size=(R, m))
    batched_check(_with_residual(inst, r), 12, prune=True)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n,R,nd", [(70, 20, 512, 3), (70, 20, 513, 3), (10, 300, 1281, 3), (5, 1024, 1281, 2), (5, 1025, 1280, 2), (5, 1025, 1281, 2), (513, 6, 512, 3), (13500, 7, 513, 3)])
def test_forms_of_the_kernel(m, n, R, nd, dtype):
    batched_check(random_batched(13300 + m + n + R, m, n, R, nd, dtype=dtype), 3, prune=True)
