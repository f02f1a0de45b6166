"""The arg-min with the l2 change as second criterion where its loop is cut differently, against the oracle: tables around one
round of a workgroup (eight values a thread) and around two, workgroups of each size, more values than threads and fewer, instances
around those that are dealt out by XCD and those that take fewer wavefronts, one variable, a ragged last XCD."""
import numpy as np
import pytest

from test_gpu_l2 import check_descent
from test_gpu_l2_tiles import test_l2_argmin_on_both_sides as check
from workloads import random_batched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rule", [1, 2])
@pytest.mark.parametrize("n,nd,R", [(1, 2, 1), (1, 2, 300), (256, 2, 3), (257, 2, 3), (171, 3, 3), (1024, 2, 64), (1025, 2, 65), (1171, 7, 63),
                                    (1025, 8, 1), (2049, 8, 2), (1024, 2, 257), (1025, 2, 258), (25, 700, 71), (3, 3000, 2), (5, 1025, 300)])
def test_rounds_and_instances(n, nd, R, rule):
    check(n, nd, R, rule)


@pytest.mark.parametrize("rule", [1, 2])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_descent_from_the_least_l2_norm(rule, dtype):
    """A start whose moves nearly all raise the l2 norm: rule 2 leaves almost none."""
    inst = random_batched(8600, 40, 300, 70, 6, dtype=dtype)
    start = 0.01 * np.random.default_rng(1).standard_normal((70, 40))
    inst.b[:] = (np.asarray(inst.x0, np.float64) @ np.asarray(inst.A, np.float64).T) * np.asarray(inst.scale, np.float64)[:, None] - start
    check_descent(inst, 6, rule)
