"""The pruned batched descent where its bookkeeping has edges: variables in words of 32 and groups of 16 that a lane looks
after (several groups per lane from 4097 variables on), first steps at the ends of D, and few rows for the screening."""
import numpy as np
import pytest

from workloads import random_batched

from test_gpu_parity import batched_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [15, 16, 17, 31, 33, 63, 65, 1025])
def test_pruned_groups(n, dtype):
    batched_check(random_batched(9700 + n, 70, n, 4, 5, dtype=dtype), 10, prune=True)
    batched_check(random_batched(9701 + n, 3, n, 3, 2, dtype=dtype), 6, prune=True)


@pytest.mark.parametrize("n", [4095, 4097, 5001])
def test_pruned_several_groups_per_lane(n):
    inst = random_batched(9800 + n, 40, n, 3, 3, dtype=np.float32)
    batched_check(inst, 12, prune=True)
    inst.x0[:] = inst.D[0]                                   # every first step downwards is at an end of D
    batched_check(inst, 8, radius=1, prune=True)
