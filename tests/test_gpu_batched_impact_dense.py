"""Impact weights of a batch where most terms of a pass count: rows taken one by one without the queue, next to passes and
instances that go through it, with remainders of rows, variables and instances; and terms that the short evaluation leaves
to the exact one, a few of them or all."""
import numpy as np
import pytest

from test_gpu_alns import batched_alns_check
from workloads import random_batched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,R,alpha", [(31, 63, 3, 0.0), (33, 33, 5, 0.001), (97, 64, 6, 0.01), (130, 129, 9, 0.03), (64, 31, 4, 0.0),
                                         (35, 200, 17, 0.1), (300, 20, 7, 0.02), (161, 100, 6, 0.3), (1000, 128, 3, 0.1), (70, 150, 1, 0.0),
                                         (70, 150, 2, 0.0)])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_batched_impact_weights_of_most_terms(m, n, R, alpha, dtype):
    inst = random_batched(8500 + m, m, n, R, 6, dtype=dtype)
    rng = np.random.default_rng(m)
    inst.A[:] = rng.choice([-1.0, 1.0], size=(m, n)) * rng.uniform(0.5, 1.0, size=(m, n))     # no small entries
    inst.A[m // 2:, ::2] *= 0.01                             # and, in half of the rows, some
    batched_alns_check(inst, 5, ls_moves=1, destroy_count=max(2, n // 8), seed=m, alpha=alpha)


@pytest.mark.parametrize("m,n,R", [(40, 70, 5), (64, 64, 4), (33, 100, 9)])
def test_batched_impact_weights_left_to_the_exact_evaluation(m, n, R):
    inst = random_batched(8600 + m, m, n, R, 5, integer=True)      # whole terms where alpha is 0
    batched_alns_check(inst, 5, ls_moves=1, destroy_count=max(2, n // 8), seed=m, alpha=0.0)
    inst.A[inst.A == 0] = 1.0
    batched_alns_check(inst, 5, ls_moves=1, destroy_count=max(2, n // 8), seed=m, alpha=0.0)
