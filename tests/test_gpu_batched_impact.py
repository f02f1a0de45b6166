"""Impact weights of a batch (worst-remove operator): the outer loop, bitwise against the oracle, where the
kernel's tiles can go wrong - row passes and row splits with remainders, ragged variables and
instances, outlier columns (queued by rows), every term counting (alpha = 0) and hardly any."""
import numpy as np
import pytest

from test_gpu_alns import batched_alns_check
from workloads import random_batched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,R,alpha", [(31, 63, 3, 0.3), (32, 64, 4, 0.3), (33, 65, 5, 0.3), (65, 40, 13, 0.0),
                                         (129, 260, 9, 3.0), (390, 70, 21, 0.3), (200, 96, 66, 1e6)])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_batched_impact_weights(m, n, R, alpha, dtype):
    inst = random_batched(7800 + m + n, m, n, R, 4, dtype=dtype)
    hot = np.random.default_rng(m).choice(n, max(1, n // 16), replace=False)
    inst.A[:, hot] *= 20.0                                   # outlier channels
    batched_alns_check(inst, 6, ls_moves=2, destroy_count=max(2, n // 10), seed=m, alpha=alpha)
