"""Impact weights of a batch where a pass's terms are between few and all of its rows: the queue fills in several
portions, ends inside a portion, and lanes hold up to the number of terms that are queued one by one."""
import numpy as np
import pytest

from test_gpu_alns import batched_alns_check
from workloads import random_batched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,R,alpha", [(64, 128, 9, 0.02), (96, 65, 8, 0.08), (97, 200, 5, 0.15)])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_batched_impact_weights_of_many_terms(m, n, R, alpha, dtype):
    inst = random_batched(7900 + m, m, n, R, 6, dtype=dtype)
    batched_alns_check(inst, 5, ls_moves=1, destroy_count=n // 8, seed=m, alpha=alpha)
