"""options.prune on a batch: the choice of the screening rows and of the workgroup, bitwise against the oracle - rows around
those that are all listed (63) and around a list's length, residuals with one row far above the rest, nearly alike, alike
in the largest value, and falling by orders of magnitude with a move; variables around the blocks of four and eight
wavefronts and of their requests ahead; instances around the number that takes eight."""
import numpy as np
import pytest

from test_gpu_parity import batched_check
from workloads import random_batched

pytestmark = pytest.mark.gpu


def _with_residual(inst, r):
    """b such that the starting point has the residual r (up to the rounding of b)."""
    x = np.asarray(inst.x0, np.float64).reshape(inst.R, -1)
    inst.b[:] = ((x @ np.asarray(inst.A, np.float64).T) * np.asarray(inst.scale, np.float64)[:, None] - r).astype(inst.b.dtype)
    return inst


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n,R,nd", [(10, 20, 4, 5), (22, 130, 3, 4), (62, 40, 3, 8), (63, 129, 5, 4), (64, 128, 5, 4), (65, 30, 6, 7), (66, 200, 2, 16),
                                      (129, 511, 2, 3), (128, 513, 2, 3), (70, 1023, 2, 3), (70, 1025, 2, 3), (70, 1537, 2, 2),
                                      (40, 140, 512, 3), (40, 140, 513, 3), (512, 129, 3, 3), (513, 129, 3, 3), (513, 256, 3, 3), (40, 257, 5, 3), (40, 257, 512, 3), (40, 257, 513, 3), (2050, 9, 3, 5)])
def test_rows_variables_and_instances_around_the_edges(m, n, R, nd, dtype):
    batched_check(random_batched(11000 + m + n, m, n, R, nd, dtype=dtype), 8, prune=True)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", ["one", "alike", "equal", "steep", "zero"])
@pytest.mark.parametrize("m,n,R", [(300, 60, 4), (700, 150, 3)])
def test_residuals_that_are_hard_to_list(m, n, R, kind, dtype):
    inst = random_batched(11100 + m, m, n, R, 6, dtype=dtype, integer=kind == "equal")
    rng = np.random.default_rng(m)
    sign = rng.choice([-1.0, 1.0], size=(R, m))
    r = {"one": np.where(rng.random((R, m)) < 2.0 / m, 100.0, 0.01), "alike": 5.0 + 1e-4 * rng.random((R, m)),
         "equal": np.full((R, m), 7.0), "steep": 10.0 ** (-6.0 * rng.random((R, m))), "zero": np.zeros((R, m))}[kind]
    batched_check(_with_residual(inst, sign * r), 12, prune=True)
