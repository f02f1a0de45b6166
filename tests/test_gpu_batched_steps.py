"""A batch stepped call by call: the arg-min of given tables (sizes around a thread's eight loads, ties, infinities), the
application of moves and max |r| over row counts around a block's rows, with instances whose move is none."""
import numpy as np
import pytest
import torch

from workloads import random_batched

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,nd", [(1, 2), (11, 93), (1024, 8), (1171, 7), (911, 19)])
def test_argmin_of_given_tables(n, nd, dtype):
    from paper_2508_13437_amd import dmmv
    R = 5
    inst = random_batched(8900 + n, 4, n, R, nd, dtype=dtype)
    rng = np.random.default_rng(n)
    table = rng.integers(5, 9, (R, n * nd)).astype(dtype)
    table[1, -1] = 4.0
    table[2, rng.integers(0, n * nd, 3)] = 4.0
    table[3, : n * nd // 2] = np.inf
    table[4] = np.inf
    with dmmv.from_instance(inst, DEV) as h:
        best, score = dmmv.dmmv_argmin_move(h, torch.from_numpy(table).to(DEV))
    for q in range(R):
        c = int(np.argmin(table[q]))
        assert int(best[q, 0]) * nd + int(best[q, 1]) == c and float(score[q]) == table[q, c], q


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,R", [(1, 2), (7, 65), (63, 3), (65, 64), (127, 4), (129, 130), (200, 5), (511, 70), (512, 2), (513, 66), (1025, 3)])
def test_apply_and_max_violation(m, R, dtype):
    """Integer data: every product and sum is exact in any order, so the residual has one value."""
    from paper_2508_13437_amd import dmmv
    n, nd = 9, 5
    inst = random_batched(9000 + m, m, n, R, nd, dtype=dtype, integer=True)
    rng = np.random.default_rng(m)
    moves = np.stack([rng.integers(0, n, R), rng.integers(0, nd, R)], 1).astype(np.int32)
    moves[1] = -1
    with dmmv.from_instance(inst, DEV) as h:
        dmmv.dmmv_set_x(h, torch.from_numpy(np.ascontiguousarray(inst.x0)).to(DEV))
        r0 = dmmv.dmmv_residual(h).cpu().numpy().reshape(R, m)
        x0 = dmmv.dmmv_get_x(h).cpu().numpy().reshape(R, n)
        dmmv.dmmv_apply_move(h, torch.from_numpy(moves).to(DEV))
        x, r, t = (a.cpu().numpy() for a in dmmv.dmmv_get_state(h))
    x, r = x.reshape(R, n), r.reshape(R, m)
    D, A = np.asarray(inst.D, dtype), np.asarray(inst.A, dtype)
    for q in range(R):
        want_r, want_x = r0[q].copy(), x0[q].copy()
        j, k = moves[q]
        if j >= 0:
            want_r += A[:, j] * (dtype(inst.scale[q]) * (D[k] - want_x[j]))
            want_x[j] = D[k]
        assert np.array_equal(x[q], want_x) and np.array_equal(r[q], want_r), q
        assert t[q] == np.abs(want_r).max(), q
