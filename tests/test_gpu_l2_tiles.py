"""The table of l2 changes where its tiles are cut differently (by values, variables and instances, for one instance and for
many), and the arg-min with the l2 change as second criterion on both sides of its choice of loop, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from workloads import random_batched, random_dense

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def tables(inst, checked):
    from paper_2508_13437_amd import dmmv as m

    print("l2 tiles", inst.name, inst.dtype, flush=True)
    scale = inst.scale if inst.scale is not None else np.ones(1, dtype=inst.dtype)
    with m.from_instance(inst, DEV, l2_rule=3) as h:
        m.dmmv_set_x(h, torch.from_numpy(np.ascontiguousarray(inst.x0)).to(DEV))
        r = m.dmmv_residual(h).cpu().numpy().reshape(inst.R, -1)
        dq = m.dmmv_l2_changes(h).cpu().numpy().reshape(inst.R, -1)
    for q in checked:
        x0 = inst.x0.reshape(inst.R, -1)[q]
        want = orc.l2_changes_dense(inst.A, inst.D, x0, r[q], scale=float(scale[q]))
        assert np.array_equal(dq[q], np.asarray(want).reshape(-1)), (inst.name, q)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,nd", [(1, 2), (63, 16), (64, 16), (65, 17), (300, 2), (9, 64), (40, 65), (3, 1024), (3, 1025), (2, 5000),
                                  (5000, 33)])
def test_l2_table_of_one_instance(n, nd, dtype):
    tables(random_dense(8000 + n + nd, 12, n, nd, dtype=dtype), (0,))


@pytest.mark.parametrize("n,R,nd", [(5, 2, 3), (64, 3, 64), (65, 4, 16), (17, 5, 100), (100, 31, 16), (100, 32, 16), (70, 33, 8),
                                    (64, 500, 16), (7, 2000, 300), (1000, 130, 2)])
def test_l2_table_of_a_batch(n, R, nd):
    tables(random_batched(8100 + n + R, 9, n, R, nd), sorted({0, 1, R // 2, R - 1}))
    if n * R * nd < 100000:
        tables(random_batched(8200 + n + R, 9, n, R, nd, dtype=np.float64), sorted({0, 1, R // 2, R - 1}))


@pytest.mark.parametrize("rule", [1, 2])
@pytest.mark.parametrize("n,nd,R", [(585, 7, 1), (586, 7, 1), (255, 32, 3), (256, 32, 3), (600, 33, 2), (8, 4, 70), (2000, 9, 2),
                                    (512, 8, 256), (512, 8, 257)])
def test_l2_argmin_on_both_sides(n, nd, R, rule):
    from paper_2508_13437_amd import dmmv as m

    inst = random_dense(8300 + n, 10, n, nd if nd <= 13 else 13, dtype=np.float32, integer=True) if R == 1 else \
        random_batched(8300 + n, 10, n, R, nd if nd <= 13 else 13, integer=True)       # (integer data: equal scores, equal changes)
    if nd > 13:
        inst = random_batched(8400 + n, 10, n, R, nd)
    print("l2 arg-min", inst.name, rule, flush=True)
    with m.from_instance(inst, DEV, l2_rule=rule) as h:
        m.dmmv_set_x(h, torch.from_numpy(np.ascontiguousarray(inst.x0)).to(DEV))
        m.dmmv_residual(h)
        s = m.dmmv_eval_moves(h).cpu().numpy().reshape(inst.R, -1)
        dq = m.dmmv_l2_changes(h).cpu().numpy().reshape(inst.R, -1)
        best, best_s = (a.cpu().numpy() for a in m.dmmv_argmin_move(h))
        # a table of few different scores, some of them infinite
        given = np.floor(s * 2) / 2
        given[:, ::7] = np.inf
        got, got_s = (a.cpu().numpy() for a in m.dmmv_argmin_move(h, torch.from_numpy(given.reshape(-1) if R == 1 else given).to(DEV)))
    levels = len(inst.D)
    for table, b, bs in ((s, best, best_s), (given.astype(s.dtype), got, got_s)):
        for q in range(inst.R):
            ok = np.ones(dq.shape[1], dtype=bool) if rule == 1 else dq[q] <= 0
            order = np.lexsort((np.arange(dq.shape[1]), dq[q], table[q]))
            order = order[ok[order]]
            c = int(order[0])
            assert (int(b.reshape(-1, 2)[q, 0]), int(b.reshape(-1, 2)[q, 1])) == (c // levels, c % levels), q
            assert bs.reshape(-1)[q] == table[q, c]
