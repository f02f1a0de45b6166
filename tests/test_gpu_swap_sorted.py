"""The swap search over sorted variables (64 to 8192 of them, at most 64 levels) against the CPU oracle's enumeration of
all pairs, bit for bit, at the edges of what it takes: sizes around a wavefront and a power of two, the largest
level count, masks that leave few variables or none, ties, rows that one variable's entries dominate, and what lies
just outside (which the other kernel takes)."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from workloads import random_batched, random_dense

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(inst, var_mask=None, swaps=2, k_eps=0, **options):
    from paper_2508_13437_amd import dmmv as m

    print("sorted swap", inst.name, inst.dtype, k_eps, flush=True)
    R = inst.R
    scale = inst.scale if inst.scale is not None else np.ones(R, dtype=inst.dtype)
    if var_mask is not None:
        options["var_mask"] = torch.from_numpy(var_mask).to(DEV)
    found = 0
    with m.from_instance(inst, DEV, **options) as h:
        m.dmmv_set_x(h, torch.from_numpy(np.ascontiguousarray(inst.x0)).to(DEV))
        m.dmmv_residual(h)
        for _ in range(swaps):
            x, r, _t = (a.cpu().numpy().reshape(R, -1) for a in m.dmmv_get_state(h))
            res = m.dmmv_swap_move(h, k_eps=k_eps)
            for q in range(R):
                vm = None if var_mask is None else var_mask.reshape(R, inst.n)[q]
                i, j, t = orc.best_swap_dense(inst.A, inst.D, x[q], r[q], scale=float(scale[q]), var_mask=vm)
                assert (int(res.i[q]), int(res.j[q])) == (i, j), (q, int(res.i[q]), int(res.j[q]), i, j)
                assert res.t[q].item() == t
                found += i >= 0
    return found


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,nd", [(63, 5), (64, 2), (65, 64), (128, 65), (129, 3), (1023, 16), (1025, 7)])
def test_sorted_swap_sizes(n, nd, dtype):
    assert check(random_dense(9100 + n, 48, n, nd, dtype=dtype)) > 0
    check(random_dense(9101 + n, 3, n, nd, dtype=dtype), k_eps=1)


@pytest.mark.parametrize("m,n,R", [(1, 70, 2), (300, 200, 3), (600, 130, 5), (40, 100, 1)])
def test_sorted_swap_batches(m, n, R):
    inst = random_batched(9200 + m, m, n, R, 9)
    inst.A[:, 3] *= np.float32(20)                             # an outlier channel
    assert check(inst) > 0
    check(inst, prune=True)                                    # without the evaluation's lists of rows
    check(random_batched(9201 + m, m, n, R, 4, dtype=np.float64))


def test_sorted_swap_largest():
    check(random_dense(9300, 2, 8192, 2, dtype=np.float32), swaps=1)
    check(random_dense(9301, 2, 8193, 2, dtype=np.float32), swaps=1)
    check(random_dense(9302, 2, 8192, 2), swaps=1)


@pytest.mark.parametrize("keep", [0.0, 0.01, 0.5])
def test_sorted_swap_masks_and_ties(keep):
    rng = np.random.default_rng(3)
    inst = random_dense(9400, 30, 150, 5, dtype=np.float32, integer=True)
    check(inst, var_mask=(rng.random(150) < keep).astype(np.uint8), swaps=3)
    inst = random_batched(9401, 30, 90, 4, 6, integer=True)
    check(inst, var_mask=(rng.random((4, 90)) < keep).astype(np.uint8), swaps=3)


def test_sorted_swap_with_nothing_to_gain():
    inst = random_dense(9500, 20, 80, 4)
    inst.x0[:] = inst.D[1]                                     # one level: no pair
    assert check(inst, swaps=1) == 0
    inst.A[:] = 0.0                                            # all pairs alike
    inst.x0[:40] = inst.D[2]
    assert check(inst, swaps=1) == 0
    inst.b[:] = 0.0                                            # t = 0
    assert check(inst, swaps=1) == 0
