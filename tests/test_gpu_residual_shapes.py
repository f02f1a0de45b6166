"""Residuals of single instances, bitwise against the oracle, at the edges of the kernels' tiles: rows longer and
shorter than a pass, empty rows, a row count that leaves a wavefront part empty, more levels than LDS
holds, more columns than a staged tile; and t = max |r| after each, rows of NaN left out of it."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from workloads import random_batched, random_dense, random_sparse

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def check(inst, want):
    from paper_2508_13437_amd import dmmv
    with dmmv.from_instance(inst, DEV) as h:
        dmmv.dmmv_set_x(h, torch.from_numpy(inst.x0).to(DEV))
        r = dmmv.dmmv_residual(h).cpu().numpy()
        t = float(dmmv.dmmv_get_state(h)[2][0])
    assert np.array_equal(r, want) and t == (np.abs(want).max() if want.size else 0.0)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n,nd,density", [(1, 1, 2, 1.0), (15, 64, 3, 1.0), (17, 65, 3, 1.0), (63, 300, 4, 0.9),
                                            (65, 129, 1500, 0.5), (200, 500, 3, 0.004), (130, 40, 5, 0.0)])
def test_csr_residual_tiles(m, n, nd, density, dtype):
    inst = random_sparse(8100 + m, m, n, nd, density=density, dtype=dtype)
    check(inst, orc.residual_csr(inst.m, inst.csr_rowptr, inst.csr_col, inst.csr_val, inst.b, inst.D, inst.x0))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,longest", [(1, 1), (255, 12), (257, 12), (300, 13), (600, 1)])
def test_csr_residual_short_rows(m, longest, dtype):
    """Rows of 0 to `longest` entries, on both sides of the length up to which a lane takes a whole row."""
    inst = random_sparse(8160 + m, m, 40, 4, density=1.0, dtype=dtype)
    rng = np.random.default_rng(m)
    lens = rng.integers(0, longest + 1, m)
    lens[m // 2] = longest
    at = np.concatenate([inst.csr_rowptr[i] + np.sort(rng.choice(40, lens[i], replace=False)) for i in range(m)]).astype(int)
    inst.csr_col, inst.csr_val = inst.csr_col[at].copy(), inst.csr_val[at].copy()
    inst.csr_rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    check(inst, orc.residual_csr(inst.m, inst.csr_rowptr, inst.csr_col, inst.csr_val, inst.b, inst.D, inst.x0))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n", [(1, 1), (17, 65), (40, 130)])
def test_csr_residual_keeps_the_sign_of_zero(m, n, dtype):
    """Products that underflow to -0: the sum is -0, also where a row is shorter than a pass of 64 entries."""
    from paper_2508_13437_amd import dmmv
    inst = random_sparse(8180 + m, m, n, 3, density=1.0, dtype=dtype)
    tiny = np.finfo(dtype).tiny
    inst.csr_val[:] = -tiny
    inst.D = np.array([0.0, tiny, 1.0], dtype)
    inst.x0[:] = tiny
    inst.b[:] = 0.0
    want = orc.residual_csr(inst.m, inst.csr_rowptr, inst.csr_col, inst.csr_val, inst.b, inst.D, inst.x0)
    with dmmv.from_instance(inst, DEV) as h:
        dmmv.dmmv_set_x(h, torch.from_numpy(inst.x0).to(DEV))
        r = dmmv.dmmv_residual(h).cpu().numpy()
    assert np.signbit(want).all() and not want.any() and not r.any()
    assert np.signbit(r).all()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n", [(1, 1), (63, 15), (65, 16), (130, 17), (64, 1023), (70, 1025), (33000, 3)])
def test_dense_residual_tiles(m, n, dtype):
    inst = random_dense(8200 + m + n, m, n, 5, dtype=dtype)
    check(inst, orc.residual_dense(inst.A, inst.b, inst.D, inst.x0))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m", [5, 128, 129, 700, 3000])
def test_max_violation_leaves_nan_rows_out(m, dtype):
    """A residual with NaN rows (one that overflowed): t is the maximum over the other rows for every storage kind, also
    when the NaN is the first row, when few rows are left and when none is."""
    from paper_2508_13437_amd import dmmv
    rng = np.random.default_rng(m)
    insts = [random_sparse(8150 + m, m, 60, 3, density=0.2, dtype=dtype), random_dense(8150 + m, m, 6, 3, dtype=dtype),
             random_batched(8150 + m, m, 6, 2, 4, dtype=dtype)]
    for inst in insts:
        R = inst.R if inst.kind == "batched" else 1
        with dmmv.from_instance(inst, DEV) as h:
            dmmv.dmmv_set_x(h, torch.from_numpy(inst.x0).to(DEV))
            for nans in (1, m // 2, m - 1, m):
                r = rng.standard_normal((R, m)).astype(dtype)
                r[:, rng.permutation(m)[:nans]] = np.nan
                if nans > 1:
                    r[:, 0] = np.nan
                for _ in range(2):
                    dmmv.dmmv_set_residual(h, torch.from_numpy(r).to(DEV).reshape(h._rshape()))
                    t = dmmv.dmmv_get_state(h)[2].cpu().numpy()
                    want = np.where(np.isnan(r), dtype(0), np.abs(r)).max(1)
                    assert np.array_equal(t, want), (inst.kind, nans)
