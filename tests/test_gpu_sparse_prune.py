"""When a sparse descent scores only the columns of the row of largest |r| unasked: the rule at its edges (row length, column
length, form of the full evaluation, size of the matrix), the options that decide it, and the same moves
whichever way is taken - with many levels, a mask, a radius and columns of any length."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from workloads import random_sparse

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
ALL, WORST_ROW = 1, 2


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def structured(m, n, row_len, long_col, dtype, seed):
    """CSR on the GPU: `row_len` entries in every row at distinct columns (one row of that length at least), column 0 in
    the first `long_col` rows."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    first = torch.randint(1, n, (m, 1), generator=g, device=DEV)
    step = (torch.arange(row_len, device=DEV) * max(1, (n - 1) // row_len))[None, :]
    col = 1 + (first + step) % (n - 1)                                  # distinct: the steps are shorter than n - 1 in all
    col[:long_col, 0] = 0
    col, _ = torch.sort(col, 1)
    rowptr = torch.arange(m + 1, device=DEV) * row_len
    val = torch.randn(m * row_len, generator=g, device=DEV, dtype=torch.float64).to(dtype)
    b = torch.randn(m, generator=g, device=DEV, dtype=torch.float64).to(dtype) * 3
    return dict(csr=(rowptr, col.reshape(-1).int(), val), m=m, n=n, b=b, device=DEV)


def descent(prob, moves, **opt):
    from paper_2508_13437_amd import dmmv
    D = [-2.0, -1.0, 0.0, 1.0, 2.0]
    with dmmv.Handle(D=D, **prob, **opt) as h:
        used = dmmv.dmmv_scoring_in_use(h, opt.get("radius", 0))
        res = dmmv.dmmv_solve(h, torch.zeros(prob["n"], device=DEV, dtype=prob["b"].dtype), moves, trace=True)
        r = dmmv.dmmv_get_state(h)[1]
        return used, [t.cpu().numpy() for t in (res.iters_done, res.trace, res.trace_t, res.x, r)]


@pytest.mark.parametrize("m,n,row_len,long_col,dtype,want", [
    (700, 160, 20, 0, torch.float32, WORST_ROW), (700, 159, 20, 0, torch.float32, ALL),          # row length: n / 8
    (700, 160, 20, 0, torch.float64, WORST_ROW), (700, 159, 20, 0, torch.float64, ALL),
    (3000, 900, 4, 1020, torch.float64, WORST_ROW), (3000, 900, 4, 1030, torch.float64, ALL),    # longest column: 1024
    (3000, 900, 4, 1030, torch.float32, WORST_ROW),                                              # one-kernel evaluation
    (40000, 20000, 3, 1030, torch.float32, ALL),                                                 # two-kernel, fp32
    (50000, 10000, 210, 1100, torch.float64, WORST_ROW),                                         # 8192 longest columns
])
def test_rule_edges_and_same_moves(m, n, row_len, long_col, dtype, want):
    print("sparse pruning rule", m, n, row_len, long_col, dtype, flush=True)
    prob = structured(m, n, row_len, long_col, dtype, m + n)
    used, got = descent(prob, 25)
    assert used == want
    for opt, scored in ((dict(sparse_eval=1), ALL), (dict(prune=True), WORST_ROW), (dict(prune=True, sparse_eval=1), WORST_ROW)):
        other, res = descent(prob, 25, **opt)
        assert other == scored
        assert all(np.array_equal(a, b) for a, b in zip(got, res)), opt
    assert got[0][0] >= 5                                               # a descent, not a start at an optimum
    assert descent(prob, 3, keep_going=True)[0] == ALL


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("nd", [3, 64, 70])
def test_unasked_pruning_with_mask_radius_and_many_levels(nd, dtype):
    from paper_2508_13437_amd import dmmv
    inst = random_sparse(9100 + nd, 900, 300, nd, density=0.03, dtype=dtype)
    rng = np.random.default_rng(nd)
    x0 = rng.choice(inst.D, inst.n).astype(dtype)
    mask = (rng.uniform(size=inst.n) < 0.6).astype(np.uint8)
    for radius, vm in ((0, None), (1, mask), (2, None), (0, mask)):
        o = orc.solve_csr(inst.m, inst.n, inst.csr_rowptr, inst.csr_col, inst.csr_val, inst.b, inst.D, x0, 40,
                          radius=radius, var_mask=vm)
        with dmmv.from_instance(inst, DEV, radius=radius, **({} if vm is None else dict(var_mask=T(vm)))) as h:
            assert dmmv.dmmv_scoring_in_use(h, radius) == WORST_ROW
            res = dmmv.dmmv_solve(h, T(x0), 40, trace=True)
            table = dmmv.dmmv_eval_moves(h).cpu().numpy()                # the records left the table's buffer fit for use
        d = int(res.iters_done[0])
        tr = res.trace.cpu().numpy()[0]
        assert d == o.iters_done and np.array_equal(tr[:d, 0], o.trace_j) and np.array_equal(tr[:d, 1], o.trace_k)
        assert np.array_equal(res.trace_t.cpu().numpy()[0, :d], o.trace_t) and np.array_equal(res.x.cpu().numpy(), o.x)
        want = orc.eval_moves_csr(inst.m, inst.n, inst.csr_rowptr, inst.csr_col, inst.csr_val, inst.D, o.x, o.r,
                                  radius=radius, var_mask=vm)
        assert np.array_equal(table, np.asarray(want).reshape(-1))
