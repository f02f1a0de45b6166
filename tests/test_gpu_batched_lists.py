"""Batched evaluation over the rows that can decide a move (fp32, 256 rows and more): score tables, arg-mins and
descents bitwise against the oracle - lists that suffice, lists that run out (rows all alike, so that every row
is scored), lists given up after a first look, ties that overflow a list, radius and mask, ragged variables, stopped and
packed instances, the largest number of rows, several groups of variables in a workgroup."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from workloads import llm_layer, random_batched

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def check(inst, radius=0, mask=None, samples=4):
    from paper_2508_13437_amd import dmmv
    nd = len(inst.D)
    kw = dict(radius=radius)
    if mask is not None:
        kw["var_mask"] = T(mask)
    with dmmv.from_instance(inst, DEV, **kw) as h:
        dmmv.dmmv_set_x(h, T(inst.x0))
        r = dmmv.dmmv_residual(h).cpu().numpy()
        table = dmmv.dmmv_eval_moves(h).cpu().numpy()
        best, best_s = dmmv.dmmv_argmin_move(h)
        best, best_s = best.cpu().numpy(), best_s.cpu().numpy()
    for q in range(inst.R):
        c = int(np.argmin(table[q]))
        assert best_s[q] == table[q, c] and best[q, 0] * nd + best[q, 1] == c, q
    for q in sorted({0, inst.R - 1, *np.random.default_rng(1).integers(0, inst.R, samples).tolist()}):
        want = orc.eval_moves_dense(inst.A, inst.D, inst.x0[q], r[q], scale=inst.scale[q], radius=radius,
                                    var_mask=None if mask is None else mask[q])
        assert np.array_equal(table[q], np.asarray(want).reshape(-1)), q


@pytest.mark.parametrize("m,n,R,nd", [(256, 64, 3, 16), (257, 65, 5, 16), (300, 300, 4, 8), (511, 130, 7, 4),
                                      (700, 70, 66, 2), (900, 100, 5, 21), (400, 257, 9, 6), (2000, 40, 3, 300)])
def test_batched_lists_random(m, n, R, nd):
    check(random_batched(8300 + m, m, n, R, nd))


@pytest.mark.parametrize("m,n,R,nd", [(256, 33, 20, 13), (600, 80, 9, 8), (1200, 20, 5, 4)])
def test_batched_lists_integer_ties(m, n, R, nd):
    check(random_batched(8400 + m, m, n, R, nd, integer=True))


def test_batched_lists_run_out():
    """Entries of one magnitude whose sign is that of the residual: a step against it lowers every row, so no score
    reaches the bound and all rows are scored."""
    rng = np.random.default_rng(3)
    inst = random_batched(8500, 800, 90, 6, 16)
    sign = rng.choice(np.float32([-1.0, 1.0]), 800)
    inst.A[:] = sign[:, None]
    inst.b[:] = -(1000.0 + rng.uniform(size=inst.b.shape)) * sign[None, :]
    check(inst)
    inst.A[:, ::3] = 0.0                                     # columns of equal values: an empty list
    inst.A[700:, 1::3] = 1e-38
    check(inst)


@pytest.mark.parametrize("m", [256, 300, 511, 512, 1040, 2100])
def test_batched_lists_given_up(m):
    """Entries of mixed size with the residual's sign: the bound after the rows that may be walked stays out of reach, for
    some variables only (the others are of mixed sign), so neighbouring tiles are decided by lists and by all rows."""
    rng = np.random.default_rng(m)
    inst = random_batched(8520 + m, m, 200, 5, 8)
    sign = rng.choice(np.float32([-1.0, 1.0]), m)
    inst.A[:, 60:140] = sign[:, None] * np.abs(inst.A[:, 60:140])
    inst.b[:] = -(1000.0 + rng.uniform(size=inst.b.shape) * 20) * sign[None, :]
    check(inst)


@pytest.mark.parametrize("m,nd", [(16384, 16), (16385, 16), (16384, 5), (16384, 4)])
def test_batched_lists_most_rows(m, nd):
    """The last number of rows whose r fits in LDS (with the score table's scratch beside it), and one more."""
    check(random_batched(8540 + m + nd, m, 70, 3, nd), samples=1)


def test_batched_lists_several_groups_and_packing():
    """Two groups of 256 variables per workgroup with a ragged last one, fewer arg-min records than groups; the descent
    packs the running instances, after which a workgroup takes one group."""
    from paper_2508_13437_amd import dmmv
    inst = random_batched(8560, 256, 2049, 1000, 4)
    check(inst)
    with dmmv.from_instance(inst, DEV) as h:
        res = dmmv.dmmv_solve(h, T(inst.x0), 300, trace=True)
    done = res.iters_done.cpu().numpy()
    few, many = int(np.argmin(done)), int(np.argmax(done))
    assert np.sort(done)[300] + 16 < done[many]              # a quarter had stopped at a polling point before the end
    sel = np.array(sorted({few, many, 0, 499, 999}))
    o = orc.solve_batched(inst.A, inst.b[sel], inst.D, inst.scale[sel], inst.x0[sel], 300)
    assert np.array_equal(done[sel], o.iters_done)
    assert np.array_equal(res.x.cpu().numpy()[sel], o.x) and np.array_equal(res.max_violation.cpu().numpy()[sel], o.t)


def test_batched_lists_radius_and_mask():
    inst = random_batched(8600, 500, 140, 10, 16)
    mask = (np.random.default_rng(4).uniform(size=(10, 140)) < 0.6).astype(np.uint8)
    check(inst, radius=2)
    check(inst, radius=1, mask=mask)


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_batched_lists_layer_descent(bits):
    """A small layer with outlier channels to its local optimum (instances stop at different moves and are packed)."""
    from paper_2508_13437_amd import dmmv
    inst = llm_layer(8700 + bits, tokens=330, features=150, rows=70, bits=bits, iters=40)
    check(inst)
    with dmmv.from_instance(inst, DEV) as h:
        res = dmmv.dmmv_solve(h, T(inst.x0), 40, trace=True)
    o = orc.solve_batched(inst.A, inst.b, inst.D, inst.scale, inst.x0, 40)
    assert np.array_equal(res.iters_done.cpu().numpy(), o.iters_done)
    assert np.array_equal(res.x.cpu().numpy(), o.x) and np.array_equal(res.max_violation.cpu().numpy(), o.t)


def test_batched_lists_of_a_pruned_handle():
    """A handle whose descents are pruned holds no r transposed of its own and sorts the columns at its first evaluation, not
    at create; a first evaluation inside a graph capture scores all rows.  Same tables and moves throughout, whatever the
    descent or the outer loop has left in the buffers in between."""
    from paper_2508_13437_amd import dmmv
    inst = random_batched(8580, 600, 300, 40, 8)
    x0 = T(inst.x0)
    with dmmv.from_instance(inst, DEV, alns=True) as h, dmmv.from_instance(inst, DEV, alns=True, prune=True) as hp:
        assert h.workspace_bytes - hp.workspace_bytes >= inst.R * inst.m * 4 - 256
        after = {}
        for name, hh in (("all", h), ("pruned", hp)):
            dmmv.dmmv_set_x(hh, x0)
            dmmv.dmmv_residual(hh)
            out = []
            for _ in range(2):
                out += [dmmv.dmmv_eval_moves(hh), *dmmv.dmmv_argmin_move(hh)]
            out += [dmmv.dmmv_solve(hh, None, 5).x, dmmv.dmmv_eval_moves(hh)]
            out += [dmmv.dmmv_alns(hh, None, 2, ls_moves=2, seed=4).x_best, dmmv.dmmv_residual(hh), dmmv.dmmv_eval_moves(hh)]
            after[name] = [t.cpu().numpy() for t in out]
    for a, b in zip(after["all"], after["pruned"]):
        assert np.array_equal(a, b)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with dmmv.from_instance(inst, DEV, prune=True, stream=stream) as h:
        with torch.cuda.stream(stream):
            dmmv.dmmv_set_x(h, x0)
            dmmv.dmmv_residual(h)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            table = dmmv.dmmv_eval_moves(h)
            best, score = dmmv.dmmv_argmin_move(h)
        for it in range(3):
            table.zero_()
            stream.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(stream):
                graph.replay()
            stream.synchronize()
            assert np.array_equal(table.cpu().numpy(), after["all"][0]), it
            assert np.array_equal(best.cpu().numpy(), after["all"][1]) and np.array_equal(score.cpu().numpy(), after["all"][2])
            with torch.cuda.stream(stream):
                eager = dmmv.dmmv_eval_moves(h)
            stream.synchronize()
            assert np.array_equal(eager.cpu().numpy(), after["all"][0]), it
