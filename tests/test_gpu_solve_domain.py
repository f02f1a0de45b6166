"""A descent from a point with a value outside D: refused, and neither x_out (here the buffer of x0 itself) nor the other
results are written; the handle then has no starting point and takes the next one as if nothing had been."""
import ctypes as C
import time

import numpy as np
import pytest
import torch

from test_gpu_parity import N, T, dmmv, oracle_solve
from workloads import random_batched, random_dense, random_sparse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("make,opt", [
    (lambda: random_dense(13000, 200, 30, 5), {}), (lambda: random_dense(13001, 200, 30, 5), dict(dense_loop=1, poll_every=2)),
    (lambda: random_dense(13002, 200, 30, 5), dict(prune=True)), (lambda: random_sparse(13003, 300, 40, 4), dict(poll_every=3)),
    (lambda: random_batched(13004, 100, 20, 6, 4), {}), (lambda: random_batched(13005, 100, 20, 6, 4), dict(prune=True))])
def test_start_outside_the_values(make, opt):
    m = dmmv()
    inst = make()
    iters = 12
    good = T(inst.x0)
    for where in (0, good.numel() - 1):
        with m.from_instance(inst, **opt) as h:
            bad = good.clone()
            bad.view(-1)[where] = float(inst.D[-1]) + 1.0
            x = bad.clone()
            t = torch.full((inst.R,), -5.0, dtype=x.dtype, device=x.device)
            done = torch.full((inst.R,), -5, dtype=torch.int32, device=x.device)
            torch.cuda.synchronize()
            status = m.load().dmmv_solve(h._h, C.c_void_p(x.data_ptr()), C.c_int32(iters), C.c_void_p(x.data_ptr()),
                                         C.c_void_p(t.data_ptr()), C.c_void_p(done.data_ptr()), None, None)
            assert status == -4
            assert torch.equal(x, bad) and bool((t == -5).all()) and bool((done == -5).all())
            with pytest.raises(m.DmmvError):
                m.dmmv_solve(h, None, iters)
            res = m.dmmv_solve(h, good, iters)
            o = oracle_solve(inst, iters)
            x_want, t_want = o.x, o.t
            assert np.array_equal(N(res.x).reshape(-1), np.asarray(x_want).reshape(-1))
            assert np.array_equal(N(res.max_violation).reshape(-1), np.asarray(t_want, N(res.max_violation).dtype).reshape(-1))


def _refused(m, h, x, t, done, trace, trace_t, iters):
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    status = m.load().dmmv_solve(h._h, C.c_void_p(x.data_ptr()), C.c_int32(iters), C.c_void_p(x.data_ptr()), C.c_void_p(t.data_ptr()),
                                 C.c_void_p(done.data_ptr()), *[C.c_void_p(v.data_ptr()) if v is not None else None for v in (trace, trace_t)])
    assert status == -4
    return time.perf_counter() - t0


@pytest.mark.parametrize("make,opt", [
    (lambda: random_dense(13010, 200, 30, 5), {}), (lambda: random_dense(13011, 4000, 20, 200), {}),
    (lambda: random_dense(13012, 200, 30, 5), dict(dense_loop=1, poll_every=2)), (lambda: random_dense(13013, 200, 30, 5), dict(dense_loop=1, poll_every=0)),
    (lambda: random_dense(13014, 200, 30, 5), dict(dense_loop=1, keep_going=True)), (lambda: random_dense(13015, 200, 30, 5), dict(prune=True, poll_every=0)),
    (lambda: random_dense(13016, 300, 12, 70), dict(value_search=True, poll_every=3)), (lambda: random_dense(13017, 100, 20, 5), dict(l2_rule=1, poll_every=3)),
    (lambda: random_dense(13018, 33000, 6, 4), dict(poll_every=3)), (lambda: random_dense(13019, 66000, 6, 4), dict(dense_loop=1, poll_every=3)),
    (lambda: random_sparse(13020, 300, 40, 4), dict(poll_every=3)), (lambda: random_sparse(13021, 300, 40, 4), dict(poll_every=0, prune=True)),
    (lambda: random_sparse(13022, 300, 40, 4), dict(keep_going=True)), (lambda: random_sparse(13023, 300, 40, 4), dict(l2_rule=2, poll_every=2))])
def test_refused_start_leaves_the_trace_alone(make, opt):
    m = dmmv()
    inst = make()
    iters = 17
    with m.from_instance(inst, **opt) as h:
        x = T(inst.x0)
        x.view(-1)[-1] = float(inst.D[0]) - 1.0
        bad = x.clone()
        t, done = torch.full((1,), -5.0, dtype=x.dtype, device=x.device), torch.full((1,), -5, dtype=torch.int32, device=x.device)
        trace = torch.full((iters, 2), -5, dtype=torch.int32, device=x.device)
        trace_t = torch.full((iters,), -5.0, dtype=x.dtype, device=x.device)
        _refused(m, h, x, t, done, trace, trace_t, iters)
        assert torch.equal(x, bad)
        for v in (t, done, trace, trace_t):
            assert bool((v == -5).all())
        good = T(inst.x0)
        res = m.dmmv_solve(h, good, iters, trace=True)
        if "l2_rule" not in opt:
            o = oracle_solve(inst, iters)
            d = int(res.iters_done[0])
            tr = N(res.trace)[0]
            assert d == o.iters_done and np.array_equal(tr[:d, 0], o.trace_j) and np.array_equal(tr[:d, 1], o.trace_k) and np.all(tr[d:] == -1)
            assert np.array_equal(N(res.trace_t)[0, :d], o.trace_t) and np.all(N(res.trace_t)[0, d:] == 0)


def test_refused_without_the_descent():
    """No iteration is run for a start that is refused, polled for or not: a small part of the time of one that is not."""
    m = dmmv()
    inst = random_sparse(13030, 300, 40, 4)
    iters = 30000
    with m.from_instance(inst, keep_going=True) as h:
        x = T(inst.x0)
        m.dmmv_solve(h, x, 100)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        m.dmmv_solve(h, x, iters)
        whole = time.perf_counter() - t0
        x.view(-1)[0] = float(inst.D[0]) - 1.0
        t, done = torch.empty(1, dtype=x.dtype, device=x.device), torch.empty(1, dtype=torch.int32, device=x.device)
        assert _refused(m, h, x, t, done, None, None, iters) < whole / 5


def test_results_of_a_wait_that_ended():
    """A forced one-launch descent that gives up its wait: an error, and no x, t or count of it."""
    m = dmmv()
    inst = random_dense(33, 256, 64, 16, dtype=np.float64)
    x0 = T(np.random.default_rng(2).choice(inst.D, size=inst.n))
    with m.from_instance(inst, dense_loop=2, wait_limit=1) as h:
        x = torch.full((inst.n,), -5.0, dtype=torch.float64, device=x0.device)
        t, done = torch.full((1,), -5.0, dtype=torch.float64, device=x0.device), torch.full((1,), -5, dtype=torch.int32, device=x0.device)
        torch.cuda.synchronize()
        status = m.load().dmmv_solve(h._h, C.c_void_p(x0.data_ptr()), C.c_int32(50), C.c_void_p(x.data_ptr()),
                                     C.c_void_p(t.data_ptr()), C.c_void_p(done.data_ptr()), None, None)
        if status == -7:
            for v in (x, t, done):
                assert bool((v == -5).all())
        else:                                                   # (every arrival was already there)
            assert status == 0 and int(done[0]) >= 0
