"""The dense descent as one launch (options.dense_loop = 2) against the CPU oracle and against
the launch-per-step loop (dense_loop = 1): traces, x, r and the error bit for bit.

Paper, section "GPU Acceleration": the iteration is to run without host-side stepping and
synchronisation; the moves are those of the single-move descent (Algorithm 2's local search).
"""
import threading

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from workloads import make_config, random_dense

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def dmmv():
    from paper_2508_13437_amd import dmmv as mod
    return mod


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def N(t):
    return t.detach().cpu().numpy()


def check(inst, iters, x0=None, keep_going=False, **opt):
    """dense_loop 2 and 1 against the oracle: trace, x, error, stored r and t."""
    m = dmmv()
    x0 = inst.x0 if x0 is None else x0
    oopt = {k: v for k, v in opt.items() if k in ("radius", "var_mask")}
    o = orc.solve_dense(inst.A, inst.b, inst.D, x0, iters, **oopt)
    hopt = dict(opt)
    if "var_mask" in hopt:
        hopt["var_mask"] = T(hopt["var_mask"])
    for loop in (2, 1):
        with m.from_instance(inst, DEV, dense_loop=loop, keep_going=keep_going, **hopt) as h:
            res = m.dmmv_solve(h, T(x0), iters, trace=True)
            d = int(res.iters_done[0])
            assert d == o.iters_done, (loop, d, o.iters_done)
            tr = N(res.trace)[0]
            assert np.array_equal(tr[:d, 0], o.trace_j) and np.array_equal(tr[:d, 1], o.trace_k), loop
            assert np.all(tr[d:] == -1)
            assert np.array_equal(N(res.trace_t)[0, :d], o.trace_t)
            assert np.array_equal(N(res.x).reshape(-1), o.x)
            assert N(res.max_violation)[0] == o.t
            x, r, t = m.dmmv_get_state(h)
            assert np.array_equal(N(x).reshape(-1), o.x) and np.array_equal(N(r), o.r) and N(t)[0] == o.t
            # the handle goes on from there: a second call finds the same local optimum state
            res2 = m.dmmv_solve(h, None, 3, trace=True)
            o2 = orc.solve_dense(inst.A, inst.b, inst.D, o.x, 3, **oopt)
            assert int(res2.iters_done[0]) == o2.iters_done and N(res2.max_violation)[0] == o2.t
    return o


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("shape", [(1, 1, 2), (5, 3, 2), (63, 7, 3), (64, 9, 16), (65, 5, 17), (257, 13, 9),
                                   (300, 40, 16), (1000, 6, 37), (130, 4, 200), (700, 48, 16), (90, 300, 3),
                                   (2000, 3, 1000)])
def test_one_launch_descent_random(shape, dtype):
    mm, nn, nd = shape
    print("one-launch descent", shape, dtype.__name__, flush=True)
    inst = random_dense(900 + mm + nn, mm, nn, nd, dtype=dtype)
    rng = np.random.default_rng(mm)
    x0 = rng.choice(inst.D, size=inst.n)
    o = check(inst, 60, x0=x0)
    assert mm < 5 or o.iters_done >= 1


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("seed", range(3))
def test_one_launch_descent_integer_ties(seed, dtype):
    """Small-integer data: exact ties between workgroups' records, the lowest index wins."""
    inst = random_dense(950 + seed, 37, 70, 5, dtype=dtype, integer=True)
    check(inst, 50)


def test_one_launch_descent_radius_mask_and_fixed_work():
    inst = random_dense(91, 90, 17, 9, dtype=np.float64)
    rng = np.random.default_rng(3)
    vm = (rng.uniform(size=inst.n) < 0.5).astype(np.uint8)
    for radius in (1, 2):
        check(inst, 30, radius=radius, var_mask=vm)
    # fixed-work mode: all iterations run, the result is that of the descent
    o = check(inst, 40, keep_going=True)
    assert o.iters_done < 40


def test_one_launch_descent_iteration_cap_and_zero_iterations():
    inst = random_dense(17, 200, 30, 8, dtype=np.float32)
    rng = np.random.default_rng(1)
    x0 = rng.choice(inst.D, size=inst.n)
    o = check(inst, 5, x0=x0)
    assert o.iters_done == 5                      # cut short by the cap, not by a local optimum
    check(inst, 0, x0=x0)


def test_one_launch_descent_on_the_dense_workloads():
    m = dmmv()
    toy = make_config(1)
    rng = np.random.default_rng(0)
    check(toy, toy.iters)
    o = check(toy, toy.iters, x0=rng.choice(toy.D, size=toy.n))
    assert o.iters_done >= 10
    fir = make_config(2)
    x0 = np.clip(fir.x0 + rng.integers(-40, 41, size=fir.n), fir.D[0], fir.D[-1])
    o = check(fir, 40, x0=x0)
    assert o.iters_done >= 10


def test_one_launch_descent_refused_when_it_does_not_fit():
    m = dmmv()
    inst = random_dense(5, 30000, 3, 4, dtype=np.float64)          # r alone exceeds the LDS
    with pytest.raises(m.DmmvError) as e:
        m.from_instance(inst, DEV, dense_loop=2)
    assert e.value.status == -8                                     # DMMV_ERR_UNSUPPORTED
    with m.from_instance(inst, DEV) as h:                            # automatic: the launch loop
        res = m.dmmv_solve(h, T(inst.x0), 3, trace=True)
    o = orc.solve_dense(inst.A, inst.b, inst.D, inst.x0, 3)
    assert int(res.iters_done[0]) == o.iters_done and N(res.max_violation)[0] == o.t


def test_one_launch_descent_bounded_wait_reports_instead_of_hanging():
    """A wait limit of one poll: a workgroup that finds another one not yet arrived gives up, every
    workgroup leaves, dmmv_solve reports the state error and the handle is still at its starting
    point.  (With so short a limit the wait may also simply succeed; then the result is checked.)"""
    m = dmmv()
    inst = random_dense(33, 256, 64, 16, dtype=np.float64)
    rng = np.random.default_rng(2)
    x0 = rng.choice(inst.D, size=inst.n)
    o = orc.solve_dense(inst.A, inst.b, inst.D, x0, 50)
    with m.from_instance(inst, DEV, dense_loop=2, wait_limit=1) as h:
        try:
            res = m.dmmv_solve(h, T(x0), 50, trace=True)
        except m.DmmvError as e:
            print("bounded wait: gave up as intended:", e, flush=True)
            assert e.status == -7                                   # DMMV_ERR_STATE
            x, r, t = m.dmmv_get_state(h)
            assert np.array_equal(N(x).reshape(-1), x0)
            assert np.array_equal(N(r), orc.residual_dense(inst.A, inst.b, inst.D, x0))
        else:
            print("bounded wait: every arrival was already there", flush=True)
            assert int(res.iters_done[0]) == o.iters_done and N(res.max_violation)[0] == o.t
    # the automatic choice falls back to the loop of launches instead of failing
    with m.from_instance(inst, DEV, wait_limit=1) as h:
        assert m.dmmv_loop_in_use(h) == 2
        res = m.dmmv_solve(h, T(x0), 50, trace=True)
        d = int(res.iters_done[0])
        assert d == o.iters_done and N(res.max_violation)[0] == o.t
        tr = N(res.trace)[0]
        assert np.array_equal(tr[:d, 0], o.trace_j) and np.array_equal(tr[:d, 1], o.trace_k) and np.all(tr[d:] == -1)
        assert np.array_equal(N(res.trace_t)[0, :d], o.trace_t)
    # the default limit on the same problem
    with m.from_instance(inst, DEV, dense_loop=2) as h:
        res = m.dmmv_solve(h, T(x0), 50, trace=True)
        assert int(res.iters_done[0]) == o.iters_done and N(res.max_violation)[0] == o.t


# ---- the descent's own one-launch kernel: intervals of the values that can improve -----------------
@pytest.mark.parametrize("dtype,shape,radius,by_interval", [
    (np.float64, (1024, 64, 16), 0, False), (np.float64, (1024, 64, 16), 1, True), (np.float64, (256, 64, 16), 0, False),
    (np.float64, (1110, 34, 14), 0, False), (np.float64, (4096, 32, 1024), 0, True), (np.float32, (3000, 100, 16), 0, True)])
def test_choice_between_the_one_launch_kernels(dtype, shape, radius, by_interval):
    """Scoring every value where the intervals' rounds, which all wavefronts share, cost more than they save."""
    m = dmmv()
    with m.from_instance(random_dense(1, *shape, dtype=dtype), DEV, radius=radius) as h:
        assert m.dmmv_loop_in_use(h) == 2
        assert (m.dmmv_scoring_in_use(h, radius) >= 4) == by_interval


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("shape", [(255, 700, 5),        # a wavefront per variable, several each
                                   (256, 33, 64), (64, 257, 9),
                                   (3000, 20, 300), (513, 5, 4000)])  # long intervals, narrowed by samples
def test_one_launch_intervals_random(shape, dtype):
    """(Without a radius most of these are taken by the kernel that scores every value.)"""
    mm, nn, nd = shape
    print("one-launch intervals", shape, dtype.__name__, flush=True)
    inst = random_dense(1900 + mm + nn, mm, nn, nd, dtype=dtype)
    x0 = np.random.default_rng(nn).choice(inst.D, size=inst.n)
    o = check(inst, 25, x0=x0)
    assert o.iters_done >= 1
    check(inst, 10, x0=x0, radius=1)


def test_one_launch_intervals_plateaus_and_zero_columns():
    """Scores that are flat over many values (rows no step can reach, columns of zeros and of one entry):
    the samples tie and every value of the interval is scored; the lowest index wins.  (So small an instance is taken
    by the kernel that scores every value.)"""
    rng = np.random.default_rng(5)
    for nd in (40, 300):
        A = np.zeros((90, 24))
        A[rng.integers(0, 90, 20), np.arange(20)] = rng.choice([-1.0, 1.0, 2.0], 20)
        A[:, 20] = rng.integers(-1, 2, 90)
        b = rng.integers(-30, 31, 90).astype(np.float64)
        b[:6] = 200.0                                     # a maximum that one or no column touches
        A[:6, 3] = 1.0
        inst = random_dense(1, 90, 24, 4)
        inst.A, inst.b = np.asfortranarray(A), b
        inst.D = np.arange(nd, dtype=np.float64) - nd // 2
        check(inst, 20, x0=rng.choice(inst.D, size=24))


INTERVAL, SHARED, COLUMNS, EIGHT = 4, 8, 16, 32        # dmmv_scoring_in_use: which of its forms a handle runs
F32, F64 = np.float32, np.float64


def check_interval(inst, iters, x0, form, radius=0, mask=None):
    """The descent on the kernel form named, against the oracle; options 0 (the automatic choice takes it) and, where the
    other one-launch kernel fits too, dense_loop = 2."""
    m = dmmv()
    kw = {} if mask is None else dict(var_mask=mask)
    o = orc.solve_dense(inst.A, inst.b, inst.D, x0, iters, radius=radius, **kw)
    hkw = {} if mask is None else dict(var_mask=T(mask))
    ran = 0
    for loop in (0, 2):
        try:
            h = m.from_instance(inst, DEV, radius=radius, dense_loop=loop, **hkw)
        except m.DmmvError as e:
            assert loop == 2 and e.status == -8
            continue
        with h:
            if loop == 0 and m.dmmv_loop_in_use(h) == 1:
                continue                                  # close to the loop of launches: only on request
            assert m.dmmv_scoring_in_use(h, radius) == form, (loop, m.dmmv_scoring_in_use(h, radius), form)
            ran += 1
            res = m.dmmv_solve(h, T(x0), iters, trace=True)
            d = int(res.iters_done[0])
            tr = N(res.trace)[0]
            assert d == o.iters_done, (loop, d, o.iters_done)
            assert np.array_equal(tr[:d, 0], o.trace_j) and np.array_equal(tr[:d, 1], o.trace_k) and np.all(tr[d:] == -1)
            assert np.array_equal(N(res.trace_t)[0, :d], o.trace_t)
            x, r, t = m.dmmv_get_state(h)
            assert np.array_equal(N(x).reshape(-1), o.x) and np.array_equal(N(r), o.r) and N(t)[0] == o.t
    assert ran >= 1
    return o


FORMS = [  # (form, type, m, n, nd, radius): every form in both types; up to 64 levels (a lane each) and more (bisection)
    (INTERVAL, F32, 7700, 262, 48, 1), (INTERVAL, F64, 3533, 264, 310, 1),
    (INTERVAL | EIGHT, F32, 4225, 1032, 26, 1), (INTERVAL | EIGHT, F64, 1743, 1046, 376, 1),
    (INTERVAL | COLUMNS, F32, 321, 311, 55, 0), (INTERVAL | COLUMNS, F64, 129, 274, 63, 0),
    (INTERVAL | COLUMNS, F64, 1000, 300, 65, 0), (INTERVAL | COLUMNS, F32, 300, 300, 300, 0), (INTERVAL | COLUMNS, F64, 78, 91, 374, 2),
    (INTERVAL | COLUMNS | EIGHT, F32, 70, 580, 54, 0), (INTERVAL | COLUMNS | EIGHT, F64, 73, 1041, 18, 0),
    (INTERVAL | COLUMNS | EIGHT, F64, 100, 700, 300, 0), (INTERVAL | COLUMNS | EIGHT, F32, 67, 163, 333, 2),
    (INTERVAL | SHARED, F32, 37070, 15, 343, 1), (INTERVAL | SHARED, F64, 16038, 39, 357, 2),
    (INTERVAL | SHARED | EIGHT, F32, 18712, 46, 391, 2), (INTERVAL | SHARED | EIGHT, F64, 10120, 35, 380, 2),
    (INTERVAL | SHARED | COLUMNS, F32, 17932, 18, 383, 2), (INTERVAL | SHARED | COLUMNS, F64, 1750, 3, 4, 0),
    (INTERVAL | SHARED | COLUMNS | EIGHT, F32, 3000, 24, 64, 0), (INTERVAL | SHARED | COLUMNS | EIGHT, F64, 1500, 24, 64, 0),
    (INTERVAL | SHARED | COLUMNS | EIGHT, F64, 2000, 24, 300, 0), (INTERVAL | SHARED | COLUMNS | EIGHT, F32, 4000, 24, 65, 0),
]


@pytest.mark.parametrize("form,dtype,mm,nn,nd,radius", FORMS)
def test_one_launch_intervals_forms(form, dtype, mm, nn, nd, radius):
    """Random instances on each form, without and with a mask."""
    print("one-launch intervals", form, dtype.__name__, mm, nn, nd, radius, flush=True)
    inst = random_dense(1900 + mm + nn, mm, nn, nd, dtype=dtype)
    rng = np.random.default_rng(nn)
    x0 = rng.choice(inst.D, size=inst.n)
    o = check_interval(inst, 12, x0, form, radius)
    assert o.iters_done >= 1
    check_interval(inst, 6, x0, form, radius, mask=(rng.uniform(size=nn) < 0.5).astype(np.uint8))


@pytest.mark.parametrize("form,dtype,mm,nn,nd", [
    (INTERVAL | COLUMNS, F64, 129, 274, 63), (INTERVAL | COLUMNS, F32, 300, 300, 300), (INTERVAL | COLUMNS | EIGHT, F64, 100, 700, 40),
    (INTERVAL | COLUMNS | EIGHT, F64, 100, 700, 300), (INTERVAL | SHARED | COLUMNS | EIGHT, F64, 1500, 24, 40),
    (INTERVAL | SHARED | COLUMNS | EIGHT, F64, 2000, 24, 300), (INTERVAL | SHARED | COLUMNS | EIGHT, F32, 4000, 24, 65)])
def test_one_launch_intervals_plateaus_ties_and_zero_columns(form, dtype, mm, nn, nd):
    """Scores that are flat over many values (rows no step can reach, columns of zeros and of one entry): the samples tie and
    every value of the interval is scored.  Integer data: exact ties between values, variables and workgroups.  The lowest
    index wins."""
    rng = np.random.default_rng(nd + mm)
    inst = random_dense(1, mm, nn, 4, dtype=dtype)
    inst.D = (np.arange(nd) - nd // 2).astype(dtype)
    A = np.zeros((mm, nn))
    k = nn - 4
    A[rng.integers(0, mm, k), np.arange(k)] = rng.choice([-1.0, 1.0, 2.0], k)
    A[:, k] = rng.integers(-1, 2, mm)
    b = rng.integers(-30, 31, mm).astype(np.float64)
    b[:6] = 200.0                                         # a maximum that one or no column touches
    A[:6, 3] = 1.0
    inst.A, inst.b = np.asfortranarray(A.astype(dtype)), b.astype(dtype)
    check_interval(inst, 15, rng.choice(inst.D, size=nn), form)
    inst.A = np.asfortranarray(rng.integers(-3, 4, (mm, nn)).astype(dtype))
    inst.b = rng.integers(-20 * nn, 20 * nn, mm).astype(dtype)
    o = check_interval(inst, 15, rng.choice(inst.D, size=nn), form)
    assert o.iters_done >= 1


@pytest.mark.parametrize("shape", [(6000, 520, 3), (9001, 12, 2000)])
def test_one_launch_intervals_columns_in_memory(shape):
    """fp64 instances whose columns do not fit beside r in LDS (the automatic choice takes them)."""
    mm, nn, nd = shape
    m = dmmv()
    inst = random_dense(1990 + mm, mm, nn, nd, dtype=np.float64)
    x0 = np.random.default_rng(nn).choice(inst.D, size=inst.n)
    o = orc.solve_dense(inst.A, inst.b, inst.D, x0, 8)
    with m.from_instance(inst, DEV) as h:
        assert m.dmmv_loop_in_use(h) == 2
        form = m.dmmv_scoring_in_use(h)
        assert form & INTERVAL and not form & COLUMNS
        res = m.dmmv_solve(h, T(x0), 8, trace=True)
        d = int(res.iters_done[0])
        assert d == o.iters_done and np.array_equal(N(res.trace)[0, :d, 0], o.trace_j)
        assert np.array_equal(N(m.dmmv_get_state(h)[1]), o.r)


@pytest.mark.parametrize("form,shape", [(INTERVAL | COLUMNS, (1024, 64, 16)), (INTERVAL | SHARED | COLUMNS | EIGHT, (1500, 24, 64))])
def test_one_launch_intervals_bounded_wait(form, shape):
    """A wait limit of one poll: the descent gives up, with the state of the starting point, or finds every arrival there."""
    m = dmmv()
    radius = 1 if not form & SHARED else 0
    inst = random_dense(34, *shape, dtype=np.float64)
    x0 = np.random.default_rng(2).choice(inst.D, size=inst.n)
    o = orc.solve_dense(inst.A, inst.b, inst.D, x0, 20, radius=radius)
    with m.from_instance(inst, DEV, dense_loop=2, wait_limit=1, radius=radius) as h:
        assert m.dmmv_scoring_in_use(h, radius) == form
        try:
            res = m.dmmv_solve(h, T(x0), 20)
        except m.DmmvError as e:
            assert e.status == -7
            x, r, t = m.dmmv_get_state(h)
            assert np.array_equal(N(x).reshape(-1), x0)
            assert np.array_equal(N(r), orc.residual_dense(inst.A, inst.b, inst.D, x0))
        else:
            assert int(res.iters_done[0]) == o.iters_done and N(res.max_violation)[0] == o.t
    with m.from_instance(inst, DEV, wait_limit=1, radius=radius) as h:
        res = m.dmmv_solve(h, T(x0), 20)
        assert int(res.iters_done[0]) == o.iters_done and np.array_equal(N(res.x), o.x)


@pytest.mark.parametrize("loop", [2, 0])
@pytest.mark.parametrize("shapes", [[(6000, 251, 64)] * 4,              # each takes nearly the whole device
                                    [(6000, 251, 64), (1024, 64, 16), (300, 20, 16), (4096, 32, 1024)]])
def test_one_launch_descents_of_several_threads(shapes, loop):
    """Handles of several threads, each on its own stream: the workgroups of one call do not keep those of another from
    starting.  None fails with dense_loop = 2, where an ended wait is an error, and all moves are those of a call by itself."""
    m = dmmv()
    rng = np.random.default_rng(29)
    work, errors = [], []
    for s, (mm, nn, nd) in enumerate(shapes):
        inst = random_dense(60 + s, mm, nn, nd)
        x0 = rng.integers(0, nd, nn)
        o = orc.solve_dense(inst.A, inst.b, inst.D, inst.D[x0], 5)
        work.append((inst, inst.D[x0], o, torch.cuda.Stream()))
    torch.cuda.synchronize()
    gate = threading.Barrier(len(work))

    def calls(inst, x0, o, stream):
        try:
            with torch.cuda.stream(stream), m.from_instance(inst, DEV, dense_loop=loop, stream=stream) as h:
                start = T(x0)
                stream.synchronize()
                gate.wait(60)
                first = None
                for _ in range(6):
                    res = m.dmmv_solve(h, start, 5)
                    assert int(res.iters_done[0]) == o.iters_done and N(res.max_violation)[0] == o.t
                    assert np.array_equal(N(res.x).reshape(-1), o.x)
                    a = m.dmmv_alns(h, start, 6, ls_moves=4, seed=5)
                    got = (N(a.x_best).tobytes(), N(a.t_best).tobytes())
                    first = first or got
                    assert got == first
        except BaseException as e:                      # noqa: BLE001 - reported by the test itself
            gate.abort()
            errors.append(e)

    threads = [threading.Thread(target=calls, args=w) for w in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


@pytest.mark.parametrize("iters", [8, 256, 300])           # before, at and past the first look at the error bit
@pytest.mark.parametrize("scoring,shape", [(1, (120, 40, 16)), (INTERVAL | COLUMNS, (1024, 64, 16))])
def test_alns_dense_one_launch_local_search_bounded_wait_runs_again(scoring, shape, iters):
    """With a wait limit of one poll the one-launch local search (either kernel) gives up; the outer loop then runs again from
    the starting point with a launch per step, and the result is the oracle's either way."""
    m = dmmv()
    inst = random_dense(77, *shape, dtype=np.float64)
    o = orc.alns_dense(inst.A, inst.b, inst.D, inst.x0, orc.alns_params(iters, ls_moves=5, seed=3, destroy_count=3))
    for limit in (0, 1):
        with m.from_instance(inst, DEV, wait_limit=limit) as h:
            assert m.dmmv_scoring_in_use(h, 1) == scoring          # the local search's neighbourhood
            for x0 in (T(inst.x0), None):
                if x0 is None:
                    m.dmmv_set_x(h, T(inst.x0))
                res = m.dmmv_alns(h, x0, iters, ls_moves=5, seed=3, destroy_count=3)
                assert np.array_equal(N(res.trace_t)[:, 0], o.t) and np.array_equal(N(res.x_best), o.x)
                assert np.array_equal(N(res.trace)[:, 2], o.moves)
