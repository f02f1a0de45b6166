"""A descent from a point with a value outside D: refused, and neither x_out (here the buffer of x0 itself) nor the other
results are written; the handle then has no starting point and takes the next one as if nothing had been."""
import ctypes as C

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
