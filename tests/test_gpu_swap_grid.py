"""The swap search over sorted variables where it is cut into more work than one workgroup takes: slices of its units, units on the
workgroup's list, several stages (whose edges integer entries hit exactly), r in LDS and not; and the kernel that
takes what it does not, in all its forms.  Against the CPU oracle's enumeration of all pairs, bit for bit, from a random start
and from a local optimum of the single moves, which is where the method calls it."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from workloads import random_batched, random_dense

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(inst, descend=0, swaps=2, k_eps=0, instances=None, **options):
    from paper_2508_13437_amd import dmmv as m

    print("swap grid", inst.name, inst.dtype, descend, flush=True)
    R = inst.R
    scale = inst.scale if inst.scale is not None else np.ones(R, dtype=inst.dtype)
    with m.from_instance(inst, DEV, **options) as h:
        m.dmmv_solve(h, torch.from_numpy(np.ascontiguousarray(inst.x0)).to(DEV), descend)
        for _ in range(swaps):
            x, r, _t = (a.cpu().numpy().reshape(R, -1) for a in m.dmmv_get_state(h))
            res = m.dmmv_swap_move(h, k_eps=k_eps)
            for q in range(R) if instances is None else instances:
                i, j, t = orc.best_swap_dense(inst.A, inst.D, x[q], r[q], scale=float(scale[q]))
                assert (int(res.i[q]), int(res.j[q])) == (i, j), (q, int(res.i[q]), int(res.j[q]), i, j)
                assert res.t[q].item() == t


@pytest.mark.parametrize("descend", [0, 300])
@pytest.mark.parametrize("m,n,nd,dtype", [(60, 300, 2, np.float32), (60, 513, 2, np.float64), (90, 700, 16, np.float32),
                                          (40, 1000, 64, np.float32), (9, 1500, 3, np.float32), (200, 260, 5, np.float64)])
def test_swap_slices(m, n, nd, dtype, descend):
    check(random_dense(9600 + n, m, n, nd, dtype=dtype), descend)


@pytest.mark.parametrize("descend", [0, 40])
@pytest.mark.parametrize("seed", range(4))
def test_swap_stage_edges(seed, descend):
    check(random_dense(9700 + seed, 24, 700, 3, dtype=np.float32, integer=True), descend, swaps=4)   # five stages
    check(random_dense(9710 + seed, 24, 200, 4, dtype=np.float64, integer=True), descend, swaps=4)   # two
    check(random_batched(9720 + seed, 16, 180, 5, 4, integer=True), descend, swaps=3)


@pytest.mark.parametrize("descend", [0, 60])
def test_swap_large_units(descend):
    # one workgroup an instance, whose units hold up to 64 x 768 pairs: more of them than its list takes
    check(random_batched(9800, 70, 1536, 300, 2), descend, swaps=1, instances=(0, 150, 299))


@pytest.mark.parametrize("m", [36536, 36537])                 # the last whose r, a filter row and the rest fit LDS; the next
def test_swap_r_in_lds_or_not(m):
    check(random_dense(9900, m, 70, 4, dtype=np.float32))
    check(random_batched(9901, m, 70, 2, 4), 20, swaps=1)


@pytest.mark.parametrize("m", [18188, 18189])
def test_swap_r_in_lds_or_not_fp64(m):
    check(random_dense(9910, m, 66, 3, dtype=np.float64), 20, swaps=1)


@pytest.mark.parametrize("n,dtype", [(8193, np.float32),       # levels in LDS with filter rows, with none, and not in LDS
                                     (8300, np.float64), (8700, np.float64), (17200, np.float32)])
def test_swap_more_variables_than_are_sorted(n, dtype):
    check(random_dense(9920 + n, 3, n, 3, dtype=dtype), swaps=1)


def test_sorted_swap_no_slower_at_its_border():
    """At a local optimum, the largest problem that is sorted against the next one up, which is not."""
    from paper_2508_13437_amd import dmmv as m

    def search_ms(n, nd, rows=2048):
        g = torch.Generator(device=DEV).manual_seed(5)
        A = torch.randn(n, rows, generator=g, device=DEV)
        x = torch.randint(0, nd, (n,), generator=g, device=DEV).float()
        b = (torch.randint(0, nd, (n,), generator=g, device=DEV).double() @ A.double()).float()
        with m.Handle(A=A.t(), b=b, D=[float(v) for v in range(nd)]) as h:
            m.dmmv_solve(h, x, 200)
            best = np.inf
            for _ in range(4):
                start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                m.dmmv_swap_move(h, apply=False)
                start.record()
                for _ in range(5):
                    m.dmmv_swap_move(h, apply=False)
                end.record()
                torch.cuda.synchronize()
                best = min(best, start.elapsed_time(end) / 5)
        return best

    for inside, outside in (((8192, 2), (8193, 2)), ((1536, 64), (1536, 65))):
        a, b = search_ms(*inside), search_ms(*outside)
        print("sorted", inside, f"{a:.3f} ms, not sorted", outside, f"{b:.3f} ms", flush=True)
        assert a < 2.0 * b
