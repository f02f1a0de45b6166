"""x values to level indices of a batch and back, by tiles as wide as the batch: one variable, one instance, powers of two and
one off, 32 and more of both, levels in LDS and not; and values outside D, wherever they are."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n,R,nd", [(1, 1, 2), (1, 3000, 3), (3000, 1, 3), (2, 1025, 5), (1025, 2, 5), (3, 700, 1000), (700, 3, 1024),
                                    (16, 130, 1025), (17, 130, 4), (31, 33, 7), (32, 32, 7), (33, 31, 7), (33, 33, 5000), (100, 9, 2),
                                    (64, 600, 9)])
def test_values_round_trip(n, R, nd, dtype):
    from paper_2508_13437_amd import dmmv as m

    print("values", n, R, nd, dtype, flush=True)
    g = torch.Generator(device=DEV).manual_seed(n * R + nd)
    D = torch.cumsum(torch.rand(nd, generator=g, device=DEV, dtype=torch.float64) + 0.1, 0).to(dtype)
    x = D[torch.randint(0, nd, (R, n), generator=g, device=DEV)].contiguous()
    A = torch.rand(n, 2, generator=g, device=DEV).to(dtype)
    b = torch.zeros(R, 2, device=DEV, dtype=dtype)
    with m.Handle(A=A.t(), b=b, D=D.tolist(), scale=np.ones(R)) as h:
        m.dmmv_set_x(h, x)
        assert torch.equal(m.dmmv_get_x(h).reshape(R, n), x)
        r = m.dmmv_residual(h).reshape(R, 2)                 # (that the indices lie where the others look for them)
        want = x.double() @ A.double()
        assert torch.allclose(r.double(), want, rtol=2e-4 if dtype == torch.float32 else 1e-11)
        for at in ((0, 0), (R - 1, n - 1), (R // 2, n // 2)):
            for bad in (float(D[-1]) + 1.0, float(D[0]) - 1.0, 0.5 * (float(D[0]) + float(D[1])), float("nan")):
                y = x.clone()
                y[at] = bad
                with pytest.raises(m.DmmvError) as e:
                    m.dmmv_set_x(h, y)
                assert e.value.status == -4
        m.dmmv_set_x(h, x)
        assert torch.equal(m.dmmv_get_x(h).reshape(R, n), x)
