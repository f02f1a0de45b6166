"""The reservoir of the rows of largest |r| where its classes of rows and ranks have edges: fewer rows than classes or threads, many
equal residuals, and large residuals in few classes (the proposed floor then lets too many rows in and is raised)."""
import numpy as np
import pytest
import torch

from test_gpu_sparse_prune import descent, structured

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [127, 128, 129, 255, 257, 1023, 1025, 8192, 9000])
@pytest.mark.parametrize("classes", [0, 1, 40, 128])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_descent_with_residuals_in_classes(m, classes, dtype):
    print("sparse reservoir", m, classes, dtype, flush=True)
    prob = structured(m, 400, 6, 0, dtype, m + classes)
    if classes:                                         # |r| of a few values only, the large ones in `classes` of 128 residues
        big = torch.arange(m, device=prob["b"].device) % 128 < classes
        prob["b"] = torch.where(big, 40 + torch.arange(m, device=big.device) % 3, 0).to(dtype)
        rowptr, col, val = prob["csr"]
        prob["csr"] = (rowptr, col, val.sign())
    _, got = descent(prob, 40, prune=True)
    _, full = descent(prob, 40, sparse_eval=1, prune=False)
    for a, b in zip(got, full):
        assert np.array_equal(a, b)
