"""Each form of the MINRES solve, forced where it is not the default (the
MBL_MINRES_LAUNCH variable), shown to run by the names of its kernels."""
import numpy as np
import pytest

from test_gpu_minres_refused import _kernels
from workloads import disorder_fields, gaussian_vector

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.mark.parametrize("precision", ["fp64", "fp32_inner"])
def test_one_launch_over_all_xcds_where_asked_for(gpu, torch, monkeypatch, precision):
    """L = 20, 40 iterations from an initial guess, against launches per
    iteration: rounding grows to at most about 1e-13 of the result in so few
    iterations (1e-4 in FP32), as in the comparison of two splits."""
    L = 20
    b = gpu.Basis(L)
    f = disorder_fields(L, 3.5, 1200)
    rhs = torch.as_tensor(gaussian_vector(b.n, 91), device="cuda")
    x0 = torch.as_tensor(gaussian_vector(b.n, 92), device="cuda")
    out = []
    for form, kernel in (("persistent", "k_minres_persistent"), ("iter", "k_minres_qdx")):
        monkeypatch.setenv("MBL_MINRES_LAUNCH", form)
        ws = gpu.Workspace(b, 0, precision)
        assert kernel in _kernels(lambda: out.append(gpu.minres_solve(
            b, f, 0.1, rhs, x=x0.clone(), kmax=40, precision=precision, ws=ws)))
    (x, info), (y, want) = out
    assert info.iters == want.iters
    assert (x - y).norm() <= (1e-11 if precision == "fp64" else 1e-3) * y.norm()
