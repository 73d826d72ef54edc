"""Each form of the MINRES solve, forced where it is not the default (the
MBL_MINRES_LAUNCH variable), shown to run by the names of its kernels."""
import numpy as np
import pytest

from kernel_trace import launched
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
        ks, res = launched(lambda: gpu.minres_solve(b, f, 0.1, rhs, x=x0.clone(), kmax=40,
                                                    precision=precision, ws=ws))
        assert kernel in ks
        out.append(res)
    (x, info), (y, want) = out
    assert info.iters == want.iters
    assert (x - y).norm() <= (1e-11 if precision == "fp64" else 1e-3) * y.norm()


def _batch_case(gpu, torch, L, R, seed):
    b = gpu.Basis(L)
    F = np.stack([disorder_fields(L, 4.0, seed + r) for r in range(R)])
    rhs = torch.randn((b.n, R), dtype=torch.float64, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(seed))
    return b, F, np.linspace(-0.4, 0.4, R), rhs / rhs.norm(dim=0)


@pytest.mark.parametrize("L", [14, 16, 18])
def test_groups_at_device_scope(gpu, torch, monkeypatch, L):
    """The form for groups whose workgroups sit on several XCDs: the same
    operations in the same order, so the same bits, with one trip per iteration
    or two, and with the rank-one term."""
    b = gpu.Basis(L)
    f = disorder_fields(L, 4.0, 1220 + L)
    rhs = torch.as_tensor(gaussian_vector(b.n, 94), device="cuda")
    x0 = torch.as_tensor(gaussian_vector(b.n, 95), device="cuda")
    out = []
    for form in ("", "fenced"):
        monkeypatch.setenv("MBL_MINRES_LAUNCH", form)
        ks, res = launched(lambda: (*gpu.minres_solve(b, f, 0.1, rhs, x=x0.clone(), kmax=301),
                                    gpu.eig_grad(b, f, 0.1, rhs / rhs.norm(), kmax=200)))
        assert "k_minres_group" in ks
        out.append(res)
    (x, info, grad), (y, yinfo, ygrad) = out
    assert torch.equal(x, y) and info == yinfo
    assert np.array_equal(grad[1], ygrad[1]) and grad[3] == ygrad[3]


@pytest.mark.parametrize("L,R", [(14, 32), (16, 16), (16, 32), (18, 16)])
def test_batched_groups_at_device_scope(gpu, torch, monkeypatch, L, R):
    b, F, sg, rhs = _batch_case(gpu, torch, L, R, 1240)
    bt = gpu.Batch(b, R)
    out = []
    for form in ("", "fenced"):
        monkeypatch.setenv("MBL_MINRES_LAUNCH", form)
        ks, res = launched(lambda: gpu.minres_solve_batched(b, bt, F, sg, rhs, kmax=150))
        assert "k_minres_group" in ks
        out.append(res)
    assert torch.equal(out[0][0], out[1][0]) and np.array_equal(out[0][2], out[1][2])
