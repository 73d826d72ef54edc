"""Each form of the MINRES solve, forced where it is not the default (the
MBL_MINRES_LAUNCH variable), shown to run by the names of its kernels."""
import numpy as np
import pytest

import test_gpu_batched
import test_gpu_campaign
import test_gpu_minres_rows
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


@pytest.mark.parametrize("L,R,kmax", [(14, 1, 3), (16, 1, 6), (18, 1, 6), (14, 32, 3), (16, 2, 4),
                                      (18, 8, 5), (18, 16, 7), (18, 32, 13)])
def test_solves_of_few_iterations(gpu, torch, L, R, kmax):
    """Below this bound of iterations the launch on chip costs more than it
    saves. The two forms take the same steps: after so few, x agrees to 1e-12."""
    b, F, sg, rhs = _batch_case(gpu, torch, L, max(R, 2), 1290)
    bt = gpu.Batch(b, max(R, 2))

    def solve(k):
        if R == 1:
            x, info = gpu.minres_solve(b, F[0], sg[0], rhs[:, 0].contiguous(), kmax=k)
            assert info.iters == k
        else:
            x, its, _, _ = gpu.minres_solve_batched(b, bt, F, sg, rhs, kmax=k)
            assert np.all(its == k)
        return x

    ks, x = launched(lambda: solve(kmax - 1))
    assert ("k_minres_qdx" if R == 1 else "k_bq") in ks and "k_minres_group" not in ks
    ks, y = launched(lambda: solve(kmax))
    assert "k_minres_group" in ks and "k_minres_qdx" not in ks and "k_bq" not in ks
    with pytest.MonkeyPatch.context() as mp:
        mp.setenv("MBL_MINRES_LAUNCH", "iter")
        assert (solve(kmax) - y).norm() <= 1e-12 * y.norm()


@pytest.fixture
def per_iteration(gpu, torch, monkeypatch):
    """Launches per iteration forced at sizes that run on chip by default."""
    monkeypatch.setenv("MBL_MINRES_LAUNCH", "iter")
    b, F, sg, rhs = _batch_case(gpu, torch, 14, 2, 1260)
    one = rhs[:, 0].contiguous()
    for kernel, solve in (
            ("k_minres_qdx", lambda: gpu.minres_solve(b, F[0], 0.1, one, kmax=20)),
            ("k_bq", lambda: gpu.minres_solve_batched(b, gpu.Batch(b, 2), F, sg, rhs, kmax=20))):
        ks, _ = launched(solve)
        assert kernel in ks and "k_minres_group" not in ks


# Tests of the launches per iteration that by default solve on chip at their
# sizes, with the form they are about.
@pytest.mark.parametrize("R", [8, 32])
def test_batched_graph_replays_match_eager(gpu, torch, per_iteration, R):
    test_gpu_campaign.test_batched_minres_graph_replays_match_eager(gpu, torch, R)


def test_schedule_knobs_keep_results(gpu, torch, per_iteration):
    test_gpu_batched.test_schedule_knobs_keep_results(gpu, torch)


def test_staged_minres_product(gpu, torch, per_iteration):
    b, F, sg, rhs = _batch_case(gpu, torch, 14, 32, 1270)
    ks, _ = launched(lambda: gpu.minres_solve_batched(b, gpu.Batch(b, 32), F, sg, rhs, kmax=20))
    assert "k_bapply_staged" in ks
    test_gpu_batched.test_staged_minres_product(gpu, torch)


@pytest.mark.parametrize("L,seed,kmax", [(16, 0, 300), (18, 0, 1500), (18, 1, 1500)])
def test_bounded_vs_oracle(gpu, torch, per_iteration, L, seed, kmax):
    test_gpu_minres_rows.test_minres_rows_bounded_vs_oracle(gpu, torch, L, seed, kmax)


def test_converged_vs_oracle(gpu, torch, per_iteration):
    test_gpu_minres_rows.test_minres_rows_converged_vs_oracle(gpu, torch, "fp64")


def test_graph_replays_match_eager(gpu, torch, per_iteration):
    test_gpu_minres_rows.test_minres_rows_graph_replays_match_eager(gpu, torch)


@pytest.mark.parametrize("precision", ["fp64", "fp32_inner"])
def test_graphs_of_the_block_staged_product_match_eager(gpu, torch, monkeypatch, precision):
    """L = 20, 170 iterations (one eager, three replays of 48, 25 eager) and the
    gradient's solve: the bits of eager launches, replay after replay, with
    eager work between."""
    L = 20
    b = gpu.Basis(L)
    f = disorder_fields(L, 3.5, 1280)
    monkeypatch.setenv("MBL_MINRES_GRAPHS", "0")
    eager = gpu.Workspace(b, 0, precision)
    first = torch.as_tensor(gaussian_vector(b.n, 98), device="cuda")
    gpu.minres_solve(b, f, 0.1, first, kmax=2, precision=precision, ws=eager)
    monkeypatch.setenv("MBL_MINRES_GRAPHS", "1")
    graphs = gpu.Workspace(b, 0, precision)
    for trial in range(3):
        rhs = torch.as_tensor(gaussian_vector(b.n, 99 + trial), device="cuda")
        out = []
        for ws in (eager, graphs):
            x, info = gpu.minres_solve(b, f, 0.1, rhs, kmax=170, precision=precision, ws=ws)
            gpu.apply_H(b, f, 0.3, rhs)
            torch.cuda.synchronize()
            grad = gpu.eig_grad(b, f, 0.1, rhs / rhs.norm(), kmax=170, ws=ws)
            out.append((x, info, grad))
        (x, info, grad), (y, yinfo, ygrad) = out
        assert torch.equal(x, y) and info == yinfo
        assert np.array_equal(grad[1], ygrad[1]) and grad[3] == ygrad[3]
