"""MINRES with its vectors on chip (registers and LDS), against the oracle.

In the problem array each chain length takes its own number of rows per
thread, and n falls just above or below whole rows of the workgroup
(n = 6, 20, 70, 252 of 512 threads; 924 of 2 x 512; 3432 of 7 x 512). Bars:
those of the problem-array tests against dense eigenpairs.
"""
import numpy as np
import pytest

from test_gpu_problems import _check_dense
from workloads import disorder_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,nev,precond", [(4, 2, "row"), (6, 3, "id"), (8, 5, "row"),
                                           (10, 4, "jacobi"), (12, 4, "id"), (14, 3, "row")])
def test_problem_array_on_chip(gpu, L, nev, precond):
    f = disorder_fields(L, 3.0, 600 + L)
    st, res = gpu.si_lanczos_problems([dict(L=L, h=f, nev=nev)], seed=4, precond=precond,
                                      minres_kmax=400_000)
    print(f"L={L} {precond}: steps {res[0].steps}, {res[0].minres_iters} iterations", flush=True)
    assert st == 0
    _check_dense(L, f, res[0], nev)


def test_problem_array_iteration_limit(gpu):
    """kmax iterations per solve and no more, and a warning."""
    f = disorder_fields(12, 3.0, 612)
    st, res = gpu.si_lanczos_problems([dict(L=12, h=f, nev=2, sigma=0.1)], mmax=3, minres_kmax=7)
    assert st == 1 and res[0].status == 1
    assert res[0].steps == 3 and res[0].minres_iters == 21


def _solve_reference(L, f, sigma, b):
    from oracle import minres, model
    return minres.solve_dense(model.hamiltonian_dense(L, f), sigma, b)


@pytest.mark.parametrize("L", [4, 8, 10, 12, 14])
@pytest.mark.parametrize("precond", ["row", "id"])
def test_single_solve_on_chip(gpu, L, precond):
    """One launch per solve: to the tolerance from x0 = 0, from an initial
    guess, and an iteration limit. The solution is bounded as in the parity
    tests of the solver, ||x - x_ref|| <= 1e-8 ||x_ref|| at tol 1e-12."""
    import torch
    from workloads import gaussian_vector
    f, sigma = disorder_fields(L, 3.0, 700 + L), -0.31
    b = gpu.Basis(L)
    rhs = gaussian_vector(b.n, 71)
    rhs /= np.linalg.norm(rhs)
    ref = _solve_reference(L, f, sigma, rhs)
    t = torch.as_tensor(rhs, device="cuda")
    x, info = gpu.minres_solve(b, f, sigma, t, precond=precond)
    assert info.status == 0
    assert np.linalg.norm(x.cpu().numpy() - ref) <= 1e-8 * np.linalg.norm(ref)
    x0 = torch.as_tensor(0.5 * ref + 0.1 * gaussian_vector(b.n, 72), device="cuda")
    y, info = gpu.minres_solve(b, f, sigma, t, x=x0.clone(), precond=precond)
    assert info.status == 0
    assert np.linalg.norm(y.cpu().numpy() - ref) <= 1e-8 * np.linalg.norm(ref)
    if b.n > 40:
        _, info = gpu.minres_solve(b, f, sigma, t, precond=precond, kmax=5)
        assert info.status == 1 and info.iters == 5


@pytest.mark.parametrize("L,R", [(12, 4), (14, 2), (14, 16), (14, 32), (16, 2), (16, 16), (16, 32),
                                 (18, 2), (18, 16)])
def test_batched_solves_on_chip(gpu, L, R):
    """Every group shape (and, at L = 18, R = 16, two realizations per group):
    the residual of each realization by the batched product, itself tested
    against the oracle. ||b - A x||_2 <= max(m)^(1/2) ||b - A x||_{M^-1}, with
    the row norms m <= L, and the recurrence drifts from it by less than the
    residual itself at these sizes: the bar is twice that bound at tol 1e-11."""
    import torch
    F = np.stack([disorder_fields(L, 4.0 + r % 3, 800 + r) for r in range(R)])
    sg = np.array([-0.45 + 0.01 * r for r in range(R)])
    b = gpu.Basis(L)
    bt = gpu.Batch(b, R)
    g = torch.Generator(device="cuda").manual_seed(5)
    rhs = torch.randn((b.n, R), dtype=torch.float64, device="cuda", generator=g)
    rhs /= rhs.norm(dim=0)
    x, its, phi, st = gpu.minres_solve_batched(b, bt, F, sg, rhs, tol=1e-11)
    assert st == 0 and np.all(its > 0) and np.all(np.abs(phi) < 1e-11)
    res = (rhs - gpu.apply_H_batched(b, bt, F, sg, x)).norm(dim=0).cpu().numpy()
    print(f"L={L} R={R}: iterations {its.min()}..{its.max()}, residual {res.max():.2e}", flush=True)
    assert np.all(res <= 2 * np.sqrt(L) * 1e-11)


def test_unsolved_realization_beside_solved_ones(gpu):
    """A realization with a zero right-hand side takes no iterations and
    gets x = 0, whatever the others do."""
    import torch
    for L, R in ((12, 2), (14, 4)):
        b = gpu.Basis(L)
        bt = gpu.Batch(b, R)
        F = np.stack([disorder_fields(L, 4.0, 900 + r) for r in range(R)])
        rhs = torch.randn((b.n, R), dtype=torch.float64, device="cuda",
                          generator=torch.Generator(device="cuda").manual_seed(6))
        rhs[:, 1] = 0.0
        x, its, phi, st = gpu.minres_solve_batched(b, bt, F, [0.1] * R, rhs, tol=1e-10)
        assert st == 0 and its[1] == 0 and phi[1] == 0 and torch.all(x[:, 1] == 0)
        assert np.all(its[[r for r in range(R) if r != 1]] > 0)


@pytest.mark.parametrize("R", [8, 32])
def test_launches_per_iteration_still_solve(gpu, monkeypatch, R):
    """The form with launches per iteration (longer chains, and where the
    on-chip launch is declined), forced at L = 14."""
    import torch
    monkeypatch.setenv("MBL_MINRES_LAUNCH", "iter")
    L = 14
    b = gpu.Basis(L)
    F = np.stack([disorder_fields(L, 4.0, 950 + r) for r in range(R)])
    sg = [-0.4 + 0.02 * r for r in range(R)]
    g = torch.Generator(device="cuda").manual_seed(7)
    rhs = torch.randn((b.n, R), dtype=torch.float64, device="cuda", generator=g)
    rhs /= rhs.norm(dim=0)
    bt = gpu.Batch(b, R)
    x, its, phi, st = gpu.minres_solve_batched(b, bt, F, sg, rhs, tol=1e-12)
    assert st == 0
    X = x.cpu().numpy()
    for r in (0, R - 1):
        ref = _solve_reference(L, F[r], sg[r], rhs[:, r].cpu().numpy())
        assert np.linalg.norm(X[:, r] - ref) <= 1e-8 * np.linalg.norm(ref)
    y, info = gpu.minres_solve(b, F[0], sg[0], rhs[:, 0].contiguous())
    ref = _solve_reference(L, F[0], sg[0], rhs[:, 0].cpu().numpy())
    assert info.status == 0 and np.linalg.norm(y.cpu().numpy() - ref) <= 1e-8 * np.linalg.norm(ref)
