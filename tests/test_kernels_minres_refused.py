"""MINRES whose on-chip launch does not end well: the failure flags of its
groups are set before the launch (MBL_MINRES_LAUNCH=refused), as a wait that
ran out sets them, so every workgroup leaves at its next long wait or finishes,
and the call solves again with launches per iteration.

Bars: those of the on-chip solves, ||x - x_ref|| <= 1e-8 ||x_ref|| at L = 14 and
a residual of at most 2 max(m)^(1/2) tol (row norms m <= L) beyond; x0 has unit
norm, so that the rounding of b - A x, some 1e-12 of its start at L = 18, is far
below the tolerance."""
import numpy as np
import pytest

from kernel_trace import launched
from test_gpu_resident import _solve_reference
from workloads import disorder_fields, gaussian_vector

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [14, 16, 18])
def test_initial_guess_survives_a_refused_launch(gpu, monkeypatch, L):
    """The fallback starts from the residual of x0, so x must still hold x0."""
    import torch
    monkeypatch.setenv("MBL_MINRES_LAUNCH", "refused")
    f, sigma, tol = disorder_fields(L, 4.0, 1100 + L), -0.31, 1e-10
    b = gpu.Basis(L)
    rhs = torch.as_tensor(gaussian_vector(b.n, 81), device="cuda")
    rhs /= rhs.norm()
    x0 = torch.as_tensor(gaussian_vector(b.n, 82), device="cuda")
    x0 /= x0.norm()
    x, info = gpu.minres_solve(b, f, sigma, rhs, x=x0.clone(), tol=tol)
    res = (rhs - gpu.apply_H(b, f, sigma, x)).norm().item()
    print(f"L={L}: {info.iters} iterations, residual {res:.2e}", flush=True)
    assert info.status == 0 and res <= 2 * np.sqrt(L) * tol
    if L == 14:
        ref = _solve_reference(L, f, sigma, rhs.cpu().numpy())
        assert np.linalg.norm(x.cpu().numpy() - ref) <= 1e-8 * np.linalg.norm(ref)


def test_batch_survives_a_refused_launch(gpu, monkeypatch):
    import torch
    monkeypatch.setenv("MBL_MINRES_LAUNCH", "refused")
    L, R = 14, 16
    b = gpu.Basis(L)
    bt = gpu.Batch(b, R)
    F = np.stack([disorder_fields(L, 4.0, 1150 + r) for r in range(R)])
    rhs = torch.randn((b.n, R), dtype=torch.float64, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(8))
    rhs /= rhs.norm(dim=0)
    x, its, phi, st = gpu.minres_solve_batched(b, bt, F, [0.1] * R, rhs, tol=1e-10)
    assert st == 0 and np.all(its > 0)
    res = (rhs - gpu.apply_H_batched(b, bt, F, [0.1] * R, x)).norm(dim=0).max().item()
    assert res <= 2 * np.sqrt(L) * 1e-10


@pytest.mark.parametrize("batched", [False, True])
def test_solves_after_a_refused_launch_take_launches_per_iteration(gpu, monkeypatch, batched):
    """A wait that runs out costs a second, so the solves of that basis pass the
    on-chip form by for ten; another basis does not."""
    import time
    import torch
    L = 14
    b, other = gpu.Basis(L), gpu.Basis(L)
    f = disorder_fields(L, 4.0, 1190)
    rhs = torch.as_tensor(gaussian_vector(b.n, 83), device="cuda")

    def solve(basis):
        gpu.minres_solve(basis, f, 0.1, rhs, kmax=60)

    monkeypatch.setenv("MBL_MINRES_LAUNCH", "refused")
    if batched:
        two = torch.stack([rhs, rhs], dim=1).contiguous()
        gpu.minres_solve_batched(b, gpu.Batch(b, 2), [f, f], [0.1, 0.1], two, kmax=60)
    else:
        solve(b)
    end = time.monotonic() + 10.5
    monkeypatch.delenv("MBL_MINRES_LAUNCH")
    ks, _ = launched(lambda: solve(b))
    assert "k_minres_qdx" in ks and "k_minres_group" not in ks
    ks, _ = launched(lambda: solve(other))
    assert "k_minres_group" in ks and "k_minres_qdx" not in ks
    if not batched:
        time.sleep(max(0.0, end - time.monotonic()))
        assert "k_minres_group" in launched(lambda: solve(b))[0]
