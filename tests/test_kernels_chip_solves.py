"""On-chip MINRES (FP64, L <= 18) where the other tests of it do not reach: an
initial guess and the Jacobi preconditioner at each group shape of the single
solve, the gradient's rank-one term, solves from two threads at once."""
import threading

import numpy as np
import pytest

from kernel_trace import launched
from oracle import adjoint, minres, model, precond, twist
from workloads import disorder_fields, gaussian_vector

pytestmark = pytest.mark.gpu


def _unit(v):
    return v / np.linalg.norm(v)


@pytest.mark.parametrize("L,kind", [(14, "jacobi"), (16, "row"), (16, "id"), (16, "jacobi"),
                                    (18, "row"), (18, "id")])
def test_single_solve_residual(gpu, L, kind):
    """From x0 = 0 and from a guess: ||b - A x||_2 <= max(m)^(1/2)
    ||b - A x||_{M^-1}, and the recurrence's drift is below the residual (the
    oracle's Alg. 2 with the Jacobi preconditioner: 1.7e-10 and 1.5e-10 at
    L = 14 and 16 for tol 1e-10), so the bar is twice that bound."""
    import torch
    f, sigma, tol = disorder_fields(L, 4.0, 1300 + L), -0.31, 1e-10
    b = gpu.Basis(L)
    m = precond.preconditioner_diagonal(model.hamiltonian_csr(L, f), sigma, kind)
    rhs = torch.as_tensor(_unit(gaussian_vector(b.n, 93)), device="cuda")
    guess = torch.as_tensor(_unit(gaussian_vector(b.n, 96)), device="cuda")
    for x0 in (torch.zeros_like(rhs), guess):
        x, info = gpu.minres_solve(b, f, sigma, rhs, x=x0.clone(), tol=tol, precond=kind)
        res = (rhs - gpu.apply_H(b, f, sigma, x)).norm().item()
        print(f"L={L} {kind}: {info.iters} iterations, residual {res:.2e}", flush=True)
        assert info.status == 0 and res <= 2 * np.sqrt(m.max()) * tol


@pytest.mark.parametrize("L", [14, 16])
def test_gradient_against_the_oracle(gpu, L):
    """d|z|^2/dh of a mid-spectrum pair against the oracle's Alg. 2 on the same
    deflated system with the same psi. Both solves end at tol in the M^-1 norm;
    off psi the operator is at least the gap g to the nearest level, so each
    solution is within sqrt(max m) tol / g, and d|z|^2/dh = lambda . (psi s_j),
    |s_j| = 1/2, |psi| = 1, within half of that."""
    import torch
    from workloads import start_vector
    tol = 1e-11
    h = disorder_fields(L, 3.0, 1330 + L)
    b = gpu.Basis(L)
    lo, hi, sg = gpu.sigma_midpoint(b, h, 1e-12)
    r = gpu.si_lanczos(b, h, sg, 4, escale=max(abs(lo), abs(hi)),
                       v0=torch.as_tensor(start_vector(b.n, 5), device="cuda"))
    assert r.nconv == 4
    E, psi = r.evals[1], r.evecs[:, 1].contiguous()
    gap = min(r.evals[1] - r.evals[0], r.evals[2] - r.evals[1])
    ks, (dE, dz2, z, info) = launched(lambda: gpu.eig_grad(b, h, E, psi, tol=tol))
    assert "k_minres_group" in ks
    assert info.status == 0
    c = psi.cpu().numpy()
    H = model.hamiltonian_csr(L, h)
    A, m = precond.shifted(H, E), precond.preconditioner_diagonal(H, E, "row")
    u = twist.twist_phases(L)
    zc = np.sum(c ** 2 * u)
    g = 4 * c * np.real(np.conj(zc) * u)
    c2 = c @ c
    g -= c * (c @ g) / c2
    lam, k, _ = minres.minres(lambda v: A @ v + c * (c @ v) / c2, np.zeros_like(g), g, 1 / m,
                              10 ** 6, tol)
    lam -= c * (c @ lam) / c2
    ref = (lam * c) @ adjoint.spin_matrix(L)
    bar = np.sqrt(m.max()) * tol / gap
    print(f"L={L}: gap {gap:.1e}, {info.iters} iterations (oracle {k}), "
          f"off by {np.abs(dz2 - ref).max():.1e}, bar {bar:.1e}", flush=True)
    assert abs(z - zc) <= 1e-12
    assert np.allclose(dE, adjoint.hellmann_feynman(L, c), rtol=0, atol=1e-12)
    # the oracle's own sums round at 1e-13 of max |dz2|
    assert np.abs(dz2 - ref).max() <= bar + 1e-12 * max(1.0, np.abs(ref).max())


def test_two_threads_solve_at_once(gpu):
    """Each thread its stream and workspace, one basis between them per length;
    a solve that the other thread's holds up falls back, so the bar is the
    residual's."""
    import torch
    tol, errs = 1e-10, []
    bases = {L: gpu.Basis(L) for L in (14, 16)}
    f = {L: disorder_fields(L, 4.0, 1360 + L) for L in bases}
    rhs = {L: torch.as_tensor(_unit(gaussian_vector(b.n, 97)), device="cuda")
           for L, b in bases.items()}
    torch.cuda.synchronize()

    def work(order):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for L in order:
                    b = bases[L]
                    x = torch.zeros(b.n, dtype=torch.float64, device="cuda")
                    x, info = gpu.minres_solve(b, f[L], -0.2, rhs[L], x=x, tol=tol,
                                               stream=s.cuda_stream)
                    y = gpu.apply_H(b, f[L], -0.2, x, stream=s.cuda_stream)
                    res = (rhs[L] - y).norm().item()
                    assert info.status == 0 and res <= 2 * np.sqrt(L) * tol, (L, res)
        except BaseException as e:   # to the main thread
            errs.append(e)

    ts = [threading.Thread(target=work, args=(o,)) for o in ((14, 16, 14, 16), (16, 14, 16, 14))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errs, errs
