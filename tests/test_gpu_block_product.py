"""The block-staged product of the chains split at 13 low bits, against the row
kernel.

Both sum a row's bonds and fields in the same order, so products agree bit for
bit, also with infinities and NaN among the entries. The row kernel takes a
vector that does not start on 16 bytes, and every vector of a basis split at 12.
"""
import numpy as np
import pytest

from workloads import disorder_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [20, 22, 24, 26])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_same_bits_as_the_row_kernel(gpu, L, dtype):
    import torch
    b = gpu.Basis(L)
    assert b.lo_bits == 13
    h = disorder_fields(L, 4.0, 70 + L)
    buf = torch.randn(b.n + 1, dtype=getattr(torch, dtype), device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(L))
    x = buf[1:]
    assert x.data_ptr() % 16 != 0
    x[[0, b.n // 3, b.n - 1]] = torch.tensor([np.inf, np.nan, -np.inf], dtype=x.dtype,
                                             device="cuda")
    row = gpu.apply_H(b, h, 0.3, x)
    block = gpu.apply_H(b, h, 0.3, x.clone())
    assert torch.isnan(row).any() and torch.equal(torch.isnan(row), torch.isnan(block))
    assert torch.equal(torch.nan_to_num(row), torch.nan_to_num(block))


@pytest.mark.parametrize("L", [20, 22, 24])
def test_solver_steps_as_by_rows(gpu, L):
    """40 MINRES iterations, plain, in FP32 and with the rank-one term of the
    gradient's solve, on both splits: the rounding of the sums over workgroups
    grows to at most about 1e-13 (6e-8 the unit in FP32, 1e-4 grown) of the
    result in so few iterations."""
    import torch
    h = disorder_fields(L, 3.5, 90 + L)
    out = []
    for lo in (13, 12):
        b = gpu.Basis(L, lo)
        rhs = torch.randn(b.n, dtype=torch.float64, device="cuda",
                          generator=torch.Generator(device="cuda").manual_seed(3))
        x, info = gpu.minres_solve(b, h, 0.1, rhs, kmax=40)
        x32, _ = gpu.minres_solve(b, h, 0.1, rhs, kmax=40, precision="fp32_inner",
                                  ws=gpu.Workspace(b, 0, "fp32_inner"))
        assert info.iters == 40
        v = rhs / rhs.norm()
        dE, dz2, z, _ = gpu.eig_grad(b, h, 0.1, v, kmax=40)
        out.append((x, x32, dE, dz2, z))
    a, c = out
    assert (a[0] - c[0]).norm() <= 1e-11 * c[0].norm()
    assert (a[1] - c[1]).norm() <= 1e-3 * c[1].norm()
    assert np.allclose(a[2], c[2], rtol=0, atol=1e-11 * np.abs(c[2]).max())
    assert np.allclose(a[3], c[3], rtol=0, atol=1e-9 * np.abs(c[3]).max())
    assert abs(a[4] - c[4]) <= 1e-11


# high bonds up to 8, 12 and 16 in the batched kernel; 11, 12 and 13 low bits
@pytest.mark.parametrize("L,R,grid", [(18, 32, 0), (20, 8, 0), (20, 16, 0), (20, 32, 512),
                                      (22, 4, 64), (22, 32, 0), (24, 16, 0), (26, 4, 0),
                                      (26, 16, 0)])
def test_batched_fp32_same_bits_as_the_row_kernel(gpu, L, R, grid):
    import torch
    b = gpu.Basis(L)
    bt = gpu.Batch(b, R)
    f = np.stack([disorder_fields(L, 4.0, 40 * L + r) for r in range(R)])
    sg = np.linspace(-0.4, 0.4, R)
    buf = torch.randn(b.n * R + 1, dtype=torch.float32, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(L + R))
    x = buf[1:].view(b.n, R)
    x[0, 0], x[b.n // 2, R - 1] = np.inf, np.nan
    row = gpu.apply_H_batched(b, bt, f, sg, x)
    bt.set_schedule(grid, 0, 0)
    block = gpu.apply_H_batched(b, bt, f, sg, x.clone())
    assert torch.isnan(row).any() and torch.equal(torch.isnan(row), torch.isnan(block))
    assert torch.equal(torch.nan_to_num(row), torch.nan_to_num(block))


def test_batched_fp32_solves_by_blocks(gpu):
    """FP32 inner solves with FP64 refinement reach the FP64 tolerance; the bar
    is 2 max(m)^(1/2) tol for row norms m <= L, as the residual is measured in
    the preconditioner's norm."""
    import torch
    L, R = 18, 32
    b = gpu.Basis(L)
    bt = gpu.Batch(b, R)
    f = np.stack([disorder_fields(L, 5.0, 300 + r) for r in range(R)])
    sg = np.linspace(-0.6, -0.5, R)
    rhs = torch.randn((b.n, R), dtype=torch.float64, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(4))
    rhs /= rhs.norm(dim=0)
    x, its, phi, st = gpu.minres_solve_batched(b, bt, f, sg, rhs, tol=1e-9,
                                               precision="fp32_inner")
    res = (rhs - gpu.apply_H_batched(b, bt, f, sg, x)).norm(dim=0).max().item()
    print(f"iterations {its.min()}..{its.max()}, residual {res:.1e}", flush=True)
    assert st == 0 and res <= 2 * np.sqrt(L) * 1e-9
