"""That the comparisons of the block-staged products with the row kernels do
compare the two, by the names of the launched kernels; and the chain lengths
that those comparisons leave out."""
import numpy as np
import pytest

from kernel_trace import launched
from workloads import disorder_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [20, 22, 24, 26, 28, 30])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_single_product(gpu, L, dtype):
    """A vector that does not start on 16 bytes goes by rows, one that does by
    blocks: the same sums in the same order, so the same bits."""
    import torch
    b = gpu.Basis(L)
    h = disorder_fields(L, 4.0, 80 + L)
    buf = torch.randn(b.n + 1, dtype=getattr(torch, dtype), device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(L))
    x = buf[1:]
    assert x.data_ptr() % 16 != 0
    ks, row = launched(lambda: gpu.apply_H(b, h, 0.3, x))
    assert "k_apply<" in ks and "k_apply_block<" not in ks
    x = x.clone()
    ks, block = launched(lambda: gpu.apply_H(b, h, 0.3, x))
    assert "k_apply_block<" in ks and "k_apply<" not in ks
    assert torch.equal(row, block)


@pytest.mark.parametrize("L,R,grid", [(18, 32, 0), (20, 8, 0), (20, 16, 0), (20, 32, 512),
                                      (22, 4, 64), (22, 32, 0), (24, 16, 0), (26, 4, 0),
                                      (26, 16, 0), (28, 4, 0)])
def test_batched_fp32_product(gpu, L, R, grid):
    import torch
    b = gpu.Basis(L)
    bt = gpu.Batch(b, R)
    bt.set_schedule(grid, 0, 0)
    f = np.stack([disorder_fields(L, 4.0, 50 * L + r) for r in range(R)])
    sg = np.linspace(-0.4, 0.4, R)
    buf = torch.randn(b.n * R + 1, dtype=torch.float32, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(L + R))
    x = buf[1:].view(b.n, R)
    ks, row = launched(lambda: gpu.apply_H_batched(b, bt, f, sg, x))
    assert "k_bapply<" in ks and "k_bapply_blocks<" not in ks
    x = x.clone()
    ks, block = launched(lambda: gpu.apply_H_batched(b, bt, f, sg, x))
    assert "k_bapply_blocks<" in ks and "k_bapply<" not in ks
    assert torch.equal(row, block)


@pytest.mark.parametrize("L", [20, 22, 24, 28, 30])
def test_minres_products(gpu, L):
    """At split 13 the solves take the block-staged product, at 12 the row
    kernel, single in both precisions and batched in FP32. After 20 iterations
    the sums of the two over workgroups have rounded to at most 1e-13 of the
    result (1e-4 in FP32)."""
    import torch
    h = disorder_fields(L, 3.5, 95 + L)
    xs = {}
    for lo, name, other in ((13, "k_apply_block<", "k_apply<"), (12, "k_apply<", "k_apply_block<")):
        b = gpu.Basis(L, lo)
        rhs = torch.randn(b.n, dtype=torch.float64, device="cuda",
                          generator=torch.Generator(device="cuda").manual_seed(3))
        for precision, T in (("fp64", "double"), ("fp32_inner", "float")):
            ks, (x, info) = launched(lambda: gpu.minres_solve(b, h, 0.1, rhs, kmax=20,
                                                              precision=precision))
            assert f"{name}{T}, 1, true" in ks and f"{other}{T}, 1" not in ks
            xs[lo, precision] = x
    for precision, bar in (("fp64", 1e-11), ("fp32_inner", 1e-3)):
        d = xs[13, precision] - xs[12, precision]
        assert d.norm() <= bar * xs[12, precision].norm()


@pytest.mark.parametrize("L", [20, 22, 24])
def test_batched_minres_products(gpu, L):
    import torch
    R, b = 8, gpu.Basis(L)
    h = disorder_fields(L, 3.5, 95 + L)
    rhs = torch.randn((b.n, R), dtype=torch.float64, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(4))
    ks, _ = launched(lambda: gpu.minres_solve_batched(
        b, gpu.Batch(b, R), [h] * R, [0.1] * R, rhs, kmax=20, precision="fp32_inner"))
    assert f"k_bapply_blocks<{R}" in ks and "k_bapply<float" not in ks
