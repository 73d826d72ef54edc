"""The library's own split of the longest chains is one that its entry points
take (1 .. 13 low bits) and its kernels' tables in LDS are made for."""
import pytest

from workloads import disorder_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [28, 30, 32])
def test_default_split_of_long_chains(gpu, L):
    """Rows are in numeric order in every split and a row's bonds are summed in
    the same order, so products at two splits agree bit for bit."""
    import torch
    b = gpu.Basis(L)
    assert b.lo_bits == 13
    h = disorder_fields(L, 4.0, 60 + L)
    x = torch.randn(b.n, dtype=torch.float32, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(L))
    y = gpu.apply_H(b, h, 0.3, x)
    del b
    z = gpu.apply_H(gpu.Basis(L, 12), h, 0.3, x)
    assert torch.equal(y, z)
