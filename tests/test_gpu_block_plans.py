"""When the plans of the batched block-staged FP32 product are laid out. The call of a new schedule is host work only, as a program
may make it between launches and under capture."""
import numpy as np
import pytest

from test_gpu_minres_refused import _kernels
from workloads import disorder_fields

pytestmark = pytest.mark.gpu


def _case(gpu, L, R):
    import torch
    b = gpu.Basis(L)
    f = np.stack([disorder_fields(L, 4.0, 7 * L + r) for r in range(R)])
    x = torch.randn((b.n, R), dtype=torch.float32, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(R))
    return b, gpu.Batch(b, R), f, np.linspace(-0.4, 0.4, R), x


def test_a_new_schedule_is_host_work(gpu):
    b, bt, f, sg, x = _case(gpu, 22, 4)
    calls = _kernels(lambda: bt.set_schedule(64, 0, 0))
    assert not [c for c in ("Malloc", "Memcpy", "StreamSynchronize") if c in calls], calls


def test_new_schedule_and_product_under_capture(gpu):
    """Captured before its plan exists, the product goes by rows: the same
    bits, replay after replay, with eager products (which lay the plan out)
    between them."""
    import torch
    b, bt, f, sg, x = _case(gpu, 20, 16)
    want = gpu.apply_H_batched(b, bt, f, sg, x)
    y = torch.zeros_like(x)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        bt.set_schedule(64, 0, 0)
        gpu.apply_H_batched(b, bt, f, sg, x, y)
    for _ in range(3):
        y.zero_()
        g.replay()
        assert torch.equal(y, want)
        assert torch.equal(gpu.apply_H_batched(b, bt, f, sg, x), want)
        torch.cuda.synchronize()
