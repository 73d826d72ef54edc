"""When the plans of the batched block-staged FP32 product are laid out, and
what counts them. The call of a new schedule is host work only, as a program
may make it between launches and under capture."""
import ctypes as C

import numpy as np
import pytest

from kernel_trace import launched, runtime_calls
from workloads import disorder_fields

pytestmark = pytest.mark.gpu


def _bytes(gpu, bt):
    v = C.c_int64()
    assert gpu.lib.mbl_batch_bytes(bt.handle, C.byref(v)) == gpu.OK
    return v.value


def _case(gpu, L, R):
    import torch
    b = gpu.Basis(L)
    f = np.stack([disorder_fields(L, 4.0, 7 * L + r) for r in range(R)])
    x = torch.randn((b.n, R), dtype=torch.float32, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(R))
    return b, gpu.Batch(b, R), f, np.linspace(-0.4, 0.4, R), x


def test_a_new_schedule_is_host_work(gpu):
    b, bt, f, sg, x = _case(gpu, 22, 4)
    calls = runtime_calls(lambda: bt.set_schedule(64, 0, 0))
    assert not [c for c in ("Malloc", "Memcpy", "StreamSynchronize") if c in calls], calls


def test_plans_are_counted_and_laid_out_once(gpu):
    """The default grid's with the workspace, a new grid's with its first FP32
    product; FP64 products need none."""
    b, bt, f, sg, x = _case(gpu, 22, 4)
    blocks, words = 0, 18 * (2 ** 13 + 32 * 14)     # split 13: 9 high bits
    for hi in range(2 ** 9):
        blocks += 0 <= 11 - bin(hi).count("1") <= 13
    plan = 96 * blocks + 4 * words
    two = gpu.Batch(b, 2)                           # R = 2: no plan; all else in proportion
    assert _bytes(gpu, bt) - 2 * _bytes(gpu, two) >= plan - 64 * 1024
    assert "k_bapply_blocks" in launched(lambda: gpu.apply_H_batched(b, bt, f, sg, x))[0]
    at_start = _bytes(gpu, bt)
    bt.set_schedule(64, 0, 0)
    gpu.apply_H_batched(b, bt, f, sg, x.double())
    assert _bytes(gpu, bt) == at_start
    for _ in range(2):
        assert "k_bapply_blocks" in launched(lambda: gpu.apply_H_batched(b, bt, f, sg, x))[0]
        assert plan <= _bytes(gpu, bt) - at_start <= plan + 4096
    bt.set_schedule(0, 0, 0)
    assert "k_bapply_blocks" in launched(lambda: gpu.apply_H_batched(b, bt, f, sg, x))[0]
    assert _bytes(gpu, bt) - at_start <= plan + 4096


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
