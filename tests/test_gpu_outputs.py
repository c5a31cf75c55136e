"""Outputs that the binding allocates: the gaps of a batch read zero, and
channels that cover the whole buffer leave none of it unwritten."""
import numpy as np
import pytest
import torch

from paper_2607_14054_amd import sosfilt as S
from paper_2607_14054_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def poison(n, dtype):
    """Blocks of the size the outputs take, left as NaN in the allocator."""
    for t in [torch.full((n,), float("nan"), device=DEV, dtype=dtype) for _ in range(4)]:
        del t


@pytest.mark.parametrize("io", ["f32", "f64"])
@pytest.mark.parametrize("gap,tail", [(0, 0), (3, 0), (0, 5)])
def test_batch_outputs_are_written_or_zero(io, gap, tail):
    dt = np.float32 if io == "f32" else np.float64
    ns = [1, 700, 33, 0, 5001, 4096]
    off = [sum(ns[:i]) + gap * i for i in range(len(ns))]
    plans = [S.Plan(W.make_sos(K, 0.5, 0.95, 50 + K), io_dtype=io, N=32) for K in (1, 8, 3, 2, 8, 16)]
    b = S.Batch(plans, ns, offsets=off)
    x = torch.from_numpy(W.make_signal(b.total + tail, 51, dt)).to(DEV)
    gy = torch.from_numpy(W.grad_seed_signal(b.total + tail, 52, dt)).to(DEV)
    y0, gx0 = torch.zeros_like(x), torch.zeros_like(x)
    S.filt_batched(b, x, y0)
    S.filt_backward_batched(b, x, gy, gx=gx0)
    poison(x.numel(), x.dtype)
    y = S.filt_batched(b, x)
    assert torch.equal(y, y0)
    del y
    poison(x.numel(), x.dtype)
    gx = S.filt_backward_batched(b, x, gy)[0]
    assert torch.equal(gx, gx0)
    del gx
    poison(x.numel(), x.dtype)
    yf, ws = S.filt_batched_for_backward(b, x)
    gx = S.filt_backward_batched_stored(b, x, gy, ws)[0]
    assert torch.equal(gx, gx0)
    want = torch.zeros_like(x)
    S.filt_batched_for_backward(b, x, y=want)
    assert torch.equal(yf, want)


def test_calls_on_another_stream():
    """The default stream's output and a side stream's agree."""
    p = S.Plan(W.make_sos(8, 0.5, 0.95, 60), io_dtype="f32")
    x = torch.from_numpy(W.make_signal(40000, 61, np.float32)).to(DEV)
    want = S.filt(p, x)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    y = S.filt(p, x, stream=s)
    with torch.cuda.stream(s):
        z = S.filt(p, x)
    s.synchronize()
    assert torch.equal(y, want) and torch.equal(z, want)
