"""Strip path of AUTO plans (one lane per strip of the time axis; start states
from products on the matrix cores) against the FP64 oracle: sizes on both
sides of its strip lengths, lengths whose last strip is too short for its
start state, impulses at strip boundaries, run-ins inside one strip, over a
few strips and over more than sixteen."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_14054_amd import sosfilt as S
from paper_2607_14054_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run(sos, x, io, N=64):
    p = S.Plan(sos, io_dtype=io, N=N)
    xt = torch.from_numpy(x).to(DEV)
    y = torch.full_like(xt, float("nan"))
    S.filt(p, xt, y)
    torch.cuda.synchronize()
    return y.cpu().numpy()


def check(y, x, sos, io):
    if io == "f32":
        err = oracle.rel_rms(y, oracle.sosfilt(x, sos))
        assert err < 1e-6, err
        return
    # the bar of the FP64 paths: 1e-12, or 4 times the oracle's own distance
    # from its long-double twin
    ld = oracle.sosfilt_ld(x, sos)
    err, own = oracle.rel_rms(y, ld), oracle.rel_rms(oracle.sosfilt(x, sos), ld)
    assert err <= max(1e-12, 4 * own), (err, own)


# FP64 strips from 2^21 samples at K = 5 .. 8, and from 3e6 with slow poles at
# any K: a multiple of the strip, one sample more, and a last strip just below
# and at the length that holds its start state (34 samples; 66 for K > 8)
@pytest.mark.parametrize("n", [1 << 21, (1 << 21) + 1, (1 << 21) + 33, (1 << 21) + 34, (1 << 21) + 127,
                               (1 << 23) + 200, 12000001])
@pytest.mark.parametrize("K", [5, 8])
def test_strips_f64(n, K):
    sos = W.make_sos(K, 0.8, 0.98, 900 + K)
    x = W.make_signal(n, 901, np.float64)
    check(run(sos, x, "f64"), x, sos, "f64")


@pytest.mark.parametrize("io", ["f64", "f32"])
@pytest.mark.parametrize("K", [1, 4, 9, 16])
def test_strips_slow_poles(io, K):
    """Run-ins of tens of thousands of samples: more than sixteen strips."""
    sos = W.make_sos(K, 0.99, 0.999, 910 + K)
    n = 3100003
    x = W.make_signal(n, 911, np.float64 if io == "f64" else np.float32)
    check(run(sos, x, io), x, sos, io)


@pytest.mark.parametrize("K,r_hi,n", [(1, 0.9, 10000003), (8, 0.95, 16777216 + 36), (3, 0.98, 33000001),
                                      (12, 0.95, 30000005), (16, 0.9, 67108864 + 61)])
def test_strips_f32(K, r_hi, n):
    """FP32 from 1e7 samples (3e7 for K > 8): run-ins over several strips and
    inside one."""
    sos = W.make_sos(K, 0.5, r_hi, 920 + K)
    x = W.make_signal(n, 921, np.float32)
    check(run(sos, x, "f32", N=32), x, sos, "f32")


@pytest.mark.parametrize("offset", [-3, -2, -1, 0, 1])
def test_strips_impulse_across_strips(offset):
    """Unit impulses around strip boundaries (strips of 256 and of 128
    samples): the response crosses into the strips after it, through the raw
    input's history and the states."""
    sos = W.make_sos(6, 0.9, 0.98, 930)
    n = 1 << 21
    x = np.zeros(n)
    for strip in (128, 256):
        for at in (1, 63, 64, 1000):
            x[strip * 5 * at + offset] += 1.0
    check(run(sos, x, "f64"), x, sos, "f64")


def test_strips_only_n_outputs_written():
    """Neither the state areas nor the last strip's tail reach past n."""
    sos = W.make_sos(8, 0.8, 0.98, 940)
    n = (1 << 21) + 5
    p = S.Plan(sos, io_dtype="f64", N=64)
    x = torch.from_numpy(W.make_signal(n, 941, np.float64)).to(DEV)
    buf = torch.full((n + 4096,), 7.0, dtype=torch.float64, device=DEV)
    S.filt(p, x, buf[:n])
    torch.cuda.synchronize()
    assert bool((buf[n:] == 7.0).all()) and bool(torch.isfinite(buf[:n]).all())


def test_strips_graph_replays_match_eager():
    """The strip launches captured in a HIP graph: every replay, with new
    inputs, equals the eager call bit for bit."""
    sos = W.make_sos(8, 0.9, 0.999, 950)
    n = 3000017
    p = S.Plan(sos, io_dtype="f32", N=32)
    xin = torch.empty(n, dtype=torch.float32, device=DEV)
    yout = torch.empty_like(xin)
    stream = torch.cuda.Stream()
    xin.normal_()
    with torch.cuda.stream(stream):
        S.filt_static(p, xin, yout, stream)
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        S.filt_static(p, xin, yout, stream)
    for seed in range(3):
        xin.copy_(torch.from_numpy(W.make_signal(n, 951 + seed, np.float32)))
        ref = S.filt(p, xin.clone())
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(yout, ref)
