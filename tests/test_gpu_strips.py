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


@pytest.mark.parametrize("io", ["f64", "f32"])
@pytest.mark.parametrize("n", [1 << 18, (1 << 18) + 1, (1 << 18) + 3, (1 << 18) + 31, (1 << 18) + 32, 300001])
@pytest.mark.parametrize("K", [4, 8, 12])
def test_strips_slow_poles_short(io, n, K):
    """From 2^18 samples in strips of 128 (K <= 8): a last strip of one sample,
    and just below and at a state's room (32 samples, FP64 16)."""
    sos = W.make_sos(K, 0.9, 0.999, 915 + K)
    x = W.make_signal(n, 916, np.float64 if io == "f64" else np.float32)
    check(run(sos, x, io), x, sos, io)


@pytest.mark.parametrize("K,r_hi,n", [(1, 0.9, 10000003), (5, 0.95, 1500001), (8, 0.98, 5000003),
                                      (6, 0.95, 9000002), (2, 0.98, 20000031), (8, 0.95, 16777216 + 36), (3, 0.98, 33000001),
                                      (12, 0.95, 30000005), (16, 0.9, 67108864 + 61)])
def test_strips_f32(K, r_hi, n):
    """FP32 from 1e7 samples (3e7 for K > 8): run-ins over several strips and
    inside one."""
    sos = W.make_sos(K, 0.5, r_hi, 920 + K)
    x = W.make_signal(n, 921, np.float32)
    check(run(sos, x, "f32", N=32 if n > 20000000 else 64), x, sos, "f32")


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


def _batch(lengths, Ks, offsets, r, seed, io, N):
    sos = [W.make_sos(k, r[0], r[1], seed + c) for c, k in enumerate(Ks)]
    plans = [S.Plan(s, io_dtype=io, N=N) for s in sos]
    return sos, plans, list(lengths), list(offsets)


def _check_batch(yb, xb, sos, lengths, offsets, io, plans=None):
    """Strips at the bar of the FP64 paths; channels below 16384 samples stay
    with the tiles, whose FP64 scans are 6.5e-11 off for K = 16 at r > 0.99:
    they are held to twice the error of the tiles' single-signal call."""
    gap = np.ones(len(xb), bool)
    for c, (s, n, o) in enumerate(zip(sos, lengths, offsets)):
        gap[o:o + n] = False
        ref = oracle.sosfilt(xb[o:o + n], s)
        if io == "f32":
            assert oracle.rel_rms(yb[o:o + n], ref) < 1e-6
        else:
            ld = oracle.sosfilt_ld(xb[o:o + n], s)
            bar = max(1e-12, 4 * oracle.rel_rms(ref, ld))
            if n < 16384:
                one = S.filt(plans[c], torch.from_numpy(xb[o:o + n].copy()).to(DEV)).cpu().numpy()
                bar = max(bar, 2 * oracle.rel_rms(one, ld))
            assert oracle.rel_rms(yb[o:o + n], ld) <= bar
    assert (yb[gap] == 7.0).all()


@pytest.mark.parametrize("io", ["f32", "f64"])
def test_strips_in_a_batch(io):
    """Run-ins long against the channels: long channels by strips (starts on
    and off 16-byte boundaries, K on both sides of 8), short ones by tiles in
    the same launch; the samples between channels stay."""
    lengths = [2000001, 16384, 5000, 1200007, 300, 700000, 65537, 1 << 20]
    Ks = [8, 3, 16, 1, 5, 16, 9, 2]
    offsets, at = [], 0
    for c, n in enumerate(lengths):
        at += (0, 1, 3, 2, 7, 5, 0, 6)[c]
        offsets.append(at)
        at += n
    dt = np.float32 if io == "f32" else np.float64
    sos, plans, lengths, offsets = _batch(lengths, Ks, offsets, (0.99, 0.999), 960, io, 32)
    b = S.Batch(plans, lengths, offsets)
    xb = W.make_signal(b.total + 9, 961, dt)
    y = torch.full((len(xb),), 7.0, dtype=torch.float32 if io == "f32" else torch.float64, device=DEV)
    S.filt_batched(b, torch.from_numpy(xb).to(DEV), y)
    torch.cuda.synchronize()
    _check_batch(y.cpu().numpy(), xb, sos, lengths, offsets, io, plans)


def test_strips_batch_graph_and_replans():
    """A captured launch of a batch with strips replays after replans (that fit its room), to
    channels that all take the tiles and back; so do eager launches."""
    big = _batch([1 << 21, 1 << 21, 300001], [8, 8, 4], [0, 1 << 21, (1 << 22) + 1], (0.99, 0.999), 970, "f32", 32)
    small = _batch([4000, 10000, 12000], [2, 8, 3], [5, 5000, 200000], (0.5, 0.9), 980, "f32", 32)
    b = S.Batch(big[1], big[2], big[3])
    stream = torch.cuda.Stream()
    xb = W.make_signal((1 << 22) + 300100, 971, np.float32)
    x = torch.from_numpy(xb).to(DEV)
    y = torch.full_like(x, 7.0)
    torch.cuda.synchronize()
    S.filt_batched(b, x, y, stream)
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        S.filt_batched(b, x, y, stream)
    for sos, plans, lengths, offsets in (big, small, big, small):
        b.replan(plans, lengths, offsets, stream)
        for launch in (g.replay, lambda: S.filt_batched(b, x, y, stream)):
            with torch.cuda.stream(stream):
                y.fill_(7.0)
                launch()
            stream.synchronize()
            _check_batch(y.cpu().numpy(), xb, sos, lengths, offsets, "f32")


def row_err(g, ref):
    scale = np.maximum(np.max(np.abs(ref), axis=1, keepdims=True), 1e-300)
    return float(np.max(np.abs(g - ref) / scale))


def check_adjoint(sos, x, g, gx, gs):
    # the bars of the FP32 adjoint paths: dL/dx 1e-6, dL/dsos 1e-9 of its row
    lx, ls = oracle.sosfilt_backward_ld(x, sos, g)
    assert not np.isnan(gx).any()
    ex, es = oracle.rel_rms(gx, lx), row_err(gs, ls)
    assert ex < 1e-6, ex
    assert es < 1e-9, es


# strips of 64 samples, one sample more, a last strip just below and at the
# length that holds its start state, longer ones (96, 160), the length that 16 strips of a long run-in need (r = 0.99, 0.998), and a run-in
# inside one strip (6.6e7 samples: 1024 a strip)
@pytest.mark.parametrize("n,r_hi", [(21846 * 96, 0.9), (21846 * 96 + 1, 0.95), (21846 * 96 + 35, 0.9),
                                    (21846 * 96 + 36, 0.9), (21846 * 96 + 31, 0.9),
                                    (21846 * 96 + 32, 0.9), (6000001, 0.95), (10000003, 0.9), (2100007, 0.99),
                                    (2100007, 0.998), (66000001, 0.9)])
def test_adjoint_strips(n, r_hi):
    sos = W.make_sos(8, 0.5, r_hi, 960)
    x, g = W.make_signal(n, 961, np.float32), W.grad_seed_signal(n, 961, np.float32)
    p = S.Plan(sos, io_dtype="f32")
    xt, gt = torch.from_numpy(x).to(DEV), torch.from_numpy(g).to(DEV)
    gx, gs = S.filt_backward(p, xt, gt, gx=torch.full_like(xt, float("nan")))
    y, ws = S.filt_for_backward(p, xt)
    gx2, gs2 = S.filt_backward_stored(p, xt, gt, ws)
    torch.cuda.synchronize()
    assert torch.equal(gx, gx2) and torch.equal(gs, gs2)
    check_adjoint(sos, x, g, gx.cpu().numpy(), gs.cpu().numpy())
    assert oracle.rel_rms(y.cpu().numpy(), oracle.sosfilt(x, sos)) < 1e-6


def test_adjoint_strips_batched():
    """Ragged channels at every offset mod 4 with gaps between them, long and
    short run-ins in one batch, and a replan to other lengths."""
    ns, his = [400001, 70000, 64, 262144, 300003, 150002, 4099, 500000], [0.9, 0.95, 0.9, 0.99, 0.95, 0.9, 0.98, 0.9]
    soss = [W.make_sos(8, 0.5, hi, 970 + i) for i, hi in enumerate(his)]
    plans = [S.Plan(s, io_dtype="f32") for s in soss]
    off, at = [], 0
    for i, n in enumerate(ns):
        off.append(at)
        at += n + (1, 2, 3, 5, 0, 7, 4, 6)[i]
    b = S.Batch(plans, ns, offsets=off)
    for lens in (ns, [n - 37 if n > 100 else n for n in ns]):
        if lens is not ns:
            b.replan(plans, lens, offsets=off)
        x, g = W.make_signal(b.total, 971, np.float32), W.grad_seed_signal(b.total, 971, np.float32)
        xt, gt = torch.from_numpy(x).to(DEV), torch.from_numpy(g).to(DEV)
        y, ws = S.filt_batched_for_backward(b, xt)
        gx = torch.full_like(xt, 7.0)
        out = S.filt_backward_batched_stored(b, xt, gt, ws, gx=gx)
        one = S.filt_backward_batched(b, xt, gt, gx=torch.full_like(xt, 7.0))
        torch.cuda.synchronize()
        gs = out[1]
        assert torch.equal(out[0], one[0])
        gx = gx.cpu().numpy()
        covered = np.zeros(b.total, bool)
        for i, (o, n) in enumerate(zip(off, lens)):
            covered[o:o + n] = True
            gi = gs[8 * i:8 * i + 8]
            check_adjoint(soss[i], x[o:o + n], g[o:o + n], gx[o:o + n], gi.cpu().numpy())
            assert oracle.rel_rms(y[o:o + n].cpu().numpy(), oracle.sosfilt(x[o:o + n], soss[i])) < 1e-6
        assert (gx[~covered] == 7.0).all()   # the gaps are left alone
