"""Edges of the strip path: cascades whose run-in is shorter than a state area,
with guard samples around the outputs."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_14054_amd import sosfilt as S
from paper_2607_14054_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def held(y, x, sos, io):
    """The bars of the filter paths: FP32 1e-6; FP64 1e-12, or 4 times the
    oracle's own distance from its long-double twin."""
    if io == "f32":
        return oracle.rel_rms(y, oracle.sosfilt(x, sos)) < 1e-6
    ld = oracle.sosfilt_ld(x, sos)
    return oracle.rel_rms(y, ld) <= max(1e-12, 4 * oracle.rel_rms(oracle.sosfilt(x, sos), ld))


# no poles, and poles near 0: run-ins of 2 to 30 samples; 31 to 32 samples a
# lane, with a remainder below a state's room, above it, and none
@pytest.mark.parametrize("n", [31 * 65536 + 1, 2050001, 32 * 65536 - 17, 32 * 65536])
@pytest.mark.parametrize("io,K,r", [("f32", 8, 0.0), ("f32", 5, 0.05), ("f32", 4, 0.2), ("f64", 8, 0.0),
                                    ("f64", 5, 0.02)])
def test_short_run_ins_write_only_their_outputs(io, K, r, n):
    sos = W.make_sos(K, r, r, 1000 + K)
    x = W.make_signal(n, 1001, np.float32 if io == "f32" else np.float64)
    p = S.Plan(sos, io_dtype=io, N=64)
    xt = torch.from_numpy(x).to(DEV)
    buf = torch.full((n + 2048,), 7.0, dtype=xt.dtype, device=DEV)
    S.filt(p, xt, buf[1024:1024 + n])
    torch.cuda.synchronize()
    assert bool((buf[:1024] == 7.0).all()) and bool((buf[1024 + n:] == 7.0).all())
    assert held(buf[1024:1024 + n].cpu().numpy(), x, sos, io)


@pytest.mark.parametrize("io", ["f32", "f64"])
@pytest.mark.parametrize("K,r", [(16, 0.0), (16, 0.05), (9, 0.1), (3, 0.1)])
def test_short_run_ins_among_slow_channels(io, K, r):
    """Channels with short run-ins at every offset mod 4, each directly behind
    a channel with slow poles and before a gap of 0 to 3 samples."""
    ns, Ks, rs = [], [], []
    for n in (16384, 20170, 20163, 20192, 17001):
        ns += [(1 << 20) + (len(ns) // 2) % 4, n]
        Ks += [8, K]
        rs += [(0.99, 0.999), (r, r)]
    off, at = [], 0
    for i, n in enumerate(ns):
        off.append(at)
        at += n + (i // 2 % 4 if i % 2 else 0)
    soss = [W.make_sos(k, lo, hi, 1010 + i) for i, (k, (lo, hi)) in enumerate(zip(Ks, rs))]
    plans = [S.Plan(s, io_dtype=io, N=32) for s in soss]
    b = S.Batch(plans, ns, off)
    x = W.make_signal(b.total + 5, 1011, np.float32 if io == "f32" else np.float64)
    y = torch.full((len(x),), 7.0, dtype=torch.float32 if io == "f32" else torch.float64, device=DEV)
    S.filt_batched(b, torch.from_numpy(x).to(DEV), y)
    torch.cuda.synchronize()
    y = y.cpu().numpy()
    gap = np.ones(len(x), bool)
    for s, n, o in zip(soss, ns, off):
        gap[o:o + n] = False
        assert held(y[o:o + n], x[o:o + n], s, io), (n, o)
    assert (y[gap] == 7.0).all()
