"""Replans of a batch whose channels all took strips when it was created, to
sets that mix channels by strips and by tiles."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_14054_amd import sosfilt as S
from paper_2607_14054_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SLOW, FAST = (0.99, 0.999), (0.5, 0.9)


def channels(spec, seed):
    soss = [W.make_sos(K, r[0], r[1], seed + i % 5) for i, (_, K, r) in enumerate(spec)]
    return soss, [S.Plan(s, io_dtype="f32", N=32) for s in soss], [n for n, _, _ in spec]


def check(y, xb, soss, lengths):
    at = 0
    for s, n in zip(soss, lengths):
        assert oracle.rel_rms(y[at:at + n], oracle.sosfilt(xb[at:at + n], s)) < 1e-6, (n, at)
        at += n


def test_replans_to_strips_and_tiles():
    """One launch captured at creation, and eager launches, over sets with
    strips only, strips and tiles, and tiles only."""
    sets = [channels(spec, 1100) for spec in (
        [(1 << 19, 8, SLOW)] * 16,
        [(1 << 19, 8, SLOW)] * 13 + [(16000, 8, FAST), (16383, 3, FAST), (5, 1, FAST)],
        [(16000, 8, FAST), (1 << 21, 8, SLOW), ((1 << 21) + 400, 8, SLOW), (16383, 3, FAST)],
        [(1 << 19, 8, SLOW)] * 16,
        [((1 << 20) + 400, 8, SLOW)] * 4 + [(16000, 8, FAST)] * 3,
        [(4000, 2, FAST), (200000, 8, FAST), (5, 1, FAST), (12000, 3, FAST)])]
    b = S.Batch(sets[0][1], sets[0][2])
    xb = W.make_signal(b.total, 1101, np.float32)
    x = torch.from_numpy(xb).to(DEV)
    y = torch.full_like(x, float("nan"))
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    S.filt_batched(b, x, y, stream)
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        S.filt_batched(b, x, y, stream)
    for soss, plans, lengths in sets:
        b.replan(plans, lengths, stream=stream)
        assert b.total <= len(xb)
        for launch in (g.replay, lambda: S.filt_batched(b, x, y, stream)):
            with torch.cuda.stream(stream):
                y.fill_(float("nan"))
                launch()
            stream.synchronize()
            got = y.cpu().numpy()
            check(got, xb, soss, lengths)
            assert np.isnan(got[b.total:]).all()


def test_replans_of_many_equal_channels():
    """The benchmark's equal slow channels, then one of them short."""
    first = channels([(1 << 17, 8, SLOW)] * 64, 1200)
    then = channels([(1 << 17, 8, SLOW)] * 63 + [(4000, 8, FAST)], 1200)
    b = S.Batch(first[1], first[2])
    xb = W.make_signal(b.total, 1201, np.float32)
    x = torch.from_numpy(xb).to(DEV)
    for soss, plans, lengths in (first, then, first):
        b.replan(plans, lengths)
        y = torch.full_like(x, float("nan"))
        S.filt_batched(b, x, y)
        torch.cuda.synchronize()
        check(y.cpu().numpy(), xb, soss, lengths)
