"""Channels of a batch by strips are independent: NaN and Inf in a neighbour's
last and first samples, or in the gaps, leave a channel's results as they are,
bit for bit, at every offset mod 4."""
import numpy as np
import pytest
import torch

from paper_2607_14054_amd import sosfilt as S
from paper_2607_14054_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def layout(ns):
    """Every second channel has neighbours directly at both ends; offsets run
    through 0 .. 3 mod 4."""
    off, at = [], 0
    for i, n in enumerate(ns):
        off.append(at)
        at += n + (0, 0, 1, 3)[i % 4]
    return off


def poison(t, ns, off, which):
    """The gaps, and the ends of the channels that are not looked at."""
    t = t.clone()
    covered = torch.zeros(t.numel(), dtype=torch.bool, device=DEV)
    for i, (n, o) in enumerate(zip(ns, off)):
        covered[o:o + n] = True
        if i not in which:
            t[o:o + 2] = float("inf")
            t[o + n - 3:o + n] = float("nan")
    t[~covered] = float("nan")
    return t


@pytest.mark.parametrize("bad", ["x", "gy", "both"])
def test_adjoint_strips_and_their_neighbours(bad):
    ns = [200001, 150002, 262147, 180001, 300002, 131073, 170003, 200000, 250001, 140002]
    off = layout(ns)
    plans = [S.Plan(W.make_sos(8, 0.5, 0.95, 1400 + i), io_dtype="f32") for i in range(len(ns))]
    b = S.Batch(plans, ns, off)
    x = torch.from_numpy(W.make_signal(b.total + 8, 1401, np.float32)).to(DEV)
    gy = torch.from_numpy(W.grad_seed_signal(b.total + 8, 1402, np.float32)).to(DEV)
    gx0, gs0, first = S.filt_backward_batched(b, x, gy)
    y0, _ = S.filt_batched_for_backward(b, x)
    assert {o % 4 for o in off} == {0, 1, 2, 3}
    for which in (set(range(0, len(ns), 2)), set(range(1, len(ns), 2))):
        xp = poison(x, ns, off, which) if bad != "gy" else x
        gp = poison(gy, ns, off, which) if bad != "x" else gy
        y, ws = S.filt_batched_for_backward(b, xp)
        for gx, gs, _ in (S.filt_backward_batched(b, xp, gp), S.filt_backward_batched_stored(b, xp, gp, ws)):
            for i in which:
                o, n, r = off[i], ns[i], int(first[i])
                assert torch.equal(y[o:o + n], y0[o:o + n]), i
                assert torch.equal(gx[o:o + n], gx0[o:o + n]), i
                assert torch.equal(gs[r:r + 8], gs0[r:r + 8]), i


@pytest.mark.parametrize("io", ["f32", "f64"])
@pytest.mark.parametrize("K", [8, 12])
def test_filter_strips_and_their_neighbours(io, K):
    ns = [(1 << 20) + 1, 600002, 700003, 1 << 20, 500001, 800002]
    off = layout(ns)
    plans = [S.Plan(W.make_sos(K, 0.99, 0.999, 1410 + i), io_dtype=io, N=32) for i in range(len(ns))]
    b = S.Batch(plans, ns, off)
    x = torch.from_numpy(W.make_signal(b.total + 8, 1411, np.float32 if io == "f32" else np.float64)).to(DEV)
    y0 = S.filt_batched(b, x)
    for which in (set(range(0, len(ns), 2)), set(range(1, len(ns), 2))):
        y = S.filt_batched(b, poison(x, ns, off, which))
        for i in which:
            assert torch.equal(y[off[i]:off[i] + ns[i]], y0[off[i]:off[i] + ns[i]]), i
