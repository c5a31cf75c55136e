"""FP64 strips where the first section's zeros lie near slow poles of the others:
no further from the long-double twin than 4 times the FP64 recurrence (and 1e-12),
the bar of the FP64 paths."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_14054_amd import sosfilt as S
from paper_2607_14054_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def notched(K, r, seed):
    """The first section's zeros on the angles of another's slow poles."""
    sos = W.make_sos(K, 0.9, r, seed)
    sos[-1, 4:] = [-2 * r * np.cos(0.4), r * r]
    sos[0, 1] = -2 * np.cos(0.4) * sos[0, 0]
    sos[0, 2] = sos[0, 0]
    return sos


@pytest.mark.parametrize("sos", [W.make_sos(11, 0.9, 0.999, 5060), notched(8, 0.999, 3), notched(12, 0.999, 4),
                                 notched(16, 0.999, 5)], ids=["drawn11", "notched8", "notched12", "notched16"])
@pytest.mark.parametrize("batch", [False, True])
def test_zeros_near_slow_poles(sos, batch):
    n = 1100003 if not batch else 387745
    x = W.make_signal(n, 60, np.float64)
    p = S.Plan(sos, io_dtype="f64", N=64)
    xt = torch.from_numpy(x).to(DEV)
    if batch:
        y = S.filt_batched(S.Batch([p] * 12, [n] * 12), xt.repeat(12))[5 * n:6 * n]
    else:
        y = S.filt(p, xt)
    ld = oracle.sosfilt_ld(x, sos)
    err, own = oracle.rel_rms(y.cpu().numpy(), ld), oracle.rel_rms(oracle.sosfilt(x, sos), ld)
    assert err <= max(1e-12, 4 * own), (err, own)
