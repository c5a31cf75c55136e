"""The framework's performance cases: what a program that uses it has it do.

Three kinds of call, each through the Python binding:

* ``filt``  one signal through one cascade (a plan kept by the program);
* ``batch`` ragged channels, each with its own cascade, in one launch;
* ``train`` a training step of one signal (``autograd.sosfilt`` and the
  gradients of x and the coefficients), or of a batch of channels (the
  two-call form a training loop uses).

Signals are N(0, 1).  Cascades follow ``workloads.py``: per section a pole
pair of radius U[r_lo, r_hi] and a zero pair on the unit circle, at angles
U[0, pi], scaled to unit peak gain.  ``exact`` filters in the frequency
domain in complex128, with zero padding long enough that the cascade's
response has decayed below 1e-20.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_14054_amd import autograd as A
from paper_2607_14054_amd import sosfilt as S

DEV = "cuda"


def listed():
    return [
        # a short buffer through a small equaliser, called in a loop: latency
        dict(name="filt_4k_K4", kind="filt", n=4000, io="f32", K=4, N=0, r_lo=0.5, r_hi=0.95, keep_y=False),
        # the smallest workload of the benchmark: FP64, N = 8
        dict(name="filt_64k_f64_N8", kind="filt", n=1 << 16, io="f64", K=8, N=8, r_lo=0.5, r_hi=0.95, keep_y=False),
        # a minute of a 16 kHz recording, default options, odd length
        dict(name="filt_1m_K6", kind="filt", n=1000003, io="f32", K=6, N=0, r_lo=0.8, r_hi=0.98, keep_y=False),
        # the same order of length with poles near the unit circle (narrow filters)
        dict(name="filt_1m_slow", kind="filt", n=1 << 20, io="f32", K=8, N=64, r_lo=0.9, r_hi=0.999, keep_y=False),
        # a long recording in FP64
        dict(name="filt_16m_f64", kind="filt", n=(1 << 24) + 5, io="f64", K=8, N=64, r_lo=0.8, r_hi=0.98,
             keep_y=False),
        # the benchmark's headline workload, output buffer kept
        dict(name="filt_256m", kind="filt", n=1 << 28, io="f32", K=8, N=64, r_lo=0.8, r_hi=0.98, keep_y=True),
        # a serving request: short channels, each with its own cascade
        dict(name="batch_64_short", kind="batch", channels=64, n_lo=1 << 10, n_hi=1 << 14, io="f32", K_lo=1, K_hi=16,
             N=32, r_lo=0.5, r_hi=0.95, shape_seed=1),
        # ragged channels over the benchmark's range of lengths and orders
        dict(name="batch_256_ragged", kind="batch", channels=256, n_lo=1 << 10, n_hi=1 << 22, io="f32", K_lo=1, K_hi=16,
             N=32, r_lo=0.5, r_hi=0.95, shape_seed=2),
        # equal channels with poles near the unit circle (the precision workload, a quarter of its channels)
        dict(name="batch_64x1m_slow", kind="batch", channels=64, n_lo=1 << 20, n_hi=1 << 20, io="f32", K_lo=8, K_hi=8,
             N=32, r_lo=0.9, r_hi=0.999, shape_seed=3),
        # one training example: filter coefficients learned by gradient
        dict(name="train_256k", kind="train", channels=1, n=1 << 18, io="f32", K=8, r_lo=0.5, r_hi=0.95),
        # a training batch: the benchmark's adjoint workload
        dict(name="train_64x256k", kind="train", channels=64, n=1 << 18, io="f32", K=8, r_lo=0.5, r_hi=0.95),
        # one long signal with gradients
        dict(name="train_32m", kind="train", channels=1, n=(1 << 25) + 1001, io="f32", K=8, r_lo=0.5, r_hi=0.95),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    r_lo, r_hi = rng.choice([(0.5, 0.95), (0.5, 0.95), (0.8, 0.98), (0.8, 0.98), (0.9, 0.999)])
    kind = rng.choice(["filt", "filt", "batch", "train"])
    if kind == "filt":
        io = rng.choice(["f32", "f32", "f64"])
        return dict(kind=kind, n=_log_int(rng, 1000, 1 << (28 if io == "f32" else 25)), io=io, K=rng.randint(1, 16),
                    N=rng.choice([0, 0, 8, 16, 64]), r_lo=r_lo, r_hi=r_hi, keep_y=rng.random() < 0.5)
    if kind == "batch":
        n_lo = _log_int(rng, 1000, 1 << 18)
        return dict(kind=kind, channels=rng.randint(8, 256), n_lo=n_lo, n_hi=_log_int(rng, n_lo, 1 << 20), io="f32",
                    K_lo=1, K_hi=rng.randint(2, 16), N=rng.choice([16, 32, 64]), r_lo=r_lo, r_hi=r_hi,
                    shape_seed=rng.randrange(1 << 20))
    channels = rng.choice([1, rng.randint(2, 64)])
    return dict(kind=kind, channels=channels, n=_log_int(rng, 2000, (1 << 24) // channels), io=rng.choice(["f32", "f32", "f64"]),
                K=rng.randint(1, 12), r_lo=0.5, r_hi=rng.choice([0.9, 0.95, 0.98]))


# ------------------------------------------------------------------ inputs

_GRID = np.exp(-1j * np.linspace(0.0, math.pi, 1025))


def _sos(K, r_lo, r_hi, seed):
    """[K, 6] rows (b0, b1, b2, a0, a1, a2)."""
    rng = np.random.default_rng(seed)
    rows = np.zeros((K, 6))
    for k in range(K):
        r, th, ph = rng.uniform(r_lo, r_hi), rng.uniform(0, math.pi), rng.uniform(0, math.pi)
        b = np.array([1.0, -2.0 * math.cos(ph), 1.0])
        a = np.array([1.0, -2.0 * r * math.cos(th), r * r])
        grid = np.concatenate([_GRID, [np.exp(-1j * th)]])
        peak = np.max(np.abs((b[0] + b[1] * grid + b[2] * grid ** 2) / (a[0] + a[1] * grid + a[2] * grid ** 2)))
        rows[k, :3], rows[k, 3:] = b / peak, a
    return rows


def _shape(case):
    """Lengths and sections per channel: the case's own, the same for every seed."""
    rng = np.random.default_rng(case["shape_seed"])
    n = np.floor(np.exp(rng.uniform(math.log(case["n_lo"]), math.log(case["n_hi"] + 1), case["channels"])))
    n = np.clip(n.astype(np.int64), case["n_lo"], case["n_hi"])
    return n, rng.integers(case["K_lo"], case["K_hi"] + 1, case["channels"])


def _cascades(case, seed):
    """(rows, length) of every channel."""
    if case["kind"] == "batch":
        n, K = _shape(case)
    else:
        n, K = [case["n"]] * case.get("channels", 1), [case["K"]] * case.get("channels", 1)
    return [(_sos(int(K[c]), case["r_lo"], case["r_hi"], 7919 * seed + c), int(n[c])) for c in range(len(n))]


def _signal(total, io, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randn(total, generator=g, device=DEV, dtype=torch.float32 if io == "f32" else torch.float64)


def prepare(case, seed):
    chans = _cascades(case, seed)
    x = _signal(sum(n for _, n in chans), case["io"], 2 * seed)
    st = {"kind": case["kind"], "x": x}
    if case["kind"] == "filt":
        st["plan"] = S.Plan(chans[0][0], io_dtype=case["io"], N=case["N"])
        st["y"] = torch.empty_like(x) if case["keep_y"] else None
        return st
    if case["kind"] == "train":
        st["gy"] = _signal(x.numel(), case["io"], 2 * seed + 1)
        if len(chans) == 1:
            # x and sos are what gradients are asked for; the program keeps its
            # coefficients on the host, as the binding's own examples do
            st["x"] = x.requires_grad_(True)
            st["sos"] = torch.from_numpy(chans[0][0]).requires_grad_(True)
            st["plan"] = A.cached_plan(chans[0][0], case["io"], 32, "auto", x.device)
            return st
    N = case.get("N", 32)
    st["batch"] = S.Batch([S.Plan(r, io_dtype=case["io"], N=N) for r, _ in chans], [n for _, n in chans])
    return st


def run(st):
    if st["kind"] == "filt":
        return S.filt(st["plan"], st["x"], st["y"])
    if st["kind"] == "batch":
        return S.filt_batched(st["batch"], st["x"])
    if "sos" in st:
        y = A.sosfilt(st["x"], st["sos"])
        gx, gsos = torch.autograd.grad(y, (st["x"], st["sos"]), st["gy"])
        return {"y": y.detach(), "gx": gx, "gsos": gsos}
    y, ws = S.filt_batched_for_backward(st["batch"], st["x"])
    gx, gsos, _ = S.filt_backward_batched_stored(st["batch"], st["x"], st["gy"], ws)
    return {"y": y, "gx": gx, "gsos": gsos}


def work(case):
    """Bytes: x read, y written (train: x and gy read, y, gx and the
    coefficients' gradients written).  Operations: the recurrence's four
    multiply-adds per section and sample forward; four backward and five for
    the coefficients' sums."""
    es = 4 if case["io"] == "f32" else 8
    if case["kind"] == "batch":
        n, K = _shape(case)
        return {"bytes": float(2 * es * n.sum()), "flops": float(8 * (n * K).sum())}
    total, K = case["n"] * case.get("channels", 1), case["K"]
    if case["kind"] == "filt":
        return {"bytes": 2 * es * total, "flops": 8 * total * K}
    return {"bytes": 4 * es * total + 48 * K * case["channels"], "flops": 26 * total * K}


# ------------------------------------------------------------------- exact

def _decay(rows):
    """Samples after which the cascade's response is below about 1e-20."""
    r = float(np.sqrt(np.max(rows[:, 5] / rows[:, 3])))
    return int(math.ceil((46.0 + 8.0 * len(rows)) / -math.log(r))) + 16


def _poly(c, z):
    return c[0] + c[1] * z + c[2] * z * z


def _fast_len(n):
    """A length of at least n with small prime factors."""
    p = 1 << max(0, (n - 1).bit_length() - 3)
    return p * -(-n // p)


def _grid(m):
    # z^-1 on the unit circle, the angle reduced to one octant's accuracy
    k = torch.arange(m // 2 + 1, device=DEV, dtype=torch.float64)
    w = -2.0 * math.pi / m * k
    return torch.complex(torch.cos(w), torch.sin(w))


def _filt_exact(x, rows, n):
    """The cascade of x[:n], by overlap-save in complex128."""
    d = _decay(rows)
    step = min(n, max(1 << 22, 8 * d))
    m = _fast_len(step + 2 * d)
    z = _grid(m)
    H = torch.ones_like(z)
    for r in rows:
        H = H * _poly(r[:3], z) / _poly(r[3:], z)
    y = torch.empty(n, device=DEV, dtype=torch.float64)
    for s in range(0, n, step):
        e, h = min(n, s + step), min(s, d)
        seg = torch.fft.irfft(torch.fft.rfft(x[s - h:e].double(), m) * H, m)
        y[s:e] = seg[h:h + e - s]
    return y


def _train_exact(x, gy, rows):
    n = x.numel()
    m = _fast_len(n + _decay(rows))
    z = _grid(m)
    num = [_poly(r[:3], z) for r in rows]
    den = [_poly(r[3:], z) for r in rows]
    back = lambda F: torch.fft.irfft(F, m)[:n]  # noqa: E731
    U = torch.fft.rfft(x.double(), m)
    ins = [x.double()]
    for b, a in zip(num, den):
        U = U * b / a
        ins.append(back(U))
    G = torch.fft.rfft(gy.double().flip(0), m)
    gsos = np.zeros((len(rows), 6))
    for k in range(len(rows) - 1, -1, -1):
        mu = back(G / den[k]).flip(0)
        lag = lambda v, j: float(torch.dot(mu[j:], v[:n - j]))  # noqa: E731
        db = [lag(ins[k], j) for j in range(3)]
        da = [-lag(ins[k + 1], j) for j in range(1, 3)]
        a0 = rows[k, 3]
        gsos[k, :3] = db
        gsos[k, 4:] = da
        gsos[k, 3] = -(np.dot(rows[k, :3], db) + np.dot(rows[k, 4:], da)) / a0
        G = G * num[k] / den[k]
    return ins[-1], back(G).flip(0), gsos


def exact(case, seed):
    chans = _cascades(case, seed)
    x = _signal(sum(n for _, n in chans), case["io"], 2 * seed)
    if case["kind"] != "train":
        y, at = torch.empty(x.numel(), device=DEV, dtype=torch.float64), 0
        for rows, n in chans:
            y[at:at + n] = _filt_exact(x[at:at + n], rows, n)
            at += n
        return y
    gy = _signal(x.numel(), case["io"], 2 * seed + 1)
    got, at = [], 0
    for rows, n in chans:
        got.append(_train_exact(x[at:at + n], gy[at:at + n], rows))
        at += n
    return {"y": torch.cat([g[0] for g in got]), "gx": torch.cat([g[1] for g in got]),
            "gsos": torch.from_numpy(np.concatenate([g[2] for g in got])).to(DEV)}
