"""Helpers for the GPU parity tests (imported by test modules, not collected)."""
import sys

import numpy as np

DEV = "cuda:0"


def note(*a):
    """Names the case about to run on the GPU (flushed, so a fault still shows it)."""
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


def torch():
    import torch as T
    return T


def dev(a):
    T = torch()
    return T.from_numpy(np.ascontiguousarray(a)).to(DEV)


def host(t):
    T = torch()
    T.cuda.synchronize()
    return t.cpu().numpy()


def empty(shape, dtype):
    T = torch()
    return T.empty(shape, dtype=dtype, device=DEV)


def fmt_dev(wl, fl, sign):
    T = torch()
    return T.tensor([wl, fl, sign, 0], dtype=T.int32, device=DEV)


def fmt_new():
    T = torch()
    return T.full((4,), -999, dtype=T.int32, device=DEV)


def fmt_host(t):
    wl, fl, sign, status = (int(v) for v in host(t))
    return wl, fl, sign, status


def decode8(codes, off):
    c = np.asarray(codes).astype(np.int64)
    return c + 128 if off else c


def predicted_outcome(v, s, wl, sign, fl_lo, fl_hi):
    """What a predicted call with the exact min / max and the right format
    reports: 0 (a hit), 2 (the window and its one clipping bound cannot decide)
    or None (fp64 does not tell).  v: the values (float64 tensor of integers
    below 2^53) at scale s."""
    qmax, qmin = 2.0 ** (wl - sign) - 1, -(2.0 ** (wl - 1)) if sign else 0.0
    mx, mn = float(v.max()), float(v.min())
    b0 = max(b for b in range(fl_lo - 1, fl_hi + 1)
             if b < fl_lo or (mx * 2.0 ** (b - s) <= qmax + 0.5 and mn * 2.0 ** (b - s) >= qmin - 0.5))
    b0 = max(b0, fl_lo)
    assert b0 < fl_hi
    b1 = b0 + 1
    if b1 == fl_hi:
        return 0
    err = min(float((((v * 2.0 ** (b - s)).round().clamp(qmin, qmax) * 2.0 ** (s - b) - v) ** 2).sum())
              for b in (b0, b1))
    t = v * 2.0 ** (b1 + 1 - s)
    clip = float(((t - t.clamp(qmin, qmax)) ** 2).sum()) * 4.0 ** (s - b1 - 1)
    return None if abs(clip - err) < 1e-6 * err else (0 if clip > err else 2)
