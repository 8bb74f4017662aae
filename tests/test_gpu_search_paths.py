"""The FL search's paths beyond its one-read window, against the CPU oracle:
int64 values (split sums in the window) and the exact pass over the candidates
above the window (fp64 sums of four candidates per read), at tensor sizes
around a packet, a block and a flush, and for C-Block values whose channel
count does / does not fit the pass's grid stride."""
import numpy as np
import pytest

import synth
from gpu_util import DEV, dev, fmt_dev, fmt_host, fmt_new, note

pytestmark = pytest.mark.gpu

FL_LO, FL_HI = -8, 15


@pytest.fixture(scope="module")
def fx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_12091_amd import fxpq
    return fxpq


@pytest.fixture(scope="module")
def h(fx):
    import torch
    hd = fx.Handle(0)
    fx.set_stream(hd, torch.cuda.current_stream())
    yield hd
    hd.close()


def values(seed, n, bits, heavy):
    """Normal integers of about `bits` bits; heavy: a few outliers far above, so that short word lengths clip them."""
    g = synth.rng_for(seed, "paths")
    v = (g.standard_normal(n) * 2.0 ** (bits - (6 if heavy else 2))).astype(np.int64)
    if heavy:
        idx = g.choice(n, max(1, n // 5000), replace=False)
        v[idx] = (2.0 ** (bits - 1) * (1 + g.random(idx.size))).astype(np.int64)
    return np.clip(v, -(2 ** bits) + 1, 2 ** bits - 1)


@pytest.mark.parametrize("n", [1, 2, 3, 513, 131_075, 700_001])
@pytest.mark.parametrize("bits,s", [(44, 30), (51, 41), (46, 20)])
def test_int64_search(fx, h, orc, n, bits, s):
    import torch
    sd = torch.tensor([s], dtype=torch.int32, device=DEV)
    for heavy in (False, True):
        v = values(n + bits, n, bits, heavy)
        vd = dev(v)
        for wl in (2, 4, 8, 12, 16):
            note("int64", n, bits, s, heavy, wl)
            out = fmt_new()
            fx.fl_search(h, fx.src_int(vd, fx.I64, sd), n, wl, fx.SIGN_AUTO, FL_LO, FL_HI, out)
            ofl, osign, _ = orc.fl_search_i64(v, s, wl, fx.SIGN_AUTO, FL_LO, FL_HI)
            assert fmt_host(out) == (wl, ofl, osign, 0), (heavy, wl)
    assert fx.sync_status(h) == 0


@pytest.mark.parametrize("channels", [1, 7, 100, 1000, 1028])  # 1028: no grid of the pass keeps its channels
def test_cblock_values_above_the_window(fx, h, orc, channels):
    import torch
    g = synth.rng_for(channels, "paths-acc")
    rows = 300_007 // channels
    acc = values(channels, rows * channels, 24, True).astype(np.int32).reshape(rows, channels)
    a1 = g.integers(2 ** 14, 2 ** 15, channels).astype(np.int32)
    ep = fx.epilogue(channels, 9, fmt_dev(8, 5, 1), scale=dev(a1), fl_scale=15)
    v, s = orc.epilogue(acc.astype(np.int64), 14, a1=a1, fl_a1=15)
    above = 0
    for wl in (3, 5, 8, 16):
        note("acc", channels, wl)
        out = fmt_new()
        fx.fl_search(h, fx.src_acc(dev(acc), ep), acc.size, wl, fx.SIGN_AUTO, FL_LO, FL_HI, out)
        ofl, osign, _ = orc.fl_search_i64(np.ravel(v), s, wl, fx.SIGN_AUTO, FL_LO, FL_HI)
        assert fmt_host(out) == (wl, ofl, osign, 0), wl
        qmax = 2 ** (wl - osign) - 1
        above += float(np.max(v)) * 2.0 ** (ofl - 1 - s) > qmax + 0.5  # best fl more than one above no saturation
    assert above  # the fixture reaches the exact pass
    assert fx.sync_status(h) == 0


@pytest.mark.parametrize("wl", [2, 5, 8, 16])
@pytest.mark.parametrize("shift", [0, 3, 9])
def test_search_at_the_saturation_bound(fx, h, orc, wl, shift):
    """The largest fl without saturation comes from the exponents of the min /
    max: extremes exactly at the bounds qmax + 1/2 and qmin - 1/2 of an fl, and
    one unit inside and outside, on either side."""
    import torch
    g = synth.rng_for(wl * 16 + shift, "bound")
    s = 14
    sd = torch.tensor([s], dtype=torch.int32, device=DEV)
    for sign in (0, 1):
        top = (2 ** (wl - sign) * 2 - 1) << shift        # 2 (qmax + 1/2)
        bot = ((2 ** wl + 1) if sign else 1) << shift    # 2 (1/2 - qmin)
        for du in (-1, 0, 1):
            for mx, mn in ((top + du, 0), (top + du, -(bot // 2)), (top // 2, -(bot + du)),
                           (0, -(bot + du))):
                if sign == 0 and mn < 0 or mx == 0 and mn == 0:
                    continue
                v = g.integers(mn // 2, mx // 2 + 1, 300).astype(np.int64)
                v[7], v[200] = mx, mn
                vd = dev(v.astype(np.int32))
                note("bound", wl, shift, sign, mx, mn)
                out = fmt_new()
                fx.fl_search(h, fx.src_int(vd, fx.I32, sd), v.size, wl, fx.SIGN_AUTO, FL_LO, FL_HI, out)
                ofl, osign, _ = orc.fl_search_i64(v, s, wl, fx.SIGN_AUTO, FL_LO, FL_HI)
                assert fmt_host(out) == (wl, ofl, osign, 0), (mx, mn)
    assert fx.sync_status(h) == 0


@pytest.mark.parametrize("n", [1, 5, 1030, 262_147])
@pytest.mark.parametrize("wl", [8, 17, 19, 24, 25, 26])
def test_int64_search_wide_values(fx, h, orc, n, wl):
    """Values of 53 to 61 bits (three-part sums of the exact pass, codes from the
    value rounded to odd) and word lengths past the window's: ties of a code's
    last bit with bits set far below, extremes, and smaller values."""
    import torch
    g = synth.rng_for(n + wl, "wide")
    s = 40
    sd = torch.tensor([s], dtype=torch.int32, device=DEV)
    for bits in (50, 54, 61):
        v = (g.standard_normal(n) * 2.0 ** (bits - 3)).astype(np.int64)
        v = np.clip(v, -(2 ** bits) + 1, 2 ** bits - 1)
        # halves of the candidates' steps, exactly and one unit off
        k = g.integers(0, 2 ** 12, n)
        half = (2 * k + 1) << g.integers(20, 40, n)
        pick = g.integers(0, 4, n)
        v = np.where(pick == 0, half, np.where(pick == 1, -half - 1, np.where(pick == 2, half - 1, v)))
        v[0] = 2 ** bits - 1
        out = fmt_new()
        note("int64 wide", n, wl, bits)
        fx.fl_search(h, fx.src_int(dev(v), fx.I64, sd), n, wl, fx.SIGN_AUTO, FL_LO, FL_HI, out)
        ofl, osign, _ = orc.fl_search_i64(v, s, wl, fx.SIGN_AUTO, FL_LO, FL_HI)
        assert fmt_host(out) == (wl, ofl, osign, 0), bits
    assert fx.sync_status(h) == 0


@pytest.mark.parametrize("n", [1, 9001])
@pytest.mark.parametrize("wl", [2, 4, 8, 16])
def test_int64_extreme_rounded_to_the_bound(fx, h, orc, n, wl):
    """A largest value one unit above (qmax + 1/2) 2^k, which fp64 rounds onto
    that bound: it saturates there, and one fl lower its error is smaller."""
    import torch
    for sign in (0, 1):
        for k in range(53 - wl + sign, 60 - wl + sign):
            s = k + 4  # the bound at fl 3
            sd = torch.tensor([s], dtype=torch.int32, device=DEV)
            for du in (-1, 0, 1):
                v = np.zeros(n, np.int64)
                v[n // 2] = ((2 ** (wl - sign) * 2 - 1) << k) + du
                out = fmt_new()
                note("int64 bound", n, wl, sign, k, du)
                fx.fl_search(h, fx.src_int(dev(v), fx.I64, sd), n, wl, sign, FL_LO, FL_HI, out)
                ofl, osign, _ = orc.fl_search_i64(v, s, wl, sign, FL_LO, FL_HI)
                assert fmt_host(out) == (wl, ofl, osign, 0), (sign, k, du)
    assert fx.sync_status(h) == 0
