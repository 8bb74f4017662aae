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


def search(fx, h, src, n, wl, lo, hi, sse=None, sign=None):
    out = fmt_new()
    fx.fl_search(h, src, n, wl, fx.SIGN_AUTO if sign is None else sign, lo, hi, out, sse)
    return fmt_host(out)


@pytest.mark.parametrize("n", [1, 5, 256, 4096, 8192, 8193, 300_001])
@pytest.mark.parametrize("wl", [2, 4, 8, 13, 16, 24])
def test_f32_search_large_values(fx, h, orc, n, wl):
    """fp32 values of 2^12 and more units of the largest fl (W = v 2^(fl_hi + 24)
    from 2^52 on): three-part sums of the exact pass, in one block and in many,
    with small and fractional W beside them; saturated at the lowest fl, ties
    of the candidates' codes."""
    import torch
    g = synth.rng_for(n + wl, "f32-large")
    for lo, hi, e in ((-8, 15, 14), (-8, 15, 22), (-20, 16, 20), (-64, 3, 30)):
        v = g.standard_normal(n) * 2.0 ** (e - 3)
        pick = g.integers(0, 4, n)
        v = np.where(pick == 0, v * 2.0 ** -g.integers(0, 60, n), v)
        v = np.where(pick == 1, (2 * g.integers(-2 ** 7, 2 ** 7, n) + 1) * 2.0 ** g.integers(-hi, 9, n), v)
        v[n // 2] = 2.0 ** e * 1.37
        v = v.astype(np.float32)
        assert 2 ** 52 <= np.abs(v).max() * 2.0 ** (hi + 24) < 2 ** 62
        note("f32 large", n, wl, lo, hi, e)
        vd = dev(v)
        ofl, osign, _ = orc.fl_search_f32(v, wl, fx.SIGN_AUTO, lo, hi)
        assert search(fx, h, fx.src_f32(vd), n, wl, lo, hi) == (wl, ofl, osign, 0)
        mm = torch.tensor([float(v.min()), float(v.max())], dtype=torch.float64, device=DEV)
        assert search(fx, h, fx.src_f32(vd, mm), n, wl, lo, hi) == (wl, ofl, osign, 0)
        if wl > 8:
            continue
        codes, y, alt = (torch.empty(n + 16, dtype=torch.int8, device=DEV) for _ in range(3))
        fx.quantize(h, vd, n, fmt_dev(wl, ofl, osign), codes, fx.C8)
        out = fmt_new()
        fx.qlayer(h, fx.src_f32(vd), n, wl, fx.SIGN_AUTO, lo, hi, out, y, fx.C8, alt)
        assert fmt_host(out) == (wl, ofl, osign, 0) and torch.equal(y[:n], codes[:n])
        miss = torch.zeros(1, dtype=torch.int32, device=DEV)
        y.fill_(99)
        fx.qlayer_predicted(h, fx.src_f32(vd), n, wl, fx.SIGN_AUTO, lo, hi, out, y, fx.C8, mm, miss)
        if int(miss) == 0:
            assert fmt_host(out) == (wl, ofl, osign, 0) and torch.equal(y[:n], codes[:n])
        else:
            assert int(miss) == 2  # the window alone does not decide
    assert fx.sync_status(h) == 0


@pytest.mark.parametrize("n", [64, 4096, 20_000])
@pytest.mark.parametrize("wl", [4, 8, 16, 20])
def test_integer_search_of_53_bits(fx, h, orc, n, wl):
    """C-Block values and residual sums of 2^52 <= |W| < 2^53."""
    g = synth.rng_for(n + wl, "53")
    ch = 32
    acc = np.clip(g.standard_normal(n) * 2.0 ** 27, -2 ** 30 + 1, 2 ** 30 - 1).astype(np.int32).reshape(-1, ch)
    acc[1, 3] = 2 ** 30 - 5
    a1 = g.integers(2 ** 22, 2 ** 23, ch).astype(np.int32)
    ep = fx.epilogue(ch, 24, fmt_dev(8, 20, 1), scale=dev(a1), fl_scale=10)
    v, s = orc.epilogue(acc.astype(np.int64), 44, a1=a1, fl_a1=10)
    assert 2 ** 52 <= np.abs(v).max() < 2 ** 53
    note("53 bits", n, wl)
    for lo, hi in ((FL_LO, FL_HI), (-30, 40)):
        ofl, osign, _ = orc.fl_search_i64(np.ravel(v), s, wl, fx.SIGN_AUTO, lo, hi)
        assert search(fx, h, fx.src_acc(dev(acc), ep), n, wl, lo, hi) == (wl, ofl, osign, 0)
    a, b = g.integers(0, 256, n), g.integers(-128, 128, n)
    a[n // 2] = 255
    src = fx.src_add(dev((a - 128).astype(np.int8)), fx.C8, fmt_dev(8, 0, 0), dev(b.astype(np.int8)), fx.C8,
                     fmt_dev(8, 45, 1), False)
    w = (a.astype(np.int64) << 45) + b
    for lo, hi in ((FL_LO, FL_HI), (-20, 44)):
        ofl, osign, _ = orc.fl_search_i64(w, 45, wl, fx.SIGN_AUTO, lo, hi)
        assert search(fx, h, src, n, wl, lo, hi) == (wl, ofl, osign, 0)
    assert fx.sync_status(h) == 0


@pytest.mark.parametrize("n", [1, 16, 1023, 1025, 24_576, 24_577])
@pytest.mark.parametrize("wl", [17, 20, 23, 24, 25])
def test_exact_pass_of_few_blocks(fx, h, orc, n, wl):
    """Word lengths past the window's, up to the values of 24 blocks (the exact
    pass takes that few) and one more: every source."""
    import torch
    g = synth.rng_for(n + wl, "few-blocks")
    v = values(n * wl, n, 24, True)
    sd = torch.tensor([9], dtype=torch.int32, device=DEV)
    note("few blocks", n, wl)
    want = (wl, *orc.fl_search_i64(v, 9, wl, fx.SIGN_AUTO, FL_LO, FL_HI)[:2], 0)
    assert search(fx, h, fx.src_int(dev(v.astype(np.int32)), fx.I32, sd), n, wl, FL_LO, FL_HI) == want
    assert search(fx, h, fx.src_int(dev(v), fx.I64, sd), n, wl, FL_LO, FL_HI) == want
    x = v.astype(np.float32)
    fl, sg, _ = orc.fl_search_f32(x * np.float32(2.0 ** -9), wl, fx.SIGN_AUTO, FL_LO, FL_HI)
    assert search(fx, h, fx.src_f32(dev(x * np.float32(2.0 ** -9))), n, wl, FL_LO, FL_HI) == (wl, fl, sg, 0)
    for ch in (1, 12, 1000):
        rows = max(1, n // ch)
        acc = g.integers(-2 ** 22, 2 ** 22, (rows, ch)).astype(np.int32)
        a1 = g.integers(2 ** 14, 2 ** 15, ch).astype(np.int32)
        ep = fx.epilogue(ch, 9, fmt_dev(8, 5, 1), scale=dev(a1), fl_scale=15)
        w, s = orc.epilogue(acc.astype(np.int64), 14, a1=a1, fl_a1=15)
        fl, sg, _ = orc.fl_search_i64(np.ravel(w), s, wl, fx.SIGN_AUTO, FL_LO, FL_HI)
        assert search(fx, h, fx.src_acc(dev(acc), ep), acc.size, wl, FL_LO, FL_HI) == (wl, fl, sg, 0)
    a, b = g.integers(0, 256, n), g.integers(-128, 128, n)
    src = fx.src_add(dev((a - 128).astype(np.int8)), fx.C8, fmt_dev(8, 5, 0), dev(b.astype(np.int8)), fx.C8,
                     fmt_dev(8, 9, 1), True)
    w = np.maximum((a.astype(np.int64) << 4) + b, 0)
    fl, sg, _ = orc.fl_search_i64(w, 9, wl, fx.SIGN_AUTO, FL_LO, FL_HI)
    assert search(fx, h, src, n, wl, FL_LO, FL_HI) == (wl, fl, sg, 0)
    assert fx.sync_status(h) == 0


@pytest.mark.parametrize("channels", [70, 1080])
def test_every_error_of_cblock_values(fx, h, orc, channels):
    """All candidates' errors (128-bit items, any number of blocks) where the
    sums would take a grid of the channels' multiple."""
    import torch
    rows = 140_001 // channels
    acc = values(channels, rows * channels, 24, True).astype(np.int32).reshape(rows, channels)
    ep = fx.epilogue(channels, 9, fmt_dev(8, 5, 1))
    for wl in (1, 6, 8, 26):
        note("every error", channels, wl)
        ofl, osign, osse = orc.fl_search_i64(np.ravel(acc).astype(np.int64), 14, wl, fx.SIGN_AUTO, FL_LO, FL_HI)
        sse = torch.zeros(FL_HI - FL_LO + 1, dtype=torch.float64, device=DEV)
        assert search(fx, h, fx.src_acc(dev(acc), ep), acc.size, wl, FL_LO, FL_HI, sse) == (wl, ofl, osign, 0)
        assert np.allclose(sse.cpu().numpy(), osse, rtol=1e-9, atol=0)
    assert fx.sync_status(h) == 0


@pytest.mark.parametrize("n", [1, 15, 300, 2049, 4096, 8192, 9000])
def test_integer_search_beyond_the_exact_pass(fx, h, orc, n):
    """Values that the window decides although the exact pass would refuse them
    (|v| 2^(fl_hi - scale) of 2^62 and more): whatever number of values a thread
    adds, the same are taken.  The best fl lies in the range's lower part, so the
    oracle's search up to fl 29 finds it."""
    import torch
    g = synth.rng_for(n, "beyond")
    for wl, bits in ((8, 41), (8, 42), (16, 33), (16, 34)):  # |W| max |q| 8 below 2^53
        s = 9
        v = np.clip(g.standard_normal(n) * 2.0 ** (bits - 3), -2 ** bits * 0.95, 2 ** bits * 0.95).astype(np.int64)
        v[n // 2] = int(2 ** bits * 0.96)
        v[n // 3] = -int(2 ** bits * 0.95)
        note("beyond", n, wl, bits)
        fl, sg, _ = orc.fl_search_i64(v, s, wl, 1, -64, 24 if bits > 40 else 32)
        sd = torch.tensor([s], dtype=torch.int32, device=DEV)
        assert search(fx, h, fx.src_int(dev(v), fx.I64, sd), n, wl, -64, 50, sign=1) == (wl, fl, sg, 0)
        # C-Block values acc * a1 of the same size
        a1 = np.array([2 ** 22 - 3], np.int32)
        acc = (v >> 22).astype(np.int32)
        ep = fx.epilogue(1, 3, fmt_dev(8, 2, 1), scale=dev(a1), fl_scale=4)
        w = acc.astype(np.int64) * int(a1[0])
        fl, sg, _ = orc.fl_search_i64(w, s, wl, 1, -64, 24 if bits > 40 else 32)
        assert search(fx, h, fx.src_acc(dev(acc.reshape(-1, 1)), ep), n, wl, -64, 50, sign=1) == (wl, fl, sg, 0)
    a, b = g.integers(0, 256, n), g.integers(-128, 128, n)
    a[n // 2] = 255
    src = fx.src_add(dev((a - 128).astype(np.int8)), fx.C8, fmt_dev(8, 0, 0), dev(b.astype(np.int8)), fx.C8,
                     fmt_dev(8, 33, 1), False)
    fl, sg, _ = orc.fl_search_i64((a.astype(np.int64) << 33) + b, 33, 8, 1, -20, 50)
    assert search(fx, h, src, n, 8, -20, 64, sign=1) == (8, fl, sg, 0)
    assert fx.sync_status(h) == 0
