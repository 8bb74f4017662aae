"""Small tensors: the search in one launch of one block (up to 8192 values, 4096
with a given min / max) and reductions finished by their last block (up to 64
blocks), on both sides of those sizes, against the oracle / numpy; and replayed
from a captured graph, where every launch has to leave the counters at zero."""
import numpy as np
import pytest

import synth
from gpu_util import DEV, dev, empty, fmt_dev, fmt_host, fmt_new, host, note

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


def values(seed, n, heavy):
    g = synth.rng_for(seed, "small")
    v = g.standard_normal(n) * (0.02 if heavy else 1.5)
    if heavy:
        v[g.integers(0, n, max(1, n // 300))] = 5.0 * (1 + g.random())
    return v.astype(np.float32)


@pytest.mark.parametrize("n", [1, 3, 255, 1024, 1027, 4096, 4097, 8191, 8192, 8193])
def test_search(fx, h, orc, n):
    import torch
    s = 12
    sd = torch.tensor([s], dtype=torch.int32, device=DEV)
    for heavy in (False, True):
        x = values(n, n, heavy)
        iv = np.rint(x.astype(np.float64) * 2.0 ** s).astype(np.int64)
        mm = torch.tensor([float(iv.min()), float(iv.max())], dtype=torch.float64, device=DEV)
        xd, v32, v64 = dev(x), dev(iv.astype(np.int32)), dev(iv)
        for wl in (1, 2, 4, 8, 16, 17):
            note("small search", n, heavy, wl)
            f32 = orc.fl_search_f32(x, wl, fx.SIGN_AUTO, FL_LO, FL_HI)[:2]
            i64 = orc.fl_search_i64(iv, s, wl, fx.SIGN_AUTO, FL_LO, FL_HI)[:2]
            for src, want in ((fx.src_f32(xd), f32), (fx.src_int(v32, fx.I32, sd), i64),
                              (fx.src_int(v64, fx.I64, sd), i64), (fx.src_int(v32, fx.I32, sd, mm), i64)):
                out = fmt_new()
                fx.fl_search(h, src, n, wl, fx.SIGN_AUTO, FL_LO, FL_HI, out)
                assert fmt_host(out) == (wl, *want, 0), wl
    assert fx.sync_status(h) == 0


def test_search_large_and_nonfinite(fx, h, orc):
    x = values(5, 700, False) * np.float32(9000.0)  # beyond the window: the 128-bit pass
    for wl in (3, 8):
        note("small search large", wl)
        out = fmt_new()
        fx.fl_search(h, fx.src_f32(dev(x)), x.size, wl, fx.SIGN_AUTO, FL_LO, FL_HI, out)
        assert fmt_host(out)[:3] == (wl, *orc.fl_search_f32(x, wl, fx.SIGN_AUTO, FL_LO, FL_HI)[:2])
    assert fx.sync_status(h) == 0
    x[13] = np.nan
    out = fmt_new()
    fx.fl_search(h, fx.src_f32(dev(x)), x.size, 8, fx.SIGN_AUTO, FL_LO, FL_HI, out)
    assert fmt_host(out)[3] != 0 and fx.sync_status(h) != 0


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 65535, 65536, 65537, 70001])
def test_layer_error(fx, h, n):
    import torch
    g = synth.rng_for(n, "err")
    c = g.integers(-128, 128, n).astype(np.int8)
    r = (c / 32.0 + g.standard_normal(n) * 0.01).astype(np.float32)
    out = empty((4,), torch.float64)
    note("small layer error", n)
    fx.layer_error(h, dev(r), dev(c), fx.I8, fmt_dev(8, 5, 1), n, out)
    d = r.astype(np.float64) - c / 32.0
    got = host(out)
    # fp64 sums of n terms in another order: n 2^-53 relative to sums of magnitudes
    assert abs(got[0] - (d * d).sum()) <= n * 2.0 ** -53 * (d * d).sum()
    assert got[1] == r.min() and got[2] == r.max()
    m2 = (r.astype(np.float64) ** 2).mean()
    assert abs(got[3] ** 2 - r.astype(np.float64).var()) <= 4 * n * 2.0 ** -53 * m2 + 2.0 ** -50 * m2


def test_replayed_from_a_graph(fx, orc):
    import torch
    n, s = 6000, 12
    g = torch.cuda.CUDAGraph()
    hd = fx.Handle(0)
    st = torch.cuda.Stream()
    x = torch.zeros(n, device=DEV)
    c = torch.zeros(n, dtype=torch.int8, device=DEV)
    out, err = fmt_new(), empty((4,), torch.float64)
    fx.set_stream(hd, st)

    def calls():
        fx.fl_search(hd, fx.src_f32(x), n, 6, fx.SIGN_AUTO, FL_LO, FL_HI, out)
        fx.layer_error(hd, x, c, fx.I8, out, n, err)

    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        calls()
    st.synchronize()
    with torch.cuda.graph(g, stream=st):
        calls()
    for rep in range(4):
        note("small calls replay", rep)
        v = values(300 + rep, n, rep % 2 == 1) * np.float32(2.0 ** rep)
        x.copy_(torch.from_numpy(v))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert fmt_host(out) == (6, *orc.fl_search_f32(v, 6, fx.SIGN_AUTO, FL_LO, FL_HI)[:2], 0)
        e = (v.astype(np.float64) ** 2).sum()  # every code is zero
        assert abs(host(err)[0] - e) <= n * 2.0 ** -53 * e
        with torch.cuda.stream(st):
            calls()  # eager work between the replays
        st.synchronize()
    assert fx.sync_status(hd) == 0
    hd.close()
