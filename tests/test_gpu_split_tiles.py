"""The contraction's small tiles with split depth: fewer slabs than waves, depths
that do not divide by the waves, tile edges in rows and columns, filter taps,
and both sides of the grid sizes where the tile shape changes, against the
oracle (codes, format, min / max are exact)."""
import numpy as np
import pytest

from gpu_util import DEV, dev, fmt_dev, fmt_host, host, note, predicted_outcome
from test_gpu_cblock import FL_HI, FL_LO, Case, decode8

pytestmark = pytest.mark.gpu

CASES = [
    # N, Cin, H, W, K, R, stride, pad, signed input, relu
    (1, 64, 1, 1, 4, 1, 1, 0, False, False),        # one slab, one row
    (1, 128, 4, 8, 32, 1, 1, 0, True, True),        # two slabs, one full tile of 32
    (1, 192, 3, 11, 36, 1, 1, 0, False, True),      # three slabs, one row and a few columns over
    (2, 256, 5, 7, 68, 1, 1, 0, True, False),       # one slab per wave
    (1, 320, 8, 8, 64, 1, 1, 0, False, False),      # five slabs, full tiles
    (2, 64, 9, 7, 40, 3, 1, 1, False, True),        # nine taps
    (3, 128, 10, 9, 96, 3, 2, 1, True, False),      # strided, two channel chunks
    (1, 64, 128, 64, 64, 1, 1, 0, False, True),     # 512 tiles of 32 x 32
    (1, 64, 128, 65, 64, 1, 1, 0, True, False),     # 64 x 64 tiles
    (1, 192, 65, 127, 64, 1, 1, 0, False, False),   # 64 x 64, ragged rows, an idle wave
    (1, 64, 60, 60, 132, 3, 1, 1, True, True),      # 64 x 64, nine taps, ragged columns
    (1, 64, 128, 128, 64, 1, 1, 0, False, False),   # 256 tiles of 64 x 64
    (1, 64, 128, 129, 64, 1, 1, 0, False, True),    # past them
    # 128 x 64 tiles
    (1, 64, 90, 91, 136, 3, 1, 1, False, True),
    (1, 48, 127, 65, 132, 1, 1, 0, True, False),
    # channels a multiple of 16 only: chunks of one slab in several taps
    (1, 16, 3, 5, 4, 1, 1, 0, True, False),         # a quarter of a slab
    (2, 16, 9, 7, 40, 3, 1, 1, False, True),        # four taps a slab, a ragged last slab
    (1, 48, 13, 11, 36, 5, 1, 2, True, False),      # slabs across taps and filter rows
    (3, 80, 10, 9, 96, 3, 2, 1, False, False),      # strided
    (1, 112, 8, 8, 64, 1, 1, 0, True, True),        # one tap, a ragged second slab
    (1, 32, 128, 65, 64, 3, 1, 1, False, True),     # 64 x 64 tiles
    (1, 48, 60, 60, 132, 2, 1, 0, True, False),     # 64 x 64, ragged both ways
]


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


@pytest.mark.parametrize("case", CASES, ids=[str(i) for i in range(len(CASES))])
def test_split_tiles(fx, h, orc, case):
    import torch
    c = Case(*case, seed=131 + CASES.index(case)).upload(fx, h)
    v, s = c.oracle_values(orc)
    exact = (float(v.min()), float(v.max()))
    vd = dev(v).double()
    hits = 0
    for wl in (8, 4):
        note("split tiles", case, wl)
        ofl, osg, _ = orc.fl_search_i64(v, s, wl, orc.SIGN_AUTO, FL_LO, FL_HI)
        codes = orc.quantize_i64(v, s, wl, ofl, osg)
        fmt, y, mm = c.unfused(fx, h, wl)
        assert fmt == (wl, ofl, osg, 0) and tuple(mm) == exact
        assert np.array_equal(decode8(y, osg == 0), codes)
        for lo, hi in ((float("nan"), float("nan")), exact):
            mmd = torch.tensor([lo, hi], dtype=torch.float64, device=DEV)
            miss = torch.zeros(1, dtype=torch.int32, device=DEV)
            out = fmt_dev(wl, ofl, osg)
            y = c.predicted(fx, h, wl, mmd, out, miss)
            assert tuple(host(mmd)) == exact
            m = int(host(miss)[0])
            if lo != lo:
                assert m == 1
                continue
            want = predicted_outcome(vd, s, wl, osg, FL_LO, FL_HI)
            assert m == want or (want is None and m != 1)
            if m == 0:
                hits += 1
                assert fmt_host(out) == (wl, ofl, osg, 0)
                assert np.array_equal(decode8(host(y), osg == 0), codes)
    assert hits
    assert fx.sync_status(h) == 0
