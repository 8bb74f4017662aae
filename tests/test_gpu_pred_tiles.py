"""The predicted C-Block where a block walks several row tiles: contractions of
one to a few slabs, every operand loader, ragged rows and columns, against
separate contraction, search and requantization (format, codes, min / max).
More row tiles than the chip holds blocks, so that some blocks take two tiles
and the last one is partial."""
import numpy as np
import pytest

from gpu_util import DEV, empty, fmt_dev, fmt_host, host, note, predicted_outcome
from test_gpu_cblock import FL_HI, FL_LO, Case

pytestmark = pytest.mark.gpu

CASES = [
    # N, Cin, H, W, K, R, stride, pad, signed input, relu
    (3, 64, 84, 85, 512, 1, 1, 0, False, False),    # LDS ring, one slab
    (3, 64, 84, 85, 512, 1, 1, 0, True, True),
    (3, 128, 84, 85, 512, 1, 1, 0, False, False),   # two slabs
    (3, 192, 84, 85, 512, 1, 1, 0, True, False),    # three
    (3, 64, 84, 85, 512, 3, 1, 1, False, True),     # nine, filter taps
    (3, 64, 84, 85, 452, 1, 1, 0, False, False),    # ragged columns
    (3, 16, 84, 85, 512, 3, 1, 1, True, True),      # ring, C % 16: four taps a slab
    (3, 48, 84, 85, 452, 3, 1, 1, False, False),    # slabs across taps, ragged columns
    (3, 80, 84, 85, 512, 1, 1, 0, False, True),     # a ragged second slab
    (5, 64, 165, 163, 64, 1, 1, 0, True, True),     # 64 columns, staged slabs
    (5, 16, 165, 163, 64, 3, 1, 1, False, False),   # C % 16
    (21, 32, 57, 57, 100, 1, 1, 0, True, False),    # ring, C % 16, half a slab, ragged
    (11, 3, 223, 221, 64, 7, 2, 3, False, False),   # padded RGB, 16-byte pixels
    (11, 3, 223, 221, 32, 11, 2, 5, True, True),    # padded RGB, three chunks per filter row
    (3, 3, 50, 47, 64, 3, 1, 1, False, True),       # one chunk
    (2, 3, 33, 61, 36, 9, 1, 4, False, False),      # three chunks, ragged columns
    (1, 3, 64, 64, 24, 5, 1, 2, True, False),       # two
    (2, 3, 40, 37, 128, 11, 1, 5, True, True),      # two column tiles
    (1, 3, 22, 19, 1824, 11, 1, 5, True, True),     # filters too large to re-lay: pixel by pixel
    (5, 3, 37, 3, 64, 3, 1, 1, False, False),       # rows narrower than a chunk
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
def test_predicted_many_tiles(fx, h, case):
    import torch
    c = Case(*case, seed=91 + CASES.index(case)).upload(fx, h)
    hits = 0
    # the C-Block's values (scale 29) from the contraction's accumulators
    acc = empty((c.n // c.K, c.K), torch.int32)
    fx.qconv(h, c.desc, c.xd, c.x_type, c.wd, c.colsum, c.ep, acc)
    assert (c.fl_in + c.fl_w, c.fl_b, c.fl_a1, c.fl_a2) == (14, 11, 15, 15)
    v = (acc.long() + c.bd.long() * 8) * c.a1d.long() + c.a2d.long() * 2 ** 14
    v = (v.clamp(min=0) if c.relu else v).double()
    for wl in (8, 6, 5, 4):
        note("predicted tiles", case, wl)
        fmt, codes, exact = c.unfused(fx, h, wl)
        miss = torch.zeros(1, dtype=torch.int32, device=DEV)
        mm = torch.full((2,), float("nan"), dtype=torch.float64, device=DEV)
        c.predicted(fx, h, wl, mm, fmt_dev(wl, fmt[1], fmt[2]), miss)
        assert int(host(miss)[0]) == 1
        assert np.array_equal(host(mm), exact)
        for rep in range(2):  # the steady state, twice
            miss.zero_()
            out = fmt_dev(wl, fmt[1], fmt[2])
            y = c.predicted(fx, h, wl, mm, out, miss)
            assert np.array_equal(host(mm), exact)
            m, want = int(host(miss)[0]), predicted_outcome(v, 29, wl, fmt[2], FL_LO, FL_HI)
            assert m == want or (want is None and m != 1)
            if m == 0:
                hits += 1
                assert fmt_host(out) == fmt
                assert np.array_equal(host(y), codes)
        # the window sums decide for themselves: the other candidate is a miss
        miss.zero_()
        c.predicted(fx, h, wl, mm, fmt_dev(wl, fmt[1] + 1, fmt[2]), miss)
        assert int(host(miss)[0]) != 0
    assert hits >= 4
    assert fx.sync_status(h) == 0
