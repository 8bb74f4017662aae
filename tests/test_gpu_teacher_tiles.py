"""The FP32 teacher's conv, bit for bit against the CPU oracle where its tiles
can go wrong: pixel, channel and depth remainders of both block sizes, channel
counts and pointers that do not allow 16-byte loads, several filter taps per
slab, and infinite or NaN values (a padded tap is skipped, not multiplied by
0); and narrow outputs, one per thread."""
import numpy as np
import pytest

import synth
from gpu_util import dev, empty, host, note

pytestmark = pytest.mark.gpu


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


CASES = [  # n, c, h, w, k, r, stride, pad
    (1, 1, 1, 1, 1, 1, 1, 0),
    (2, 3, 9, 7, 5, 3, 1, 1),       # four and more taps per slab, scalar loads
    (1, 4, 31, 33, 64, 7, 2, 3),    # padded RGB
    (1, 16, 8, 8, 33, 3, 1, 1),     # channels one past a small block
    (3, 20, 11, 11, 36, 5, 2, 2),
    (1, 32, 6, 6, 64, 1, 1, 0),     # depth of one small-block slab
    (5, 2048, 1, 1, 1000, 1, 1, 0),
    (33, 48, 33, 31, 132, 3, 1, 1),  # large blocks (over four per CU), remainders in every direction
    (17, 7, 65, 63, 67, 3, 1, 0),    # large blocks, scalar loads
    (2, 3, 9, 7, 45, 3, 1, 1),       # small blocks, four and more taps per slab, scalar loads
    (1, 1, 33, 9, 40, 5, 1, 2),      # a tap per value
    # narrow: shallow, few input channels, few output channels
    (3, 1, 28, 29, 31, 1, 1, 0),
    (1, 3, 300, 251, 6, 5, 1, 2),
    (5, 16, 131, 120, 4, 1, 1, 0),
    (2, 12, 7, 9, 3, 1, 2, 1),
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("special", ["none", "x", "w", "shifted"])
def test_teacher_conv_tiles(fx, h, orc, case, special):
    import torch
    n, c, hh, ww, k, r, st, pd = case
    big = n * hh * ww * k * c * r * r > 10 ** 8
    if big and special != "none":
        n = 2  # the same remainders in small blocks
    g = synth.rng_for(n * c + k, "teacher-tiles")
    x = synth.normal(1, "tx", (n, c, hh, ww))
    w = synth.normal(2, "tw", (k, c, r, r))
    if special == "x":
        x.ravel()[g.integers(0, x.size, 3)] = [np.inf, -np.inf, np.nan]
        x.ravel()[g.integers(0, x.size, 3)] = [-0.0, 1e-42, 3e38]
    elif special == "w":
        w.ravel()[g.integers(0, w.size, 2)] = [np.inf, np.nan]
        w.ravel()[w.size // 2] = -np.inf
    note("teacher tiles", case, special)
    want = orc.teacher_conv2d(x, w, st, pd)
    ho, wo = want.shape[2:]

    def up(a):
        a = np.ascontiguousarray(a).ravel()
        if special != "shifted":
            return dev(a)
        t = torch.zeros(a.size + 1, dtype=torch.float32, device="cuda:0")  # 4-byte aligned only
        t[1:] = dev(a)
        return t[1:]

    y = empty((n, ho, wo, k), torch.float32)
    xd, wd = up(x.transpose(0, 2, 3, 1)), up(w.transpose(2, 3, 1, 0))
    fx.teacher_conv(h, fx.conv_desc(n, hh, ww, c, k, r, r, st, pd), xd, wd, y)
    got = host(y).transpose(0, 3, 1, 2)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    ok = ~np.isnan(want)
    assert np.array_equal(got[ok].view(np.uint32), want[ok].view(np.uint32))
