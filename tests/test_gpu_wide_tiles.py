"""The wide contraction's tiles: fewer slabs than waves, waves that start inside
a plane pair, 32 x 32 and 64 x 64 tiles with ragged rows and columns, int64 and
128-bit sums, channel multiples of 16 and padded RGB, against the oracle's exact
values."""
import numpy as np
import pytest

from gpu_util import host
from test_gpu_wide import fx, h, orc, run_case  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, stride, pad, (wl_x, S_x), (wl_w, S_w), relu, bias, scale
CASES = [
    (1, 16, 1, 1, 4, 1, 1, 0, (9, 0), (8, 1), False, True, False),      # two slabs
    (1, 16, 3, 11, 36, 1, 1, 0, (16, 1), (9, 1), True, False, True),    # four slabs, one over in rows and columns
    (2, 48, 9, 7, 36, 3, 1, 1, (16, 1), (16, 1), True, True, False),    # slabs across taps, ragged last slab
    (1, 112, 6, 6, 64, 2, 2, 0, (24, 0), (10, 1), False, True, True),   # three input planes
    (1, 80, 130, 127, 36, 1, 1, 0, (16, 0), (10, 1), True, True, False),  # 64 x 64 tiles
    (2, 16, 75, 61, 68, 3, 1, 1, (12, 1), (12, 1), False, False, True),
    (1, 3, 9, 11, 20, 3, 1, 1, (16, 0), (10, 1), False, True, False),   # padded RGB
    (2, 3, 150, 151, 64, 7, 2, 3, (16, 1), (10, 1), True, False, True),  # 64 x 64 tiles
    (1, 3, 33, 35, 20, 5, 1, 2, (24, 1), (24, 1), True, True, False),   # 128-bit sums
    (1, 32, 64, 65, 40, 1, 1, 0, (24, 0), (24, 1), False, True, False),
]


@pytest.mark.parametrize("case", CASES, ids=[str(i) for i in range(len(CASES))])
def test_wide_tiles(fx, h, orc, case):  # noqa: F811
    v, sc, want, s_out, _ = run_case(fx, h, orc, case, seed=210 + CASES.index(case))
    assert int(host(sc)[0]) == s_out
    assert np.array_equal(host(v), want)
    assert fx.sync_status(h) == 0
