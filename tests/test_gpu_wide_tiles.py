"""The wide contraction's tiles, against the oracle's exact values: 32 x 32 ones
with split depth (fewer slabs than waves, waves that start inside a plane pair)
and 128 x 64 ones (grids above eight 32 x 32 tiles per CU), ragged rows and
columns, int64 and 128-bit sums, channel multiples of 16 and padded RGB, and both
forms of the epilogue."""
import numpy as np
import pytest

from gpu_util import host
from test_gpu_wide import draw, fx, h, orc, run_case  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, stride, pad, (wl_x, S_x), (wl_w, S_w), relu, bias, scale
CASES = [
    (1, 16, 1, 1, 4, 1, 1, 0, (9, 0), (8, 1), False, True, False),      # two slabs
    (1, 16, 3, 11, 36, 1, 1, 0, (16, 1), (9, 1), True, False, True),    # four slabs, one over in rows and columns
    (2, 48, 9, 7, 36, 3, 1, 1, (16, 1), (16, 1), True, True, False),    # slabs across taps, ragged last slab
    (1, 112, 6, 6, 64, 2, 2, 0, (24, 0), (10, 1), False, True, True),   # three input planes
    (1, 80, 130, 127, 36, 1, 1, 0, (16, 0), (10, 1), True, True, False),  # 1032 tiles
    (2, 16, 75, 61, 68, 3, 1, 1, (12, 1), (12, 1), False, False, True),
    (1, 3, 9, 11, 20, 3, 1, 1, (16, 0), (10, 1), False, True, False),   # padded RGB
    (2, 3, 150, 151, 64, 7, 2, 3, (16, 1), (10, 1), True, False, True),  # 714
    (1, 3, 33, 35, 20, 5, 1, 2, (24, 1), (24, 1), True, True, False),   # 128-bit sums
    (1, 32, 64, 65, 40, 1, 1, 0, (24, 0), (24, 1), False, True, False),
]


@pytest.mark.parametrize("case", CASES, ids=[str(i) for i in range(len(CASES))])
def test_wide_tiles(fx, h, orc, case):  # noqa: F811
    v, sc, want, s_out, _ = run_case(fx, h, orc, case, seed=210 + CASES.index(case))
    assert int(host(sc)[0]) == s_out
    assert np.array_equal(host(v), want)
    assert fx.sync_status(h) == 0


# more 32 x 32 tiles than eight per CU of the largest chip: 128 x 64 tiles
LARGE = [
    (1, 16, 182, 181, 36, 1, 1, 0, (16, 0), (10, 1), True, True, False),    # a quarter of a slab per pair
    (2, 48, 105, 107, 68, 3, 1, 1, (16, 1), (16, 1), True, True, False),    # slabs across taps, two column tiles
    (1, 80, 115, 117, 132, 3, 1, 1, (12, 1), (12, 1), False, False, True),  # a slab over, three column tiles
    (3, 16, 187, 201, 100, 3, 2, 0, (24, 0), (10, 1), True, True, True),    # three input planes, strided
    # padded RGB in chunks of four taps
    (1, 3, 183, 181, 36, 3, 1, 1, (16, 0), (10, 1), False, True, False),    # one chunk per filter row
    (2, 3, 211, 215, 68, 7, 2, 3, (16, 1), (16, 1), True, False, True),     # two
    (1, 3, 233, 235, 132, 7, 2, 0, (12, 0), (9, 1), False, True, False),
    (1, 3, 190, 187, 36, (2, 11), 1, 2, (16, 1), (10, 1), False, True, True),  # three
    (20, 3, 400, 5, 36, 3, 1, 1, (16, 1), (12, 1), True, True, False),      # rows of one pixel more than a chunk
    (1, 3, 183, 181, 36, 5, 1, 2, (16, 0), (10, 1), False, True, False),    # rows that do not fit: 32 x 32 tiles
]

# 128-bit sums of few slabs in more 32 x 32 tiles than 24 per CU: 64 x 64 tiles
LARGE128 = [
    (1, 16, 317, 311, 36, 1, 1, 0, (24, 0), (16, 1), True, True, False),   # a quarter of a slab per pair
    (1, 48, 230, 231, 100, 1, 1, 0, (24, 1), (16, 1), False, False, True),  # two column tiles
    (3, 16, 130, 263, 52, 2, 1, 1, (32, 1), (24, 1), False, True, False),  # four taps, sixteen pairs
    (1, 3, 317, 313, 36, 3, 1, 1, (24, 1), (16, 1), True, True, False),    # padded RGB
    (2, 3, 226, 227, 36, (1, 9), 1, 0, (32, 1), (15, 0), False, True, False),  # three chunks per filter row
    (1, 16, 260, 259, 68, 1, 1, 0, (24, 0), (16, 1), True, True, False),   # an odd number of column tiles: 32 x 32
]


def many_tiles(case, per_cu=8):
    import torch
    N, _, H, W, K, R, stride, pad = case[:8]
    R, S = R if isinstance(R, tuple) else (R, R)
    M = N * ((H + 2 * pad - R) // stride + 1) * ((W + 2 * pad - S) // stride + 1)
    assert M % 128 and K % 64
    return -(-M // 32) * -(-K // 32) > per_cu * torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("case", LARGE, ids=[str(i) for i in range(len(LARGE))])
def test_wide_large_tiles(fx, h, orc, case):  # noqa: F811
    assert many_tiles(case)
    v, sc, want, s_out, _ = run_case(fx, h, orc, case, seed=240 + LARGE.index(case))
    assert int(host(sc)[0]) == s_out
    assert np.array_equal(host(v), want)
    assert fx.sync_status(h) == 0


@pytest.mark.parametrize("case", LARGE128, ids=[str(i) for i in range(len(LARGE128))])
def test_wide_large_tiles_128_bits(fx, h, orc, case):  # noqa: F811
    assert many_tiles(case, 24)
    v, sc, want, s_out, _ = run_case(fx, h, orc, case, seed=250 + LARGE128.index(case))
    assert int(host(sc)[0]) == s_out
    assert np.array_equal(host(v), want)
    assert fx.sync_status(h) == 0


@pytest.mark.parametrize("case", [
    (1, 16, 182, 181, 36, 1, 1, 0, (16, 0), (10, 1), False, False, True),
    (1, 3, 183, 181, 36, 3, 1, 1, (16, 1), (10, 1), False, False, True),
    (1, 16, 9, 7, 36, 1, 1, 0, (16, 1), (10, 1), False, False, True),  # 32 x 32 tiles
], ids=["ring", "rgb", "small"])
def test_wide_epilogue_bounds(fx, h, orc, case):  # noqa: F811
    """Values of 62 bits: beyond the bound that leaves out the steps' own checks
    (2^61), and one bit more: values beyond 62 bits are 0 and raise the flag."""
    assert many_tiles(case) or case[2] == 9
    seed, K, R = 260, case[4], case[5]
    acc = orc.conv2d(draw(seed, "wx", (case[0], case[1], case[2], case[3]), *case[8]),
                     draw(seed, "ww", (K, case[1], R, R), *case[9]), case[6], case[7])
    top = {}

    def exact(acc, s, bias, fl_b, a1, fl_a1, a2, fl_a2, relu):
        v = (acc * a1.astype(np.int64).reshape(1, -1, 1, 1)) * 2 ** (fl_a2 - s - fl_a1)
        v = v + a2.astype(np.int64).reshape(1, -1, 1, 1)
        top["max"] = np.abs(v).max()
        return np.where(np.abs(v) < 2 ** 62, v, 0), fl_a2

    # |acc a1| < 2^15 max |acc|, its scale 36: the power of two that takes the largest value to 62 bits
    room = 61 - int(np.abs(acc).max()).bit_length() - 15
    for fl in range(36 + room, 36 + room + 17):
        v, sc, want, s_out, _ = run_case(fx, h, orc, case, seed, fl_a2=fl, epilogue=exact)
        assert int(host(sc)[0]) == s_out == fl
        assert np.array_equal(host(v), want)
        flags = fx.sync_status(h)
        if top["max"] >= 2 ** 62:
            assert flags != 0
            return
        assert flags == 0
    assert False, "no value beyond 62 bits"
