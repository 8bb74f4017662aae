"""Tensors beyond 32-bit indices, against the same calls on cut-outs."""
import pytest

from gpu_util import DEV, note

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_12091_amd import fxpq
    return fxpq


@pytest.fixture
def h(fx):
    import torch
    hd = fx.Handle(0)
    fx.set_stream(hd, torch.cuda.current_stream())
    yield hd
    hd.close()
    torch.cuda.empty_cache()


def rgb_filters(g, K, R, lo, hi, dtype):
    """[K][R * R * 4 padded to 64] filters, the padded channel and tail zero."""
    import torch
    kd = R * R * 4
    w = torch.zeros((K, (kd + 63) // 64 * 64), dtype=dtype, device=DEV)
    f = torch.randint(lo, hi, (K, R * R, 4), generator=g, device=DEV).to(dtype)
    f[..., 3] = 0
    w[:, :kd] = f.reshape(K, kd)
    return w


def test_first_layer_over_2_32_pixels(fx, h):
    """A padded RGB image of 66000 x 65540 pixels: the rows past pixel 2^32."""
    import torch
    H, W, K, R, st = 66000, 65540, 8, 3, 257
    g = torch.Generator(device=DEV).manual_seed(3)
    note("rgb image of more than 2^32 pixels")
    x = torch.full((1, H, W, 4), 9, dtype=torch.int8, device=DEV)
    top = (H - R) // st * st  # first input row of the last output row
    cut = torch.randint(-128, 128, (1, R, W, 4), generator=g, device=DEV).to(torch.int8)
    x[:, top:top + R] = cut
    w = rgb_filters(g, K, R, -128, 128, torch.int8)
    colsum = torch.empty(K, dtype=torch.int32, device=DEV)
    fx.weight_colsum(h, w, K, w.shape[1], colsum)
    Ho, Wo = (H - R) // st + 1, (W - R) // st + 1
    acc = torch.empty((Ho, Wo, K), dtype=torch.int32, device=DEV)
    want = torch.empty((1, Wo, K), dtype=torch.int32, device=DEV)
    fx.qconv(h, fx.conv_desc(1, H, W, 4, K, R, R, st, 0), x, fx.U8OFF, w, colsum, None, acc)
    fx.qconv(h, fx.conv_desc(1, R, W, 4, K, R, R, st, 0), cut, fx.U8OFF, w, colsum, None, want)
    torch.cuda.synchronize()
    assert torch.equal(acc[-1:], want)
