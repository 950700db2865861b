"""GPU parity: the convolution kernels, through the C ABI, against the oracle's direct
convolution on the same seeded tensors (several tiles, ragged tails, both strides)."""
import numpy as np
import pytest
import torch

import paper_2107_00961_amd as R
from oracle import layers as L
from tests.gpu_util import assert_close

pytestmark = pytest.mark.gpu

#         N   H   W   C    K   R st pad
CASES = [(2, 16, 16, 16, 16, 3, 1, 1),      # tiny config's block shape
         (3, 12, 12, 64, 128, 3, 2, 1),     # stride 2, ragged M = 108
         (4, 16, 16, 64, 64, 3, 1, 1),      # several M tiles
         (2, 8, 8, 64, 256, 1, 1, 0),       # 1x1
         (2, 8, 8, 64, 128, 1, 2, 0),       # 1x1 stride 2 (downsample shortcut)
         (3, 10, 10, 32, 64, 1, 1, 0),      # stem-as-GEMM shape
         (2, 6, 6, 48, 80, 3, 1, 1),        # channel counts that are not multiples of the K-chunk
         (32, 32, 32, 64, 256, 3, 1, 1),    # large enough for the 128x128 tile
         (2, 8, 8, 512, 512, 3, 1, 1),      # 128x128 weight-gradient tile
         (5, 14, 14, 32, 32, 3, 2, 1),      # stride 2 with odd output size 7
         (2, 12, 12, 16, 32, 5, 1, 2),      # 5x5
         (2, 14, 14, 16, 32, 5, 2, 2),      # 5x5 stride 2: three and two taps per parity class
         (1, 9, 9, 16, 16, 7, 1, 3),        # 7x7
         (2, 16, 16, 8, 16, 7, 2, 3),       # 7x7 stride 2 pad 3 (the ImageNet stem's filter geometry)
         (2, 10, 18, 32, 32, 3, 1, 1),      # images that are not square
         (3, 12, 20, 16, 32, 3, 2, 1),      # ... stride 2 (parity classes of 6 x 10 pixels)
         (2, 6, 14, 32, 64, 1, 1, 0),       # ... 1x1
         (4, 1, 1, 32, 64, 1, 1, 0),        # one pixel per image: four GEMM rows
         (1, 3, 3, 16, 16, 3, 1, 0),        # one output pixel in all
         (3, 2, 2, 16, 16, 3, 2, 1)]        # 2x2 input, stride 2: one output pixel per image, three of four parity classes empty of taps


def _tensors(case, seed=0):
    N, H, W, C, K, RS, st, pad = case
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((N, C, H, W), dtype=np.float32)
    w = (rng.standard_normal((K, C, RS, RS), dtype=np.float32) / np.sqrt(C * RS * RS)).astype(np.float32)
    P, Q = (H + 2 * pad - RS) // st + 1, (W + 2 * pad - RS) // st + 1
    dy = rng.standard_normal((N, K, P, Q), dtype=np.float32)
    return x, w, dy


def _nhwc(a):
    return torch.from_numpy(np.ascontiguousarray(a.transpose(0, 2, 3, 1))).cuda()


@pytest.mark.parametrize("case", CASES)
def test_conv_forward(case):
    print("case", case, flush=True)
    x, w, _ = _tensors(case)
    st, pad = case[6], case[7]
    y = R.conv2d_forward(_nhwc(x), _nhwc(w), st, pad)
    torch.cuda.synchronize()
    want = L.conv2d_fwd(x, w, st, pad)
    assert_close(y.cpu().numpy().transpose(0, 3, 1, 2), want, f"conv fwd {case}")


@pytest.mark.parametrize("case", CASES)
def test_conv_dgrad(case):
    print("case", case, flush=True)
    x, w, dy = _tensors(case, 1)
    N, H, W, C, K, RS, st, pad = case
    dx = R.conv2d_dgrad(_nhwc(dy), _nhwc(w), (N, H, W, C), st, pad)
    torch.cuda.synchronize()
    want = L.conv2d_dgrad(dy, w, x.shape, st, pad)
    assert_close(dx.cpu().numpy().transpose(0, 3, 1, 2), want, f"conv dgrad {case}")


@pytest.mark.parametrize("case", CASES)
def test_conv_wgrad(case):
    print("case", case, flush=True)
    x, w, dy = _tensors(case, 2)
    N, H, W, C, K, RS, st, pad = case
    # keep the sums O(1) so the absolute floor of the bound means what it means for real gradients:
    # an fp32 sum of L products of O(1) terms carries an absolute error ~ sqrt(L) * 2^-24 * sqrt(L)
    dy = (dy / np.sqrt(dy.shape[0] * dy.shape[2] * dy.shape[3])).astype(np.float32)
    dw = R.conv2d_wgrad(_nhwc(dy), _nhwc(x), (K, RS, RS, C), st, pad)
    torch.cuda.synchronize()
    want = L.conv2d_wgrad(dy, x, w.shape, st, pad)
    assert_close(dw.cpu().numpy().transpose(0, 3, 1, 2), want, f"conv wgrad {case}")


# ---- fp32 3x3 stride-1 layers of at least 48 input channels: operands taken apart into three bf16 parts --------------
# Edges of the 64- and 128-pixel tiles, of the 64-channel chunks (the last one ragged, an odd and an even number of them)
# and of the 64-wide output tiles; images one pixel wide, smaller than a tile, and at and past the widest that is staged.
# (All but two of these have so few output tiles that they run on the small-output kernel; see SPLIT_LARGE_CASES.)
#              N   H   W   C    K   R st pad
SPLIT_CASES = [(1, 1, 1, 64, 16, 3, 1, 1), (5, 3, 1, 48, 80, 3, 1, 1), (1, 8, 8, 64, 64, 3, 1, 1), (1, 5, 13, 52, 68, 3, 1, 1),
               (13, 5, 2, 128, 48, 3, 1, 1), (2, 3, 56, 64, 32, 3, 1, 1), (2, 3, 57, 64, 32, 3, 1, 1), (129, 4, 4, 132, 1028, 3, 1, 1),
               (2, 127, 31, 64, 300, 3, 1, 1), (3, 9, 7, 192, 64, 3, 1, 1)]


@pytest.mark.parametrize("case", SPLIT_CASES)
def test_conv_split_forward_and_dgrad(case):
    print("case", case, flush=True)
    x, w, _ = _tensors(case, 8)
    y = R.conv2d_forward(_nhwc(x), _nhwc(w), 1, 1)
    N, H, W, C, K = case[:5]
    # the data gradient of the layer with in- and output channels exchanged has the same tiles
    dx = R.conv2d_dgrad(_nhwc(x), _nhwc(np.ascontiguousarray(w.transpose(1, 0, 2, 3))), (N, H, W, K), 1, 1)
    torch.cuda.synchronize()
    assert_close(y.cpu().numpy().transpose(0, 3, 1, 2), L.conv2d_fwd(x, w, 1, 1), f"conv fwd {case}")
    want = L.conv2d_dgrad(x, w.transpose(1, 0, 2, 3), (N, K, H, W), 1, 1)
    assert_close(dx.cpu().numpy().transpose(0, 3, 1, 2), want, f"conv dgrad {case}")


# nine-tap weight gradient: ragged channel tiles and pixel chunks, one split and several, the ring of staged pixels run
# through many times, images one pixel wide and the widest that is staged, and a layer just too small for it
# (Most of these are too small for that kernel; see WGRAD3_EDGE_CASES.)
#              N   H   W   C    K   R st pad
WGRAD3_CASES = [(3, 3, 1, 700, 680, 3, 1, 1), (1, 5, 5, 512, 344, 3, 1, 1), (2, 45, 56, 36, 40, 3, 1, 1), (7, 19, 33, 64, 64, 3, 1, 1),
                (64, 16, 16, 16, 16, 3, 1, 1), (63, 16, 16, 16, 16, 3, 1, 1), (130, 4, 4, 80, 132, 3, 1, 1), (2, 31, 57, 64, 64, 3, 1, 1)]


@pytest.mark.parametrize("case", WGRAD3_CASES)
def test_conv_nine_tap_wgrad(case):
    print("case", case, flush=True)
    x, w, dy = _tensors(case, 10)
    N, H, W, C, K = case[:5]
    dy = (dy / np.sqrt(N * H * W)).astype(np.float32)
    dw = R.conv2d_wgrad(_nhwc(dy), _nhwc(x), (K, 3, 3, C), 1, 1)
    torch.cuda.synchronize()
    assert_close(dw.cpu().numpy().transpose(0, 3, 1, 2), L.conv2d_wgrad(dy, x, w.shape, 1, 1), f"conv wgrad {case}")


def _same_values(got, want, what):
    # infinities and NaN where float64 has them, everything else close (values next to the largest float included)
    with np.errstate(over="ignore"):
        np.testing.assert_allclose(got.transpose(0, 3, 1, 2), want.astype(np.float32), rtol=1e-4, atol=1e-4, equal_nan=True, err_msg=what)


def test_conv_split_infinities():
    x, w, _ = _tensors((4, 8, 8, 64, 96, 3, 1, 1), 9)
    x[0, 5, 2, 3], x[1, 7, 0, 0], x[2, 9, 7, 7] = np.inf, -np.inf, np.nan
    x[3, 1, 4, 4] = 3.4e38   # finite, but its leading bf16 part is an infinity
    y = R.conv2d_forward(_nhwc(x), _nhwc(w), 1, 1)
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        _same_values(y.cpu().numpy(), L.conv2d_fwd(x.astype(np.float64), w, 1, 1), "fwd")


def test_conv_nine_tap_wgrad_infinities():
    case = (8, 16, 16, 72, 72, 3, 1, 1)
    x, w, dy = _tensors(case, 11)
    dy /= 64
    x[0, 5, 2, 3], x[1, 66, 8, 0], x[2, 9, 7, 7], dy[3, 70, 9, 9] = np.inf, -np.inf, np.nan, np.inf
    x[4, 2, 8, 8] = 3.4e38
    dw = R.conv2d_wgrad(_nhwc(dy), _nhwc(x), (72, 3, 3, 72), 1, 1)
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        _same_values(dw.cpu().numpy(), L.conv2d_wgrad(dy.astype(np.float64), x, w.shape, 1, 1), "wgrad")


def _launched(f):
    """The result of f and the names of the kernels it launched."""
    R.profile_enable(True)
    try:
        out = f()
        return out, {k["name"] for k in R.profile_read()}
    finally:
        R.profile_enable(False)


# forward (or data gradient) on 64- and on 128-pixel tiles, and the weight gradient of the same layers; the last one ragged
# in every size
#                   N   H   W   C    K   R st pad
SPLIT_EDGE_CASES = [((33, 8, 8, 96, 288, 3, 1, 1), "64x64"), ((65, 16, 16, 64, 128, 3, 1, 1), "128x64"),
                    ((53, 9, 7, 52, 300, 3, 1, 1), "64x64")]


def _split_layer(case, x, w, dy):
    """y and dx (of the layer with in- and output channels exchanged) and dw on the kernels that take operands apart."""
    (N, H, W, C, K, *_), tile = case
    wt = np.ascontiguousarray(w.transpose(1, 0, 2, 3))
    xd, wd, wtd, dyd = _nhwc(x), _nhwc(w), _nhwc(wt), _nhwc(dy)
    (y, dx, dw), ran = _launched(lambda: (R.conv2d_forward(xd, wd, 1, 1), R.conv2d_dgrad(xd, wtd, (N, H, W, K), 1, 1),
                                          R.conv2d_wgrad(dyd, xd, (K, 3, 3, C), 1, 1)))
    assert {"conv3_f32_fwd_" + tile, "conv3_f32_bwd_" + tile, "wgrad3_f32"} <= ran, ran
    return [t.cpu().numpy() for t in (y, dx, dw)]


# the edges of SPLIT_CASES on layers of more than 256 tiles of 32x32, by the tile they run on (None: not taken apart)
#                      N   H   W   C    K   R st pad
SPLIT_LARGE_CASES = [((700, 3, 1, 48, 300, 3, 1, 1), "64x64"), ((1, 5, 13, 52, 2756, 3, 1, 1), "64x64"), ((170, 5, 2, 128, 324, 3, 1, 1), "64x64"),
                     ((3, 29, 56, 64, 200, 3, 1, 1), "64x64"), ((3, 29, 57, 64, 200, 3, 1, 1), None), ((3, 29, 56, 44, 200, 3, 1, 1), None),
                     ((129, 16, 16, 132, 68, 3, 1, 1), "128x64"), ((11, 60, 56, 48, 68, 3, 1, 1), "128x64"), ((2, 127, 31, 64, 300, 3, 1, 1), "128x64")]


@pytest.mark.parametrize("case", SPLIT_LARGE_CASES)
def test_conv_split_large(case):
    _, ran = _launched(lambda: test_conv_split_forward_and_dgrad(case[0]))
    names = {n for n in ran if n.startswith("conv3_f32")}
    assert names == ({"conv3_f32_fwd_" + case[1], "conv3_f32_bwd_" + case[1]} if case[1] else set()), ran


# which weight gradient a layer gets: around 2^14 pixels per 64 x 64 channels and around 640 pixels, ragged channel tiles and pixel
# chunks, one split and several, images one pixel wide, the widest that the nine-tap kernel stages and a wider one
#                     N   H   W   C    K   R st pad
WGRAD3_EDGE_CASES = [((64, 16, 16, 16, 16, 3, 1, 1), True), ((63, 16, 16, 16, 16, 3, 1, 1), False), ((700, 3, 1, 140, 200, 3, 1, 1), True),
                     ((3, 3, 1, 700, 680, 3, 1, 1), False), ((16, 4, 4, 512, 512, 3, 1, 1), True), ((2, 16, 16, 432, 432, 3, 1, 1), False),
                     ((10, 8, 8, 324, 328, 3, 1, 1), True), ((9, 8, 8, 324, 328, 3, 1, 1), False), ((7, 45, 56, 36, 40, 3, 1, 1), True),
                     ((5, 64, 57, 64, 64, 3, 1, 1), False), ((27, 19, 33, 64, 64, 3, 1, 1), True), ((200, 4, 4, 80, 132, 3, 1, 1), True)]


@pytest.mark.parametrize("case", WGRAD3_EDGE_CASES)
def test_conv_wgrad_route(case):
    print("case", case, flush=True)
    (N, H, W, C, K, *_), nine = case
    x, w, dy = _tensors(case[0], 17)
    dy = (dy / np.sqrt(N * H * W)).astype(np.float32)
    xd, dyd = _nhwc(x), _nhwc(dy)
    dw, ran = _launched(lambda: R.conv2d_wgrad(dyd, xd, (K, 3, 3, C), 1, 1))
    assert ("wgrad3_f32" in ran) == nine, ran
    assert_close(dw.cpu().numpy().transpose(0, 3, 1, 2), L.conv2d_wgrad(dy, x, w.shape, 1, 1), f"conv wgrad {case}")


@pytest.mark.parametrize("case", SPLIT_EDGE_CASES)
def test_conv_split_products_near_the_largest_float(case):
    """v * v is finite in fp32, the product of the bf16 numbers next to v is not."""
    print("case", case, flush=True)
    x, w, dy = _tensors(case[0], 14)
    v = np.float32((2 - 2.0 ** -9.5) * 2.0 ** 63)
    x[1, 5, 2, 3], x[2, 6, 7, 5] = v, -v
    w[3, 5, 1, 1] = w[7, 6, 0, 2] = v
    dy /= 64
    dy[1, 9, 2, 3] = v
    want = [L.conv2d_fwd(x, w, 1, 1), L.conv2d_dgrad(x, w.transpose(1, 0, 2, 3), (len(x), len(w)) + x.shape[2:], 1, 1),
            L.conv2d_wgrad(dy, x, w.shape, 1, 1)]
    for got, t, what in zip(_split_layer(case, x, w, dy), want, ("fwd", "dgrad", "wgrad")):
        assert np.abs(t).max() > 3.39e38 and np.isfinite(t.astype(np.float32)).all()
        _same_values(got, t, what)


@pytest.mark.parametrize("case", SPLIT_EDGE_CASES)
def test_conv_split_infinities_on_both_tiles(case):
    """As the tests of infinities above, on layers too large for the 32x32 tiles; tiles with and without one."""
    print("case", case, flush=True)
    x, w, dy = _tensors(case[0], 16)
    dy /= 64
    x[0, 5, 2, 3], x[1, 37, 0, 0], x[2, 9, 7, 5], dy[3, 50, 4, 3] = np.inf, -np.inf, np.nan, np.inf
    x[4, 1, 4, 4] = 3.4e38   # finite, but its leading bf16 part is an infinity
    with np.errstate(invalid="ignore", over="ignore"):
        X = x.astype(np.float64)
        want = [L.conv2d_fwd(X, w, 1, 1), L.conv2d_dgrad(X, w.transpose(1, 0, 2, 3), (len(x), len(w)) + x.shape[2:], 1, 1),
                L.conv2d_wgrad(dy.astype(np.float64), X, w.shape, 1, 1)]
        for got, t, what in zip(_split_layer(case, x, w, dy), want, ("fwd", "dgrad", "wgrad")):
            assert np.isfinite(t).any() and not np.isfinite(t).all()
            _same_values(got, t, what)


@pytest.mark.parametrize("e", [-100, -104, -110, -118, -126, -134])
@pytest.mark.parametrize("case", SPLIT_EDGE_CASES)
def test_conv_split_small_operands(case, e):
    """Operands so small that bf16 has no numbers for their lower parts, against others large enough for normal results."""
    print("case", case, e, flush=True)
    x, w, dy = _tensors(case[0], 15)
    dy = dy / np.float32(64)
    s = np.float32(2.0 ** 60)
    for small_x in (True, False):
        t = np.ldexp(np.float32(1), e).astype(np.float32)
        xs, ws, ds = (x * t, w * s, dy * s) if small_x else (x * s, w * t, dy * t)
        y, dx, dw = _split_layer(case, xs, ws, ds)
        r = 1 / (float(t) * float(s))
        X, W, D = xs.astype(np.float64), ws.astype(np.float64) * r, ds.astype(np.float64) * r
        shape = (len(x), len(w)) + x.shape[2:]
        for got, want, what in ((y, L.conv2d_fwd(X, W, 1, 1), "fwd"), (dx, L.conv2d_dgrad(X, W.transpose(1, 0, 2, 3), shape, 1, 1), "dgrad"),
                                (dw, L.conv2d_wgrad(D, X, w.shape, 1, 1), "wgrad")):
            # up to 2592 fp32 additions, each rounding by at most 2^-24 of a partial sum, in random directions
            assert np.linalg.norm(got.transpose(0, 3, 1, 2) * r - want) <= np.sqrt(2592) * 2.0 ** -24 * np.linalg.norm(want), what


@pytest.mark.parametrize("case", SPLIT_EDGE_CASES)
def test_conv_split_one_small_operand(case):
    """A single small operand among zeros, wherever it is staged: every tap of the filter in a 64-channel tile of its own, one
    pixel an image."""
    print("case", case, flush=True)
    x, w, dy = _tensors(case[0], 18)
    (N, H, W, C, K, *_), tile = case
    big, small = np.float32(2.0 ** 60), np.float32(1.2345678e-36)   # 2^-119.3
    r = float(big) * float(small)
    tiles = (K + 63) // 64
    rng = np.random.default_rng(19)
    for first in range(0, 9, tiles):
        w1 = np.zeros_like(w)
        for t in range(first, min(9, first + tiles)):
            w1[64 * (t - first) + 7 + t, (t * 11 + 3) % C, t // 3, t % 3] = small
        (y, dx, _) = _split_layer(case, x * big, w1, dy)
        shape = (N, K, H, W)
        for got, want, what in ((y, L.conv2d_fwd(x, w1 / float(small), 1, 1), "fwd"),
                                (dx, L.conv2d_dgrad(x, w1.transpose(1, 0, 2, 3) / float(small), shape, 1, 1), "dgrad")):
            # one product: its rounding, and that of x * big and of small against what the oracle takes
            assert np.linalg.norm(got.transpose(0, 3, 1, 2) / r - want) <= 2.0 ** -23 * np.linalg.norm(want), (first, what)
    x1, d1 = np.zeros_like(x), np.zeros_like(dy)
    for n in range(N):
        x1[n, rng.integers(C), rng.integers(H), rng.integers(W)] = small
        d1[n, rng.integers(K), rng.integers(H), rng.integers(W)] = small
    y, dx, dw = _split_layer(case, x1, w * big, dy * big)
    _, _, dw2 = _split_layer(case, x * big, w, d1)
    X, D = x1 / float(small), d1 / float(small)
    for got, want, what in ((y, L.conv2d_fwd(X, w, 1, 1), "fwd"), (dx, L.conv2d_dgrad(X, w.transpose(1, 0, 2, 3), shape, 1, 1), "dgrad"),
                            (dw, L.conv2d_wgrad(dy, X, w.shape, 1, 1), "wgrad, x"), (dw2, L.conv2d_wgrad(D, x, w.shape, 1, 1), "wgrad, dy")):
        # a few products at most
        assert np.linalg.norm(got.transpose(0, 3, 1, 2) / r - want) <= 2.0 ** -22 * np.linalg.norm(want), what


# ---- small outputs: 32x32 tiles, the reduction split among eight waves ------------------------------------------------
# One tile and 256 (and just past them: the larger tiles), ragged pixel and channel tiles, channels that fill a part of a
# 128-byte unit, fewer units than waves, an odd share, strides, 1x1 / 5x5 / 7x7 filters, parity classes without a tap
#              N   H   W   C    K   R st pad
SMALL_CASES = [(1, 1, 1, 144, 8, 1, 1, 0), (1, 4, 4, 512, 512, 3, 1, 1), (1, 7, 7, 520, 40, 3, 1, 1), (2, 5, 3, 16, 24, 3, 1, 1),
               (4, 16, 16, 128, 256, 3, 1, 1), (33, 8, 8, 128, 128, 3, 1, 1), (3, 9, 11, 1032, 72, 1, 1, 0), (2, 14, 14, 256, 64, 3, 2, 1),
               (1, 8, 8, 640, 96, 1, 2, 0), (5, 4, 6, 64, 136, 5, 1, 2), (2, 8, 10, 48, 32, 7, 2, 3), (1, 2, 2, 1024, 2048, 1, 1, 0)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("case", SMALL_CASES)
def test_conv_small_forward_and_dgrad(case, dt):
    print("case", case, dt, flush=True)
    N, H, W, C, K, R_, st, pad = case
    x, w, _ = _tensors(case, 12)
    bf = dt == "bf16"
    wt = np.ascontiguousarray(w.transpose(1, 0, 2, 3))   # layer K -> C
    rnd = (lambda t: torch.from_numpy(t).bfloat16().float().numpy()) if bf else (lambda t: t)
    dev = (lambda t: _nhwc(t).bfloat16()) if bf else _nhwc
    x, w, wt = rnd(x), rnd(w), rnd(wt)
    y = R.conv2d_forward(dev(x), dev(w), st, pad)
    P, Q = (H + 2 * pad - R_) // st + 1, (W + 2 * pad - R_) // st + 1
    # data gradient of a layer K -> C, whose output gradient [N][P][Q][C] makes the reduction as long as the forward's
    g = rnd(np.random.default_rng(13).standard_normal((N, C, P, Q)).astype(np.float32))
    dx = R.conv2d_dgrad(dev(g), dev(wt), (N, H, W, K), st, pad)
    torch.cuda.synchronize()
    # results are of order 1.  bf16: the output's own rounding, 2^-9 of a value; fp32: each of up to 4680 additions rounds by at
    # most 2^-24 of a partial sum of order 1, in random directions: sqrt(4680) * 2^-24 = 4e-6, and 5 times that for the largest
    tol = dict(rtol=2.0 ** -8, atol=2e-3) if bf else dict(rtol=1e-5, atol=2e-5)
    np.testing.assert_allclose(y.float().cpu().numpy().transpose(0, 3, 1, 2), L.conv2d_fwd(x, w, st, pad), err_msg=f"fwd {case}", **tol)
    np.testing.assert_allclose(dx.float().cpu().numpy().transpose(0, 3, 1, 2), L.conv2d_dgrad(g, wt, (N, K, H, W), st, pad),
                               err_msg=f"dgrad {case}", **tol)


# ---- bf16 operands, fp32 accumulation ---------------------------------------------------------
# Inputs are bfloat16 numbers, so the oracle's float64 result is the exact convolution of what the
# kernel reads.  Outputs stored as bfloat16 carry half a bfloat16 ulp (2^-9 relative, 2^-8 of the
# value's power of two) on top of the fp32 accumulation error; weight gradients are fp32.
BF16_CASES = [c for c in CASES if c[3] % 8 == 0 and c[4] % 8 == 0]


def _bf16_tensors(case, seed):
    x, w, dy = _tensors(case, seed)
    r = lambda a: torch.from_numpy(a).to(torch.bfloat16)
    return r(x), r(w), r(dy)


def _nhwc_t(t):
    return t.permute(0, 2, 3, 1).contiguous().cuda()


def _f64(t):
    return t.to(torch.float64).numpy()


@pytest.mark.parametrize("case", BF16_CASES)
def test_conv_forward_bf16(case):
    print("case", case, flush=True)
    x, w, _ = _bf16_tensors(case, 3)
    st, pad = case[6], case[7]
    y = R.conv2d_forward(_nhwc_t(x), _nhwc_t(w), st, pad)
    torch.cuda.synchronize()
    assert y.dtype == torch.bfloat16
    want = L.conv2d_fwd(_f64(x), _f64(w), st, pad)
    assert_close(y.cpu().to(torch.float64).numpy().transpose(0, 3, 1, 2), want, f"bf16 conv fwd {case}",
                 rtol=2.0 ** -8, atol=1e-5)


@pytest.mark.parametrize("case", BF16_CASES)
def test_conv_dgrad_bf16(case):
    print("case", case, flush=True)
    x, w, dy = _bf16_tensors(case, 4)
    N, H, W, C, K, RS, st, pad = case
    dx = R.conv2d_dgrad(_nhwc_t(dy), _nhwc_t(w), (N, H, W, C), st, pad)
    torch.cuda.synchronize()
    assert dx.dtype == torch.bfloat16
    want = L.conv2d_dgrad(_f64(dy), _f64(w), tuple(x.shape), st, pad)
    assert_close(dx.cpu().to(torch.float64).numpy().transpose(0, 3, 1, 2), want, f"bf16 conv dgrad {case}",
                 rtol=2.0 ** -8, atol=1e-5)


# one filter row per workgroup (bf16 3x3 weight gradients from 2^28 products a tap, or 2^18 pairs of channels): ragged channel
# tiles, one split and several, odd and even numbers of 64-pixel chunks, the ring of staged rows run through many times, images
# one pixel wide and wide ones, and a layer just too small for it
#                  N   H   W   C    K   R st pad
WGRAD_ROW_CASES = [(1, 5, 5, 512, 512, 3, 1, 1), (3, 7, 1, 520, 512, 3, 1, 1), (2, 1, 90, 584, 456, 3, 1, 1), (7, 4, 4, 1032, 264, 3, 1, 1),
                   (5, 64, 45, 136, 152, 3, 1, 1), (33, 45, 45, 64, 64, 3, 1, 1), (16, 64, 64, 64, 64, 3, 1, 1), (16, 64, 63, 64, 64, 3, 1, 1)]


@pytest.mark.parametrize("case", BF16_CASES + WGRAD_ROW_CASES)
def test_conv_wgrad_bf16(case):
    print("case", case, flush=True)
    x, w, dy = _bf16_tensors(case, 5)
    N, H, W, C, K, RS, st, pad = case
    dy = (dy.to(torch.float32) / float(np.sqrt(dy.shape[0] * dy.shape[2] * dy.shape[3]))).to(torch.bfloat16)
    dw = R.conv2d_wgrad(_nhwc_t(dy), _nhwc_t(x), (K, RS, RS, C), st, pad)
    torch.cuda.synchronize()
    assert dw.dtype == torch.float32
    want = L.conv2d_wgrad(_f64(dy), _f64(x), tuple(w.shape), st, pad)
    assert_close(dw.cpu().numpy().transpose(0, 3, 1, 2), want, f"bf16 conv wgrad {case}")


# which bf16 weight gradient a layer gets: long reductions of few tiles (two workgroups a compute unit), 64 tiles up to 2^12
# pixels and beyond
#                        N   H   W   C    K   R st pad
WGRAD_ROW_EDGE_CASES = [((201, 32, 32, 40, 40, 3, 1, 1), True), ((49, 16, 16, 256, 256, 3, 1, 1), True),
                        ((64, 8, 8, 512, 456, 3, 1, 1), True), ((65, 8, 8, 512, 456, 3, 1, 1), False)]


@pytest.mark.parametrize("case", WGRAD_ROW_EDGE_CASES)
def test_conv_wgrad_bf16_route(case):
    _, ran = _launched(lambda: test_conv_wgrad_bf16(case[0]))
    assert ("wgrad3_row_bf16" in ran) == case[1], ran


# ---- the stem convolution: implicit GEMM straight from the [N,C,H,W] fp32 image ----------------------------
#              N  C   H   W   K  R st pad
STEM_CASES = [(4, 3, 16, 16, 16, 3, 1, 1),       # the tiny configuration's stem
              (5, 3, 32, 32, 64, 3, 1, 1),       # CIFAR-shaped: four output rows per tile
              (3, 3, 40, 40, 16, 7, 2, 3),       # 7x7 stride 2: 20 x 20 outputs, five rows per tile
              (2, 3, 224, 224, 64, 7, 2, 3),     # ImageNet-shaped: one 112-pixel row per tile
              (2, 3, 18, 30, 32, 3, 1, 1),       # rectangular, 32 output channels (one tile of channels)
              (2, 4, 12, 12, 96, 5, 2, 2),       # four input channels, 96 output channels (64 + 32), 5x5
              (1, 1, 9, 9, 16, 3, 1, 0),         # one channel, no padding
              (2, 3, 26, 134, 48, 3, 1, 1),      # 134 output columns: tiles of 67 columns (rows not a multiple of 4 wide)
              (1, 3, 8, 256, 16, 3, 1, 1),       # two tiles of 128 columns along a row that is staged in 16-byte pieces
              (1, 3, 6, 268, 16, 3, 1, 1)]       # four tiles of 67 columns: every tile starts at another offset mod 4


def _stem_tensors(case, seed, bf16):
    N, C, H, W, K, RS, st, pad = case
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((N, C, H, W), dtype=np.float32)
    w = (rng.standard_normal((K, C, RS, RS), dtype=np.float32) / np.sqrt(C * RS * RS)).astype(np.float32)
    P, Q = (H + 2 * pad - RS) // st + 1, (W + 2 * pad - RS) // st + 1
    dy = (rng.standard_normal((N, K, P, Q), dtype=np.float32) / np.sqrt(N * P * Q)).astype(np.float32)
    if bf16:   # bfloat16 numbers, so the float64 result is the exact convolution of what the kernel multiplies
        x, w, dy = (torch.from_numpy(a).to(torch.bfloat16).to(torch.float32).numpy() for a in (x, w, dy))
    return x, w, dy


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("case", STEM_CASES)
def test_stem_conv_forward(case, bf16):
    print("case", case, "bf16" if bf16 else "f32", flush=True)
    x, w, _ = _stem_tensors(case, 6, bf16)
    st, pad = case[6], case[7]
    y = R.stem_conv2d_forward(torch.from_numpy(x).cuda(), _nhwc(w), st, pad, bf16=bf16)
    torch.cuda.synchronize()
    want = L.conv2d_fwd(x, w, st, pad)
    got = y.cpu().to(torch.float64).numpy().transpose(0, 3, 1, 2)
    if bf16:
        assert_close(got, want, f"bf16 stem fwd {case}", rtol=2.0 ** -8, atol=1e-5)
    else:
        assert_close(got, want, f"stem fwd {case}")


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("case", STEM_CASES)
def test_stem_conv_wgrad(case, bf16):
    print("case", case, "bf16" if bf16 else "f32", flush=True)
    x, w, dy = _stem_tensors(case, 7, bf16)
    N, C, H, W, K, RS, st, pad = case
    dyd = _nhwc(dy)
    if bf16:
        dyd = dyd.to(torch.bfloat16)
    dw = R.stem_conv2d_wgrad(dyd, torch.from_numpy(x).cuda(), (K, RS, RS, C), st, pad)
    torch.cuda.synchronize()
    want = L.conv2d_wgrad(dy, x, w.shape, st, pad)
    assert_close(dw.cpu().numpy().transpose(0, 3, 1, 2), want, f"stem wgrad {case} {'bf16' if bf16 else 'f32'}")


def test_stem_conv_rejects_bad_shapes():
    x = torch.zeros((1, 5, 8, 8), device="cuda")
    with pytest.raises(R.ResistError):
        R.stem_conv2d_forward(x, torch.zeros((16, 3, 3, 5), device="cuda"), 1, 1)        # five input channels
    with pytest.raises(R.ResistError):
        R.stem_conv2d_forward(torch.zeros((1, 3, 8, 8), device="cuda"), torch.zeros((24, 3, 3, 3), device="cuda"), 1, 1)   # K = 24


def test_conv_rejects_bad_shapes():
    x = torch.zeros((1, 4, 4, 6), device="cuda")
    w = torch.zeros((8, 3, 3, 6), device="cuda")
    with pytest.raises(R.ResistError):
        R.conv2d_forward(x, w, 1, 1)          # C not a multiple of 4
    x = torch.zeros((1, 5, 5, 8), device="cuda")
    w = torch.zeros((8, 3, 3, 8), device="cuda")
    with pytest.raises(R.ResistError):
        R.conv2d_dgrad(torch.zeros((1, 3, 3, 8), device="cuda"), w, (1, 5, 5, 8), 2, 1)   # odd size, stride 2


# 3x3 layers on filters in matrix fragments, by the tile they run on, the data gradient on the layer with in- and output channels
# exchanged: 96 pixels (two to four chunks, the last tile ragged, 65 and 130 output channels' worth of column tiles), filters larger than
# the pixels (tiles ordered along the pixels), bf16 from 256 channels (one that ends in mid-chunk, images one pixel wide and
# the widest)
#                       dt  N   H   W   C    K   R st pad
FRAGMENT_CASES = [(("f32", 77, 8, 8, 256, 256, 3, 1, 1), "96x64"), (("f32", 160, 11, 11, 128, 68, 3, 1, 1), "96x64"), (("f32", 171, 5, 5, 192, 260, 3, 1, 1), "96x64"),
                  (("f32", 40, 4, 4, 512, 512, 3, 1, 1), "64x64"), (("bf16", 33, 8, 8, 256, 256, 3, 1, 1), "64x64"), (("bf16", 13, 9, 7, 264, 336, 3, 1, 1), "64x64"),
                  (("bf16", 300, 3, 1, 320, 320, 3, 1, 1), "64x64"), (("bf16", 1, 19, 56, 256, 264, 3, 1, 1), "64x64"), (("bf16", 40, 4, 4, 512, 520, 3, 1, 1), "64x64")]


def _bf16_exact(a):
    return torch.from_numpy(a).to(torch.bfloat16).float().numpy()


@pytest.mark.parametrize("case", FRAGMENT_CASES)
def test_conv_filter_fragments(case):
    (dt, *shape), tile = case
    print("case", case, flush=True)
    N, H, W, C, K = shape[:5]
    x, w, _ = _tensors(tuple(shape), 21)
    bf16 = dt == "bf16"
    if bf16:
        x, w = _bf16_exact(x), _bf16_exact(w)
    dev = lambda a: _nhwc(a).to(torch.bfloat16 if bf16 else torch.float32)
    xd, wd, wtd = dev(x), dev(w), dev(np.ascontiguousarray(w.transpose(1, 0, 2, 3)))
    from tests import internals as I
    # the data gradient leaves the fragments of the transposed filter in its workspace, which are those of w for a forward pass
    ws = I.workspace((N, H, W, K, C, 3, 1, 1), bf16)
    y = torch.empty((N, H, W, K), device="cuda", dtype=xd.dtype)
    dx, ran = _launched(lambda: I.dgrad_call((N, H, W, K, C, 3, 1, 1), xd, wtd, ws))
    assert {n for n in ran if n.startswith("conv3_")} == {f"conv3_{dt}_bwd_{tile}"}, ran
    _, ran = _launched(lambda: I.conv_fwd(I.geom(N, H, W, C, K, 3, 1, 1), int(bf16), xd, wd, y, prep=ws))
    assert {n for n in ran if n.startswith("conv3_")} == {f"conv3_{dt}_fwd_{tile}"}, ran
    for got, want, what in ((y, L.conv2d_fwd(x, w, 1, 1), "fwd"), (dx, L.conv2d_dgrad(x, w.transpose(1, 0, 2, 3), (N, K, H, W), 1, 1), "dgrad")):
        got = got.float().cpu().numpy().transpose(0, 3, 1, 2)
        if bf16:   # half an ulp of the stored result beside the fp32 sums
            np.testing.assert_allclose(got, want, rtol=2.0 ** -8, atol=1e-5, err_msg=what)
        else:
            assert_close(got, want, f"{what} {case}")


# fp32 3x3 layers without room for the filter's fragments run on its rows, in the same tiles: 64, 96 and 128 pixels, images up to 32
# and up to 56 wide, one chunk of channels and several, input channels that end in mid-chunk at a multiple of eight and of four,
# ragged pixels and output channels
#                     N   H   W   C    K
LITTLE_WS_CASES = [((40, 8, 8, 64, 320), "64x64"), ((77, 8, 8, 256, 256), "96x64"), ((160, 11, 11, 128, 68), "96x64"), ((65, 16, 16, 52, 132), "128x64"),
                   ((65, 16, 17, 200, 128), "128x64"), ((3, 40, 37, 76, 72), "64x64"), ((17, 56, 56, 64, 48), "128x64"), ((11, 44, 56, 136, 96), "128x64")]


@pytest.mark.parametrize("case", LITTLE_WS_CASES)
@pytest.mark.parametrize("odd_values", [False, True])
def test_conv_forward_and_dgrad_with_little_workspace(case, odd_values):
    """Bit for bit the results of the calls with all the workspace they are told to bring; the forward call leaves its as it is."""
    from tests import internals as I
    print("case", case, odd_values, flush=True)
    (N, H, W, C, K), tile = case
    x, w, _ = _tensors((N, H, W, C, K, 3, 1, 1), 22)
    if odd_values:   # tiles that are computed again in fp32
        x[0, 5, 2, 3], x[N // 2, C - 1, 0, 0] = np.inf, np.nan
        w[K // 2, 7, 1, 2] = np.float32(1.2345678e-36)
    xd, wd, wtd = _nhwc(x), _nhwc(w), _nhwc(np.ascontiguousarray(w.transpose(1, 0, 2, 3)))
    back = (N, H, W, K, C, 3, 1, 1)   # the data gradient of the layer with in- and output channels exchanged
    ws, least = I.workspace(back, False), torch.empty(K * 9 * C, device="cuda")
    dx, ran = _launched(lambda: I.dgrad_call(back, xd, wtd, ws))
    assert f"conv3_f32_bwd_{tile}" in ran, ran
    dx0, ran = _launched(lambda: I.dgrad_call(back, xd, wtd, least))
    assert f"conv3_f32_bwd_{tile}" in ran, ran
    y = torch.empty((N, H, W, K), device="cuda")
    I.conv_fwd(I.geom(N, H, W, C, K, 3, 1, 1), 0, xd, wd, y, prep=ws)
    full = torch.full_like(I.workspace((N, H, W, C, K, 3, 1, 1), False), 0x5a)
    y0, ran = _launched(lambda: I.forward_call((N, H, W, C, K, 3, 1, 1), xd, wd, None))
    assert f"conv3_f32_fwd_{tile}" in ran, ran
    y1 = I.forward_call((N, H, W, C, K, 3, 1, 1), xd, wd, full)
    torch.cuda.synchronize()
    bits = lambda t: t.view(torch.int32)
    assert torch.equal(bits(dx), bits(dx0)) and torch.equal(bits(y), bits(y0)) and torch.equal(bits(y), bits(y1))
    assert bool((full == 0x5a).all())
    assert bool(torch.isfinite(y).all()) != odd_values
    if not odd_values:
        assert_close(y.cpu().numpy().transpose(0, 3, 1, 2), L.conv2d_fwd(x, w, 1, 1), "fwd")
        assert_close(dx.cpu().numpy().transpose(0, 3, 1, 2), L.conv2d_dgrad(x, w.transpose(1, 0, 2, 3), (N, K, H, W), 1, 1), "dgrad")
    with pytest.raises(R.ResistError):
        I.dgrad_call(back, xd, wtd, least[:-1])


def test_conv_fragments_second_pass_on_96_pixel_tiles():
    """Infinities in the pixels, one value of the filter too small for three parts: tiles with and without them."""
    shape = (171, 5, 5, 192, 260, 3, 1, 1)
    N, H, W, C, K = shape[:5]
    x, w, _ = _tensors(shape, 23)
    x[0, 5, 2, 3], x[40, 150, 0, 0], x[99, 9, 4, 4] = np.inf, np.nan, 3.4e38
    small = np.float32(1.2345678e-36)
    w[200, 70, 1, 2] = small
    x[3, 70, 2, 2] = np.float32(2.0 ** 120)   # times the small value: 1.6
    wt = np.ascontiguousarray(w.transpose(1, 0, 2, 3))
    xd, wd, wtd = _nhwc(x), _nhwc(w), _nhwc(wt)
    (y, dx), ran = _launched(lambda: (R.conv2d_forward(xd, wd, 1, 1), R.conv2d_dgrad(xd, wtd, (N, H, W, K), 1, 1)))
    assert {"conv3_f32_fwd_96x64", "conv3_f32_bwd_96x64"} <= ran, ran
    with np.errstate(invalid="ignore", over="ignore"):
        X = x.astype(np.float64)
        for got, want in ((y, L.conv2d_fwd(X, w, 1, 1)), (dx, L.conv2d_dgrad(X, wt, (N, K, H, W), 1, 1))):
            assert np.isfinite(want).any() and not np.isfinite(want).all()
            _same_values(got.cpu().numpy(), want, "fwd or dgrad")


# streamed 1x1 layers, forward and the data gradient of the layer with in- and output channels exchanged: the fewest pixels, a last
# range and a last 32 pixels that are ragged, input channels that fill no 16, 64, 128 or 256, output channels that fill no 32 or 128,
# and on either side of each limit
#                     N   H   W   C    K   taken
CONV1_CASES = [((64, 8, 8, 64, 128), True), ((65, 9, 7, 64, 128), False), ((66, 9, 7, 64, 128), True), ((1, 67, 71, 8, 136), True), ((5, 29, 31, 72, 200), True),
               ((5, 29, 31, 104, 208), True), ((5, 29, 31, 104, 200), False), ((18, 23, 23, 136, 1000), True), ((9, 23, 23, 136, 1000), False),
               ((35, 23, 23, 256, 512), True), ((34, 23, 23, 256, 512), False), ((19, 23, 23, 264, 1056), False), ((4097, 1, 1, 16, 152), True), ((70, 9, 7, 56, 120), False)]


@pytest.mark.parametrize("case", CONV1_CASES)
def test_conv_streamed_1x1(case):
    print("case", case, flush=True)
    (N, H, W, C, K), taken = case
    x, w, _ = _tensors((N, H, W, C, K, 1, 1, 0), 24)
    x, w = _bf16_exact(x), _bf16_exact(w)
    dev = lambda a: _nhwc(a).to(torch.bfloat16)
    xd, wd, wtd = dev(x), dev(w), dev(np.ascontiguousarray(w.transpose(1, 0, 2, 3)))
    (y, dx), ran = _launched(lambda: (R.conv2d_forward(xd, wd, 1, 0), R.conv2d_dgrad(xd, wtd, (N, H, W, K), 1, 0)))
    assert len([n for n in ran if n.startswith("conv1_")]) == (2 if taken else 0), ran
    want = L.conv2d_fwd(x, w, 1, 0)
    for got in (y, dx):   # the data gradient of the exchanged layer is the same product
        np.testing.assert_allclose(got.float().cpu().numpy().transpose(0, 3, 1, 2), want, rtol=2.0 ** -8, atol=1e-5)


# bf16 tiles chosen by how their last round fills the compute units: just past one round of 128x64, just past one of 128x128, a second
# round of 64x64 and a reduction long enough for chunks of 128 channels; ragged rows and columns, forward and, with in- and output channels
# exchanged, the data gradient
TILE_CASES = [((35, 16, 16, 512, 256, 1), "128x128x64_w8"), ((45, 16, 16, 192, 320, 1), "128x64x64_w8"), ((135, 16, 16, 256, 136, 1), "64x64x64"),
              ((9, 16, 15, 256, 264, 1), "64x64x128"), ((47, 13, 13, 1024, 256, 1), "128x64x128_w8"), ((349, 7, 7, 128, 184, 3), "128x64x64_w8"),
              ((200, 16, 16, 256, 200, 1), "128x128x64")]


@pytest.mark.parametrize("case", TILE_CASES)
def test_conv_bf16_tiles(case):
    print("case", case, flush=True)
    (N, H, W, C, K, r), tile = case
    x, w, _ = _tensors((N, H, W, C, K, r, 1, r // 2), 26)
    x, w = _bf16_exact(x), _bf16_exact(w)
    dev = lambda a: _nhwc(a).to(torch.bfloat16)
    # the data gradient turns the filter's taps round
    xd, wd, wtd = dev(x), dev(w), dev(np.ascontiguousarray(w.transpose(1, 0, 2, 3)[:, :, ::-1, ::-1]))
    (y, dx), ran = _launched(lambda: (R.conv2d_forward(xd, wd, 1, r // 2), R.conv2d_dgrad(xd, wtd, (N, H, W, K), 1, r // 2)))
    assert {n for n in ran if n != "prepare_filters"} == {f"igemm_bf16_fwd_{tile}", f"igemm_bf16_bwd_{tile}"}, ran
    want = L.conv2d_fwd(x, w, 1, r // 2)
    for got in (y, dx):
        np.testing.assert_allclose(got.float().cpu().numpy().transpose(0, 3, 1, 2), want, rtol=2.0 ** -8, atol=1e-5)


# fp32: 64x64 tiles in chunks of 64 channels up to two to a compute unit, in chunks of 32 from there up, forward and strided data gradient (whose four
# parity classes count), ragged rows and columns
F32_TILE_CASES = [((63, 16, 16, 128, 72, 1, 1), "64x64x64", None), ((65, 16, 17, 64, 68, 1, 1), "64x64x32", None), ((9, 56, 56, 64, 72, 3, 2), "64x64x64", "64x64x32"),
                  ((130, 14, 14, 64, 128, 3, 2), "64x64x64", "64x64x64")]


@pytest.mark.parametrize("case", F32_TILE_CASES)
def test_conv_f32_tiles(case):
    print("case", case, flush=True)
    (N, H, W, C, K, r, st), tile, back = case
    x, w, dy = _tensors((N, H, W, C, K, r, st, r // 2), 27)
    xd, wd, dyd = _nhwc(x), _nhwc(w), _nhwc(dy)
    y, ran = _launched(lambda: R.conv2d_forward(xd, wd, st, r // 2))
    assert {n for n in ran if n.startswith("igemm")} == {f"igemm_f32_fwd_{tile}"}, ran
    assert_close(y.cpu().numpy().transpose(0, 3, 1, 2), L.conv2d_fwd(x, w, st, r // 2), f"fwd {case}")
    if back:
        dx, ran = _launched(lambda: R.conv2d_dgrad(dyd, wd, (N, H, W, C), st, r // 2))
        assert {n for n in ran if n.startswith("igemm")} == {f"igemm_f32_bwd_{back}"}, ran
        assert_close(dx.cpu().numpy().transpose(0, 3, 1, 2), L.conv2d_dgrad(dy, w, x.shape, st, r // 2), f"dgrad {case}")


# Ranges of pixels of a streamed 1x1 layer that run to thousands: every pixel but the first of each 64 holds one value, so that each of a lane's
# additions is rounded the same way and the error of a long fp32 sum grows with its length.  A sum of 128 pixels is nine roundings deep (four
# pixels a lane, five exchanges), and there is one to a difference and one to the stored value: 12 * 2^-24 of it at most.
def _same_values_but_first(M, channels, seed):
    rng = np.random.default_rng(seed)
    first, rest = rng.uniform(2.0 ** -9, 2.0 ** -8, channels), rng.uniform(1.0, 2.0, channels)
    v = torch.from_numpy(rest.astype(np.float32)).cuda().to(torch.bfloat16).repeat(M, 1)
    v[::64] = torch.from_numpy(first.astype(np.float32)).cuda().to(torch.bfloat16)
    return v


def test_conv_streamed_1x1_long_sums():
    from tests import internals as I
    N, H, W, C, K = 1, 2048, 2048, 16, 128
    M = N * H * W
    g = I.geom(N, H, W, C, K, 1, 1, 0)
    x = torch.zeros(M, C, device="cuda", dtype=torch.bfloat16)
    x[:, 0] = 1.0
    x[:, 1] = 1.0
    x[::64, 1] = 0.0     # output channel k: w[k][0], and w[k][0] + w[k][1] in all but the first pixel of each 64
    v = _same_values_but_first(64, K, 51)
    w = torch.zeros(K, C, device="cuda", dtype=torch.bfloat16)
    w[:, 0], w[:, 1] = v[0], v[1] - v[0]
    y = torch.empty(M, K, device="cuda", dtype=torch.bfloat16)
    stats = torch.zeros(3 * ((M + 63) // 64) * K, device="cuda")
    (parts, rows), ran = _launched(lambda: I.conv_fwd(g, 1, x, w, y, stats))
    assert any(n.startswith("conv1_") for n in ran) and rows % 64 == 0 and rows > 2048 and (parts - 1) * rows < M <= parts * rows
    bound = 12 * 2.0 ** -24
    k, s1, s2 = (t.double() for t in stats[:3 * parts * K].view(3, parts, K))
    for p in range(0, parts, 29):
        d = y[p * rows:(p + 1) * rows].double() - k[p]
        for got, want in ((s1[p], d.sum(0)), (s2[p], d.square().sum(0))):
            assert float(((got - want).abs() / want.abs()).max()) <= bound, p

    # backward: the output gradient's sum, and that of its product with the normalised input
    gd = I.geom(N, H, W, K, C, 1, 1, 0)   # data gradient of a narrowing layer: K channels come out
    dx = torch.empty(M, K, device="cuda", dtype=torch.bfloat16)
    inp = _same_values_but_first(M, K, 52)
    bn = dict(y=inp, mean=torch.full((K,), 0.3, device="cuda"), invstd=torch.full((K,), 1.7, device="cuda"), scale=torch.ones(K, device="cuda"),
              shift=torch.zeros(K, device="cuda"), self=False, sums=torch.zeros(2 * ((M + 63) // 64) * K, device="cuda"))
    (parts, rows), ran = _launched(lambda: I.conv_dgrad(gd, 1, x, w, dx, bn=bn))
    assert any(n.startswith("conv1_bf16_bwd") for n in ran) and rows % 64 == 0 and rows > 2048 and (parts - 1) * rows < M <= parts * rows
    s1, s2 = (t.double() for t in bn["sums"][:2 * parts * K].view(2, parts, K))
    for p in range(0, parts, 29):
        gm, yy = dx[p * rows:(p + 1) * rows].double(), inp[p * rows:(p + 1) * rows].double()
        mean, invstd = bn["mean"].double(), bn["invstd"].double()
        for got, want in ((s1[p], gm.sum(0)), (s2[p], (gm * (yy - mean)).sum(0) * invstd)):
            assert float(((got - want).abs() / want.abs()).max()) <= bound, p


@pytest.mark.parametrize("shape", [(128, 8, 8, 256, 256), (77, 16, 16, 128, 128), (31, 14, 14, 256, 200), (40, 4, 4, 512, 512)])
def test_wgrad_of_a_step_adds_like_the_layer_call(shape):
    """fp32 3x3: beside the other kernels of a step no accumulator runs over more rows than alone -- bit for bit the same sums."""
    from tests import internals as I
    N, H, W, C, K = shape
    g = I.geom(N, H, W, C, K, 3, 1, 1)
    gen = torch.Generator(device="cuda").manual_seed(53)
    x, dy = torch.randn(N, H, W, C, generator=gen, device="cuda"), torch.randn(N, H, W, K, generator=gen, device="cuda")
    (alone, step), ran = _launched(lambda: (I.conv_wgrad(g, 0, dy, x, False), I.conv_wgrad(g, 0, dy, x, True)))
    assert "wgrad3_f32" in ran and torch.equal(alone, step)


# Which kernel a bf16 layer runs on, by shape alone (the kernels' values: above): one round of 128x128 tiles and a long reduction; tiles left only
# for a clear gain where statistics are taken; 3x3 data gradients whose 128x128 tiles fill their rounds, and do not
#                       N   H   C    K   R  call
BF16_ROUTES = [((64, 14, 1024, 256, 3, "fwd"), "igemm_bf16_fwd_128x128x64_w8"), ((31, 14, 256, 1024, 1, "stats"), "igemm_bf16_fwd_128x128x64"),
               ((31, 14, 256, 1024, 1, "fwd"), "igemm_bf16_fwd_128x64x64_w8"), ((128, 16, 512, 256, 3, "dgrad"), "igemm_bf16_bwd_128x128x64"),
               ((64, 28, 256, 256, 3, "dgrad"), "conv3_bf16_bwd_64x64"), ((128, 8, 256, 256, 3, "dgrad"), "conv3_bf16_bwd_64x64")]


@pytest.mark.parametrize("case", BF16_ROUTES)
def test_conv_bf16_routes(case):
    from tests import internals as I
    (N, H, C, K, r, call), kernel = case
    x, w = (torch.zeros(s, device="cuda", dtype=torch.bfloat16) for s in ((N, H, H, C), (K, r, r, C)))
    dy, stats = torch.zeros(N, H, H, K, device="cuda", dtype=torch.bfloat16), torch.zeros(3 * ((N * H * H + 31) // 32) * K, device="cuda")
    f = {"fwd": lambda: R.conv2d_forward(x, w, 1, r // 2), "stats": lambda: I.conv_fwd(I.geom(N, H, H, C, K, r, 1, r // 2), 1, x, w, dy, stats),
         "dgrad": lambda: R.conv2d_dgrad(dy, w, (N, H, H, C), 1, r // 2)}[call]
    _, ran = _launched(f)
    assert {n for n in ran if not n.startswith("prepare")} == {kernel}, ran


# Streamed 1x1 layers as a step calls them: statistics of the outputs, and data gradients with an addend (which may be the output), a mask and
# the sums for a BN, each there or not.  Sums are compared with those of the values as stored: 12 roundings as above, of the sum of magnitudes.
#                        N    H   W   C    K
CONV1_SIDE_CASES = [(66, 9, 7, 64, 128), (1, 67, 71, 8, 136), (50, 29, 31, 72, 200), (18, 23, 23, 136, 1000), (35, 23, 23, 256, 512), (4097, 1, 1, 16, 152)]


@pytest.mark.parametrize("case", CONV1_SIDE_CASES)
def test_conv_streamed_1x1_in_a_step(case):
    from tests import internals as I
    print("case", case, flush=True)
    N, H, W, C, K = case
    M, bound = N * H * W, 12 * 2.0 ** -24
    gen = torch.Generator(device="cuda").manual_seed(55)
    T = lambda *s: torch.randn(*s, generator=gen, device="cuda").to(torch.bfloat16)
    x, w = T(M, C), (T(K, C).float() / C ** 0.5).to(torch.bfloat16)
    prod = x.double() @ w.double().t()
    y, stats = torch.empty(M, K, device="cuda", dtype=torch.bfloat16), torch.zeros(3 * ((M + 63) // 64) * K, device="cuda")
    (parts, rows), ran = _launched(lambda: I.conv_fwd(I.geom(N, H, W, C, K, 1, 1, 0), 1, x, w, y, stats))
    assert any(n.startswith("conv1_bf16_fwd") for n in ran), ran
    assert bool(((y.double() - prod).abs() <= 2.0 ** -8 * prod.abs() + 1e-5).all())
    k, s1, s2 = (t.double() for t in stats[:3 * parts * K].view(3, parts, K))
    for p in range(parts):
        d = y[p * rows:(p + 1) * rows].double() - k[p]
        assert bool(((s1[p] - d.sum(0)).abs() <= bound * d.abs().sum(0)).all()) and bool(((s2[p] - d.square().sum(0)).abs() <= bound * d.square().sum(0)).all())
    g = I.geom(N, H, W, K, C, 1, 1, 0)
    add, mask, by = T(M, K), T(M, K), T(M, K)
    mask[0], mask[1, ::2] = 0, float("nan")   # neither is larger than zero
    mean, invstd = (torch.rand(K, generator=gen, device="cuda") + 0.5 for _ in range(2))
    for addend in ("none", "own", "out"):
        for masked in (False, True):
            for sums in (False, True):
                dx = add.clone() if addend == "out" else torch.empty_like(add)
                bn = dict(y=by, mean=mean, invstd=invstd, scale=mean, shift=mean, self=False, sums=torch.zeros(2 * ((M + 63) // 64) * K, device="cuda")) if sums else None
                (parts, rows), ran = _launched(lambda: I.conv_dgrad(g, 1, x, w, dx, dx if addend == "out" else add if addend == "own" else None,
                                                                    mask if masked else None, bn))
                assert any(n.startswith("conv1_bf16_bwd") for n in ran), ran
                want = prod + (add.double() if addend != "none" else 0.0)
                if masked:
                    want = torch.where(mask > 0, want, torch.zeros_like(want))
                assert bool(((dx.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5).all()), (addend, masked, sums)
                if sums:
                    s1, s2 = (t.double() for t in bn["sums"][:2 * parts * K].view(2, parts, K))
                    for p in range(parts):
                        gm, c = dx[p * rows:(p + 1) * rows].double(), (by[p * rows:(p + 1) * rows].double() - mean.double()) * invstd.double()
                        assert bool(((s1[p] - gm.sum(0)).abs() <= bound * gm.abs().sum(0)).all()), (addend, masked, p)
                        assert bool(((s2[p] - (gm * c).sum(0)).abs() <= bound * (gm * c).abs().sum(0)).all()), (addend, masked, p)
