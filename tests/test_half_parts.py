"""Operands in two fp16 parts (split_mfma.h): what their scales, taken from samples, do not fit is computed again in fp32, image by
image and kernel by kernel.  Outputs keep the error bound of a sum in fp32 beside what parts may lose of the largest of the few sums of a
kernel that are judged together; the tests say which bound they hold outputs to."""
import ctypes

import numpy as np
import pytest

from oracle.conv_oracle import conv_ref
from paper_2012_15667_amd.inputs import make_inputs
from tests import plan_host
from tests.test_split_kernels import _bound, gpu  # noqa: F401

pytestmark = pytest.mark.gpu

# (These four run in three bf16 parts, which hold every value: the same data through the other kind of parts.  Layers in two parts: TWO_PARTS.)
# N, C, H, W, K, R, stride, pad: whole images in a block, parts of one, a window of one row and of one pixel, chunks of 16 and 32
LAYERS = [(6, 48, 7, 7, 40, 3, 1, 1), (3, 72, 30, 31, 64, 3, 1, 1), (5, 64, 16, 15, 130, 3, 2, 1), (2, 40, 40, 40, 24, 5, 1, 2)]


def _images_apart(x, w):
    """A scale per image, over 2^80; zeros in the first one."""
    for i in range(x.shape[0]):
        x[i] *= np.float32(2.0) ** ((i * 37) % 80 - 50)
    x[0] = 0


def _dark_corner(x, w):
    """Pixels far below the rest of their image: sums of them alone; one of them not zero at all, one channel of it not tiny."""
    x[:, :, :5, :5] *= np.float32(1e-6)
    x[:, :, 6:, :2] *= np.float32(1e-12)
    x[:, 1:, 1, 1] = 0
    x[-1, 3, 2, 2] = 1


def _outliers(x, w):
    """Single values far above the sample, of inputs and of kernels."""
    x[:, x.shape[1] // 2, -1, -1] = 3e5
    x[-1, -1, 2, 2] = -2e30
    w[-1, -1, 0, 0] = 1e7


def _tiny_kernels(x, w):
    """Kernels far below 1, one of zeros; channels of one that are far below its others, met by inputs in those channels alone: as many
    as are judged together, eight with a window, 128 without."""
    n = 8 if w.shape[2] > 1 else 128
    w[0] *= np.float32(1e-25)
    w[1] = 0
    w[2, :n] *= np.float32(1e-9)
    w[3, 1:] = 0
    x[:, n:] = 0


def _sparse(x, w):
    """Nine in ten inputs are zero, most of the others small."""
    rng = np.random.default_rng(x.size)
    x *= (rng.random(x.shape) < 0.1) * np.exp2(-12 * rng.random(x.shape)).astype(np.float32)


@pytest.mark.parametrize("layer", LAYERS)
@pytest.mark.parametrize("change", [_images_apart, _dark_corner, _outliers, _tiny_kernels, _sparse])
def test_direct_outputs_keep_the_bound_of_fp32(gpu, layer, change):  # noqa: F811
    torch, B = gpu
    N, C, H, W, K, R, stride, pad = layer
    assert B.iolb_route(B.make_shape(N, C, H, W, K, R, R, stride, pad))[0] == B.ROUTE_SPLIT
    x, w = make_inputs(N, C, H, W, K, R, R, "u11", "he", seed=C + K)
    x, w = x + np.copysign(np.float32(2.0 ** -6), x), w.copy()
    change(x, w)
    run = lambda a: B.conv_direct(torch.from_numpy(a).cuda(), torch.from_numpy(w).cuda(), stride, pad).cpu().numpy()  # noqa: E731
    y = run(x)
    assert (np.abs(y - conv_ref(x, w, stride, pad)) <= _bound(x, w, stride, pad) + 2.0 ** -149).all()
    # what another image holds does not change an image's bits
    other = x.copy()
    other[N - 1] *= np.float32(1e-20)
    assert np.array_equal(run(other)[:N - 1], y[:N - 1])


def _relative(torch, y, ref, lim):
    return float(((y.double() - ref).abs() / (lim + 2.0 ** -149)).max())


@pytest.mark.parametrize("layer", [(12, 768, 17, 17, 192, 1), (70, 515, 7, 5, 500, 1), (4, 300, 61, 61, 450, 2)])
@pytest.mark.parametrize("layout", ["chw", "hwc"])
@pytest.mark.parametrize("change", [_images_apart, _dark_corner, _outliers, _tiny_kernels, _sparse])
def test_pointwise_outputs_keep_the_bound_of_fp32(gpu, layer, layout, change):  # noqa: F811
    torch, B = gpu
    N, C, H, W, K, stride = layer
    lay = B.LAYOUT_HWC if layout == "hwc" else B.LAYOUT_CHW
    assert B.iolb_route(B.make_shape(N, C, H, W, K, 1, 1, stride, 0), lay)[0] == B.ROUTE_SPLIT
    x, w = make_inputs(N, C, H, W, K, 1, 1, "u11", "he", seed=C + K)
    x, w = x + np.copysign(np.float32(2.0 ** -6), x), w.copy()
    change(x, w)
    wd = torch.from_numpy(w).cuda()

    def run(a):
        a = torch.from_numpy(a).cuda()
        if layout == "chw":
            return B.conv_direct(a, wd, stride, 0)
        return B.conv_direct_layout(a.permute(0, 2, 3, 1).contiguous(), wd, stride, 0, lay).permute(0, 3, 1, 2)

    y = run(x)
    xs = torch.from_numpy(x).cuda()[:, :, ::stride, ::stride].double().flatten(2).contiguous()
    wk = wd.double().view(1, K, C).expand(N, K, C).contiguous()
    lim = (12 * -(-C // 8) + 16) * 2.0 ** -23 * torch.bmm(wk.abs(), xs.abs())
    assert _relative(torch, y.flatten(2), torch.bmm(wk, xs), lim) <= 1
    other = x.copy()
    other[N - 1] *= np.float32(1e-20)
    assert torch.equal(run(other)[:N - 1], y[:N - 1])


# products of their own between the transforms, every m
@pytest.mark.parametrize("m,N,C,H,W,K", [(2, 64, 512, 7, 7, 512), (3, 33, 525, 7, 8, 485), (4, 9, 277, 35, 37, 233), (6, 5, 284, 29, 30, 497),
                                          (2, 5, 365, 33, 34, 227), (4, 5, 365, 33, 35, 227)])
def test_winograd_product_with_kernels_the_scales_do_not_fit(gpu, m, N, C, H, W, K):  # noqa: F811
    """Images and kernels of very different scale, channels of one kernel far below its others, an outlier: from w and from kernels
    transformed before, within the guard of each image and kernel by itself."""
    torch, B = gpu
    from tests.test_split_kernels import GUARD_WINO, _winograd_ref
    assert B.iolb_route(B.make_shape(N, C, H, W, K, algo=B.WINO_ALGO[m]))[0] == B.ROUTE_SPLIT
    x, w = make_inputs(N, C, H, W, K, 3, 3, "u11", "he", seed=m + C)
    x, w = x.copy(), w.copy()
    x[1] *= np.float32(1e-9)
    x[2] *= np.float32(1e12)
    x[3, :, 1, 1] *= np.float32(1e4)
    w[1] *= np.float32(1e-20)
    w[2] *= np.float32(1e15)
    w[3, :64] *= np.float32(1e-8)
    w[4] = 0
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    ref, U = _winograd_ref(torch, xd, wd, 1), B.winograd_transform_kernels(wd, m)[0]
    for y in (B.conv_winograd(xd, wd, m), B.conv_winograd_pre(xd, U, K, m)):
        for i in range(5):
            for k in range(6):
                r = ref[i, k].cpu().numpy()
                assert np.abs(y[i, k].cpu().numpy() - r).max() <= GUARD_WINO[m] * max(np.sqrt(np.mean(r * r)), 1e-300), (i, k)


# one kernel, both tiles and blocks, columns read in every way; 64 channels and more, a batch of small images in a block
@pytest.mark.parametrize("m,N,C,H,W,K,pad", [(2, 8, 128, 56, 56, 128, 1), (2, 6, 182, 125, 125, 102, 1), (2, 30, 128, 40, 41, 128, 3), (4, 16, 100, 64, 64, 64, 1),
                                             (4, 64, 256, 14, 14, 256, 1), (4, 8, 80, 126, 126, 144, 1), (4, 64, 128, 15, 14, 96, 1), (4, 20, 64, 100, 99, 17, 2)])
def test_fused_winograd_with_values_the_scales_do_not_fit(gpu, m, N, C, H, W, K, pad):  # noqa: F811
    torch, B = gpu
    from tests.test_split_kernels import GUARD_WINO, _runs_fused, _winograd_ref
    x, w = make_inputs(N, C, H, W, K, 3, 3, "u11", "he", seed=m + C)
    x, w = x.copy(), w.copy()
    x[1] *= np.float32(1e-9)
    x[2] *= np.float32(1e12)
    x[3, :, 1, 1] *= np.float32(1e4)
    x[4, :, :8, :8] *= np.float32(1e-7)
    w[1] *= np.float32(1e-20)
    w[2] *= np.float32(1e15)
    w[3, :64] *= np.float32(1e-8)
    w[4] = 0
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    ref = _winograd_ref(torch, xd, wd, pad)
    y = _runs_fused(B, lambda: B.conv_winograd(xd, wd, m, pad=pad))
    for i in range(5):
        for k in range(6):
            r = ref[i, k].cpu().numpy()
            assert np.abs(y[i, k].cpu().numpy() - r).max() <= GUARD_WINO[m] * max(np.sqrt(np.mean(r * r)), 1e-300), (i, k)
    # the dark corner by itself
    e = 8 - m - 2 + pad
    r = ref[4, 0, :e, :e].cpu().numpy()
    assert np.abs(y[4, 0, :e, :e].cpu().numpy() - r).max() <= 8 * GUARD_WINO[m] * np.sqrt(np.mean(r * r))
    # an image's bits do not depend on what another one holds
    other = xd.clone()
    other[N - 1] *= 1e-20
    assert torch.equal(_runs_fused(B, lambda: B.conv_winograd(other, wd, m, pad=pad))[:N - 1], y[:N - 1])


@pytest.mark.parametrize("layer", [(3, 16, 9, 8, 5, 1), (2, 17, 13, 11, 33, 2), (1, 21, 40, 41, 70, 1), (4, 40, 23, 23, 257, 1), (5, 151, 1, 30, 64, 1), (2, 64, 30, 31, 48, 3)])
def test_small_pointwise_layers_with_channels_innermost(gpu, layer):  # noqa: F811
    """From 16 channels on, whatever their size: fewer channels than a chunk, fewer pixels and kernels than a block, strides."""
    torch, B = gpu
    N, C, H, W, K, stride = layer
    shape = B.make_shape(N, C, H, W, K, 1, 1, stride, 0)
    assert B.iolb_route(shape, B.LAYOUT_HWC)[0] == B.ROUTE_SPLIT
    x, w = make_inputs(N, C, H, W, K, 1, 1, "u11", "he", seed=C + K)
    xh = np.ascontiguousarray(x.transpose(0, 2, 3, 1))
    wd = torch.from_numpy(w).cuda()
    y = B.conv_direct_layout(torch.from_numpy(xh).cuda(), wd, stride, 0, B.LAYOUT_HWC).cpu().numpy().transpose(0, 3, 1, 2)
    assert (np.abs(y - conv_ref(x, w, stride, 0)) <= _bound(x, w, stride, 0)).all()
    # inputs and outputs off 16 bytes
    buf = torch.zeros(xh.size + 1, device="cuda")
    xo = buf[1:].view(xh.shape)
    xo.copy_(torch.from_numpy(xh))
    out = torch.full((y.size + 2,), 7.0, device="cuda")
    P, Q = y.shape[2:]
    yo = out[1:-1].view(N, P, Q, K)
    B.conv_direct_layout(xo, wd, stride, 0, B.LAYOUT_HWC, y=yo)
    assert np.array_equal(yo.cpu().numpy().transpose(0, 3, 1, 2), y) and float(out[0]) == 7 and float(out[-1]) == 7


# ---- operands of one sum that differ in size ------------------------------------------------------
# What a kernel's parts and a pixel's cannot hold beside a larger operand may be all of an output, where that operand meets a small or a
# zero partner.  The groups do not follow those that the kernels judge together: single channels, parts of eight, the last ones.
def _identity(x, w):
    w[:] = 0
    for k in range(w.shape[0]):
        w[k, k % w.shape[1], w.shape[2] // 2, w.shape[3] // 2] = 1
    x *= np.float32(2.0) ** -(np.arange(x.shape[1]) % 64)[None, :, None, None].astype(np.float32)


def _balanced(r):
    def change(x, w):
        x[:, 3] *= np.float32(r)
        w[:, 3] /= np.float32(r)
    return change


def _pruned(s):
    def change(x, w):
        w[:, 0] = 0
        x[:, 1:] *= np.float32(s)
    return change


def _some_small_kernels(n):
    def change(x, w):
        m = min(n, w.shape[1] - 1)
        w[2::3, :m] *= np.float32(1e-8)
        x[:, m:] = 0
    return change


def _last_channels(x, w):
    n = w.shape[1] % 16 or 3
    w[::2, -n:] *= np.float32(1e-9)
    x[:, :-n] = 0


def _halves(x, w):
    w[:, ::2] *= np.float32(1e-8)
    x[:, 1::2] *= np.float32(1e-8)


def _beside_outliers(x, w):
    """Beside pixels whose sums are not finite, or computed again for a reason of their own."""
    _halves(x, w)
    x[:, 0, ::4, ::3] *= np.float32(1e6)
    x[0, 2, -1, -1] = np.float32(3e30)


def _one_image_of_it(x, w):
    """In one image of the batch only, the others as they are: they do not speak for it."""
    w[:, 0] = 0
    x[1, 1:] *= np.float32(1e-9)


APART = {"identity": _identity, "balanced_1e3": _balanced(1e3), "balanced_1e5": _balanced(1e5), "balanced_1e7": _balanced(1e7), "balanced_1e9": _balanced(1e9),
         "pruned_1e-8": _pruned(1e-8), "pruned_1e-12": _pruned(1e-12), "small_1": _some_small_kernels(1), "small_4": _some_small_kernels(4),
         "small_7": _some_small_kernels(7), "small_100": _some_small_kernels(100), "last": _last_channels, "halves": _halves,
         "beside_outliers": _beside_outliers, "one_image": _one_image_of_it}


def _conv64(torch, xd, wd, stride, pad):
    """The layer in 64 bits, [N][K][P Q]."""
    (N, C, H, W), (K, _, R, S) = xd.shape, wd.shape
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    xp = torch.nn.functional.pad(xd.double(), (pad,) * 4)
    y = torch.zeros(N, K, P * Q, dtype=torch.float64, device="cuda")
    for r in range(R):
        for s in range(S):
            win = xp[:, :, r:r + stride * (P - 1) + 1:stride, s:s + stride * (Q - 1) + 1:stride].reshape(N, C, P * Q).contiguous()
            y += torch.bmm(wd[:, :, r, s].double().unsqueeze(0).expand(N, K, C).contiguous(), win)
    return y.view(N, K, P, Q)


def _each_kernel_by_itself(torch, y, xd, wd, stride, pad, each_output=False):
    """Error per image and kernel against the size of its sums (the root of the sum of squared products, which no cancellation makes
    small).  Sums of n products in fp32, a rounding of up to 2^-24 of a running sum of 0.7 of that size in the mean each, are off by some
    0.7 sqrt(n) 2^-24 of it: three times that, for images of one or six outputs, and what goes unmarked, 2^-21 of sums of up to
    twice that size; one output four times both.  A cut that is not taken again was 1e-4 and more."""
    ref, size = _conv64(torch, xd, wd, stride, pad), _conv64(torch, xd.double() ** 2, wd.double() ** 2, stride, pad).sqrt()
    err, lim = (y.double() - ref).abs(), 2.1 * wd[0].numel() ** 0.5 * 2.0 ** -24 + 2.0 ** -20
    rms = lambda a: (a * a).mean((2, 3)).sqrt()  # noqa: E731
    tiny = 2.0 ** -149
    if each_output:
        assert bool((err <= 8 * lim * size + tiny).all()), float((err / (lim * size + tiny)).max())
    assert bool((rms(err) <= lim * rms(size) + tiny).all()), float((rms(err) / (lim * rms(size) + tiny)).max())
    assert bool((err.amax((2, 3)) <= 4 * lim * size.amax((2, 3)) + tiny).all()), float((err.amax((2, 3)) / (lim * size.amax((2, 3)) + tiny)).max())


# N, C, H, W, K, R, stride, pad of layers that run in two parts (asserted): one image and several in a block, stride 2, 5 x 5, channels
# and kernels that fill no block, one pixel, every kind of workgroup they get
TWO_PARTS = [(12, 72, 30, 31, 64, 3, 1, 1), (8, 129, 28, 28, 130, 3, 2, 1), (2, 96, 27, 27, 256, 5, 1, 2), (64, 128, 4, 4, 512, 3, 1, 1),
             (200, 130, 3, 2, 257, 3, 1, 1), (2, 604, 9, 9, 600, 3, 1, 1), (20, 64, 1, 1, 32, 3, 1, 1), (20, 64, 56, 56, 64, 3, 1, 1)]


def _two_parts(N, C, H, W, K, R, stride, pad):
    block = (ctypes.c_int * 7)()
    return plan_host.lib().split_block(N, C, H, W, K, R, R, stride, pad, block) == 1 and block[0] == 2


def _in_every_layout(torch, B, xd, wd, stride, pad):
    """The layer in [N][K][P][Q], from every layout and from channels innermost off 16 bytes."""
    yield B.conv_direct(xd, wd, stride, pad)
    xh = xd.permute(0, 2, 3, 1).contiguous()
    yield B.conv_direct_layout(xh, wd, stride, pad, B.LAYOUT_HWC).permute(0, 3, 1, 2)
    off = torch.zeros(xh.numel() + 1, device="cuda")[1:].view(xh.shape)
    off.copy_(xh)
    yield B.conv_direct_layout(off, wd, stride, pad, B.LAYOUT_HWC).permute(0, 3, 1, 2)
    yield B.conv_direct_layout(xd.permute(0, 1, 3, 2).contiguous(), wd, stride, pad, B.LAYOUT_CWH).permute(0, 1, 3, 2)


@pytest.mark.parametrize("layer", TWO_PARTS)
@pytest.mark.parametrize("change", list(APART))
def test_direct_kernels_whose_operands_differ_in_size(gpu, layer, change):  # noqa: F811
    torch, B = gpu
    N, C, H, W, K, R, stride, pad = layer
    assert _two_parts(*layer) and _two_parts(N, C, W, H, K, R, stride, pad)
    x, w = (a.copy() for a in make_inputs(N, C, H, W, K, R, R, "u11", "he", seed=C + K))
    APART[change](x, w)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    for y in _in_every_layout(torch, B, xd, wd, stride, pad):
        _each_kernel_by_itself(torch, y, xd, wd, stride, pad, change == "beside_outliers")
    # what another image holds does not change an image's bits
    y = B.conv_direct(xd, wd, stride, pad)
    other = xd.clone()
    other[N - 1] *= 1e-20
    other[N - 1, 1:] = 0
    assert torch.equal(B.conv_direct(other, wd, stride, pad)[:N - 1], y[:N - 1])


@pytest.mark.parametrize("layout,layer", [(o, n) for n in [(12, 768, 17, 17, 192, 1), (70, 515, 7, 5, 500, 1), (4, 300, 61, 61, 450, 2)] for o in ("chw", "hwc")] +
                         [("hwc", (90, 256, 1, 1, 400, 1)), ("hwc", (11, 81, 3, 5, 70, 1))])
@pytest.mark.parametrize("change", list(APART))
def test_pointwise_kernels_whose_operands_differ_in_size(gpu, layer, layout, change):  # noqa: F811
    torch, B = gpu
    N, C, H, W, K, stride = layer
    lay = B.LAYOUT_HWC if layout == "hwc" else B.LAYOUT_CHW
    assert B.iolb_route(B.make_shape(N, C, H, W, K, 1, 1, stride, 0), lay)[0] == B.ROUTE_SPLIT
    x, w = (a.copy() for a in make_inputs(N, C, H, W, K, 1, 1, "u11", "he", seed=C + K))
    APART[change](x, w)
    wd = torch.from_numpy(w).cuda()

    def run(a):
        if layout == "chw":
            return B.conv_direct(a, wd, stride, 0)
        return B.conv_direct_layout(a.permute(0, 2, 3, 1).contiguous(), wd, stride, 0, lay).permute(0, 3, 1, 2)

    xd = torch.from_numpy(x).cuda()
    y = run(xd)
    _each_kernel_by_itself(torch, y, xd, wd, stride, 0, change == "beside_outliers")
    other = xd.clone()
    other[N - 1] *= 1e-20
    other[N - 1, 1:] = 0
    assert torch.equal(run(other)[:N - 1], y[:N - 1])


# root mean square per image and kernel, of the kernel's outputs in that image (of 4 x 4 outputs and more): a fifth of the guards of single outputs
# (GUARD_WINO); a cut that is not taken again was 1e-3 and more
WINO_EACH = {2: 1e-5, 3: 6e-5, 4: 1e-4, 6: 1.2e-4}


def _winograd_each(torch, B, run, xd, wd, m, pad):
    from tests.test_split_kernels import _winograd_ref
    ref = _winograd_ref(torch, xd, wd, pad)
    rms = lambda a: (a * a).mean((2, 3)).sqrt()  # noqa: E731
    y = run(xd)
    err = rms(y.double() - ref)
    assert bool((err <= WINO_EACH[m] * rms(ref) + 2.0 ** -149).all()), float((err / (rms(ref) + 2.0 ** -149)).max())
    other, n = xd.clone(), xd.shape[0] - 1
    other[n] *= 1e-20
    other[n, 1:] = 0
    assert torch.equal(run(other)[:n], y[:n])


@pytest.mark.parametrize("m,N,C,H,W,K", [(2, 64, 512, 7, 7, 512), (3, 33, 525, 7, 8, 485), (4, 9, 277, 35, 37, 233), (6, 5, 284, 29, 30, 497),
                                          (4, 128, 512, 5, 5, 512), (6, 100, 512, 4, 4, 512), (2, 96, 516, 13, 13, 516),
                                          (6, 11, 272, 8, 7, 128), (2, 40, 272, 4, 5, 64)])
@pytest.mark.parametrize("change", list(APART))
def test_winograd_product_kernels_whose_operands_differ_in_size(gpu, m, N, C, H, W, K, change):  # noqa: F811
    torch, B = gpu
    assert B.iolb_route(B.make_shape(N, C, H, W, K, algo=B.WINO_ALGO[m]))[0] == B.ROUTE_SPLIT
    x, w = (a.copy() for a in make_inputs(N, C, H, W, K, 3, 3, "u11", "he", seed=m + C))
    APART[change](x, w)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    U = B.winograd_transform_kernels(wd, m)[0]
    _winograd_each(torch, B, lambda a: B.conv_winograd(a, wd, m), xd, wd, m, 1)
    _winograd_each(torch, B, lambda a: B.conv_winograd_pre(a, U, K, m), xd, wd, m, 1)


@pytest.mark.parametrize("m,N,C,H,W,K", [(4, 16, 100, 64, 64, 64), (2, 8, 130, 56, 56, 128)])
def test_fused_winograd_blocks_taken_again_read_the_callers_kernels(gpu, m, N, C, H, W, K):  # noqa: F811
    """A corner too small for its image's scale has its blocks taken again; its sums are of the last channels alone, whose weights the parts
    have lost beside those of the other channels."""
    torch, B = gpu
    from tests.test_split_kernels import _runs_fused, _winograd_ref
    x, w = (a.copy() for a in make_inputs(N, C, H, W, K, 3, 3, "u11", "he", seed=m))
    n = C % 16
    x[:, :, :9, :9] *= np.float32(1e-7)
    x[:, :-n, :9, :9] = 0
    w[::2, -n:] *= np.float32(1e-9)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    ref = _winograd_ref(torch, xd, wd, 1)[:, :, :4, :4]
    U = B.winograd_transform_kernels(wd, m)[0]
    for y in (_runs_fused(B, lambda: B.conv_winograd(xd, wd, m)), _runs_fused(B, lambda: B.conv_winograd_pre(xd, U, K, m))):
        err = (y[:, :, :4, :4].double() - ref).abs().amax((2, 3))
        assert bool((err <= 8 * WINO_EACH[m] * ref.abs().amax((2, 3))).all()), float((err / ref.abs().amax((2, 3))).max())


@pytest.mark.parametrize("m,N,C,H,W,K,pad", [(2, 8, 128, 56, 56, 128, 1), (2, 6, 182, 125, 125, 102, 1), (4, 16, 100, 64, 64, 64, 1), (4, 64, 256, 14, 14, 256, 1),
                                             (4, 64, 128, 15, 14, 96, 1), (4, 20, 68, 100, 99, 17, 2)])
@pytest.mark.parametrize("change", list(APART) + ["last_and_nan"])
def test_fused_winograd_kernels_whose_operands_differ_in_size(gpu, m, N, C, H, W, K, pad, change):  # noqa: F811
    torch, B = gpu
    from tests.test_split_kernels import _runs_fused
    x, w = (a.copy() for a in make_inputs(N, C, H, W, K, 3, 3, "u11", "he", seed=m + C))
    nan = change == "last_and_nan"                            # blocks that are taken again whatever these kernels hold
    APART["last" if nan else change](x, w)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    U = B.winograd_transform_kernels(wd, m)[0]
    for pre in (False, True) if pad == 1 else (False,):
        def run(a):
            if nan:
                a, k = a.clone(), wd.clone()
                k[0] = float("nan")
                V = B.winograd_transform_kernels(k, m)[0]
            else:
                k, V = wd, U
            y = _runs_fused(B, lambda: B.conv_winograd_pre(a, V, K, m) if pre else B.conv_winograd(a, k, m, pad=pad))
            if nan:
                assert bool(torch.isnan(y[:, 0]).all())
                y[:, 0] = B.conv_direct(a, wd[:1].contiguous(), 1, pad)[:, 0]
            return y
        _winograd_each(torch, B, run, xd, wd, m, pad)
