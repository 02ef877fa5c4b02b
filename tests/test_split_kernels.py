"""The kernels that take fp32 products as bf16 products of parts (direct_split.hip, split_point.hip): edges of their
blocks, remainders, layouts, values whose parts do not fit bf16, and the layers' other entry points."""
import numpy as np
import pytest

from oracle.conv_oracle import conv_ref, conv_ref_cwh, conv_ref_hwc
from paper_2012_15667_amd.inputs import make_inputs
from tests.conftest import rel_err

pytestmark = pytest.mark.gpu

GUARD_WINO = {2: 5e-5, 3: 3e-4, 4: 5e-4, 6: 6e-4}          # as in test_gpu_parity.py


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (run with -m 'not gpu' on a CPU box)")
    from paper_2012_15667_amd import binding
    binding.lib()
    return torch, binding


def _bound(x, w, stride, pad, ref_of=conv_ref):
    """Largest error of a sum of products taken in three bf16 parts, per output: a running sum is rounded six times per
    step of four (tap, eight channels) units and every rounding, inside the instruction too, is at most 2^-23 of the sum
    of magnitudes so far (twice 2^-24: truncation is allowed for); the products left out add 3 * 2^-24.  Layers in two fp16 parts round half as often
    (three products a step) and lose 2^-21 of each product at most, 4 of the 16 units that stand beside the steps here: the bound holds
    for them with half to spare."""
    C, RS = w.shape[1], w.shape[2] * w.shape[3]
    steps = -(-C // 8) * RS
    return (12 * steps + 16) * 2.0 ** -23 * ref_of(np.abs(x), np.abs(w), stride, pad)


CASES = [
    # N, C, H, W, K, R, S, stride, pad
    (1, 9, 7, 7, 1, 3, 3, 1, 1),            # second channel group nearly empty, one kernel
    (2, 16, 9, 8, 15, 3, 3, 1, 1),          # exactly one chunk of 16: a single LDS buffer
    (2, 17, 12, 11, 17, 3, 3, 1, 1),        # one channel and one kernel over a block
    (1, 33, 9, 10, 130, 3, 3, 1, 0),        # chunk of 32 and one channel; K over 128
    (3, 40, 14, 14, 64, 3, 3, 1, 1),        # whole images in a block, several images
    (5, 48, 7, 7, 96, 3, 3, 1, 1),          # batch not a multiple of the images per block
    (2, 31, 23, 29, 24, 3, 3, 2, 1),        # stride 2: residue classes of odd width
    (1, 20, 31, 30, 40, 2, 2, 3, 0),        # stride beyond the kernel: rows and columns nobody uses
    (2, 24, 17, 17, 32, 1, 7, 1, 0),        # one-sided kernels (no padding here)
    (2, 24, 17, 17, 32, 7, 1, 1, 0),
    (20, 64, 1, 1, 32, 3, 3, 1, 1),         # a single pixel per image
    (2, 12, 35, 20, 20, 5, 5, 1, 2),
    (2, 3, 51, 47, 30, 11, 11, 4, 0),       # three channels: products summed apart per step
    (1, 5, 30, 30, 64, 7, 7, 2, 3),
    (2, 8, 19, 19, 33, 5, 5, 1, 2),
]
# fewer than 16 pixels in all: no block of the split kernel is half full, the tuned tile stays
FEW_PIXELS = [(1, 33, 5, 6, 130, 3, 3, 1, 0), (2, 64, 1, 1, 32, 3, 3, 1, 1)]


@pytest.mark.parametrize("case", CASES + FEW_PIXELS)
def test_split_direct_layouts_within_the_bound(gpu, case):
    torch, B = gpu
    N, C, H, W, K, R, S, stride, pad = case
    for layout in (B.LAYOUT_CHW, B.LAYOUT_HWC, B.LAYOUT_CWH):
        assert B.iolb_route(B.make_shape(*case), layout)[0] == (B.ROUTE_TILE if case in FEW_PIXELS else B.ROUTE_SPLIT)
    x, w = make_inputs(N, C, H, W, K, R, S, "u11", "he", seed=sum(case))
    ref, lim = conv_ref(x, w, stride, pad), _bound(x, w, stride, pad)
    wd = torch.from_numpy(w).cuda()
    y = B.conv_direct(torch.from_numpy(x).cuda(), wd, stride, pad).cpu().numpy()
    assert (np.abs(y - ref) <= lim).all()
    # channels innermost: the same sums in the same order
    xh = np.ascontiguousarray(x.transpose(0, 2, 3, 1))
    yh = B.conv_direct_layout(torch.from_numpy(xh).cuda(), wd, stride, pad, B.LAYOUT_HWC).cpu().numpy()
    assert np.array_equal(yh, y.transpose(0, 2, 3, 1))
    # the transposed image: the taps in another order
    xt = np.ascontiguousarray(x.transpose(0, 1, 3, 2))
    yt = B.conv_direct_layout(torch.from_numpy(xt).cuda(), wd, stride, pad, B.LAYOUT_CWH).cpu().numpy()
    assert (np.abs(yt - conv_ref_cwh(xt, w, stride, pad)) <= lim.transpose(0, 1, 3, 2)).all()


@pytest.mark.parametrize("taps", [(1, 2), (1, 15), (4, 4), (1, 17), (5, 5), (4, 8), (3, 11), (7, 9), (1, 65)])
@pytest.mark.parametrize("C,K", [(3, 16), (9, 17), (17, 5), (40, 130)])
def test_kernels_reach_their_steps_for_every_window(gpu, taps, C, K):
    """Kernels go to the matrix steps in slices of 16 taps, and the first steps of the input tile are loaded ahead:
    windows around the slices' edges, channels and kernels beyond a block's, whole numbers (every sum is exact)."""
    torch, B = gpu
    R, S = taps
    case = (3, C, R + 8, S + 12, K, R, S, 1, 0)
    if C > 8 or R * S >= 25:
        assert B.iolb_route(B.make_shape(*case), B.LAYOUT_CHW)[0] == B.ROUTE_SPLIT
    rng = np.random.default_rng(R * 100 + S + C)
    x = rng.integers(-4, 5, (3, C, R + 8, S + 12)).astype(np.float32)
    w = rng.integers(-4, 5, (K, C, R, S)).astype(np.float32)
    y = B.conv_direct(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 0).cpu().numpy()
    assert np.array_equal(y, conv_ref(x, w, 1, 0))
    xt = np.ascontiguousarray(x.transpose(0, 1, 3, 2))
    yt = B.conv_direct_layout(torch.from_numpy(xt).cuda(), torch.from_numpy(w).cuda(), 1, 0, B.LAYOUT_CWH).cpu().numpy()
    assert np.array_equal(yt, y.transpose(0, 1, 3, 2))


# N, C, H, W, K, R, S, stride, pad of layers whose workgroups prepare their own kernels, up to 6144 values each: few and many
# channels and workgroups, kernels beyond the last block ...
OWN_LAYERS = [
    (3, 32, 15, 15, 32, 3, 3, 1, 1), (2, 30, 14, 15, 17, 3, 3, 2, 1), (3, 9, 12, 13, 100, 4, 4, 1, 2), (40, 16, 14, 14, 16, 3, 3, 1, 1),
    (400, 16, 14, 14, 16, 3, 3, 1, 1), (7, 16, 114, 114, 16, 3, 3, 1, 1), (2, 3, 100, 100, 16, 5, 5, 1, 1), (2, 5, 100, 100, 15, 6, 6, 1, 1),
    (7, 21, 9, 9, 306, 3, 1, 1, 0),
]
# ... and of layers beyond that, in values or in workgroups
NOT_OWN_LAYERS = [
    (1, 34, 15, 15, 32, 3, 3, 1, 1), (2, 3, 60, 60, 7, 7, 7, 2, 3), (6, 3, 148, 148, 48, 7, 7, 2, 3), (2, 48, 13, 13, 16, 3, 3, 1, 1),
    (64, 16, 114, 114, 16, 3, 3, 1, 1),
]
MANY_BLOCKS = (4352, 9, 14, 14, 512, 3, 3, 1, 1)


@pytest.mark.parametrize("case", OWN_LAYERS + NOT_OWN_LAYERS[:4])
def test_small_layers_prepare_their_own_kernels(gpu, case):
    """Workgroups of small layers prepare their own kernels (which do: a test of the planner, by the same lists): within the bound,
    with an infinite input and a weight beyond the parts' range, and replayed in a graph."""
    torch, B = gpu
    N, C, H, W, K, R, S, stride, pad = case
    x, w = make_inputs(N, C, H, W, K, R, S, "u11", "he", seed=sum(case))
    ref, lim = conv_ref(x, w, stride, pad), _bound(x, w, stride, pad)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    y = B.conv_direct(xd, wd, stride, pad)
    assert (np.abs(y.cpu().numpy() - ref) <= lim).all()
    x[0, C - 1, H // 2, W // 2] = np.inf
    w[K - 1, 0, 0, 0] = -1e35
    ref = conv_ref(x, w, stride, pad)
    xi, wi = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    z = B.conv_direct(xi, wi, stride, pad).cpu().numpy()
    fine = np.isfinite(ref)
    assert np.array_equal(np.isnan(z), np.isnan(ref)) and np.array_equal(z[~fine], ref[~fine], equal_nan=True)
    assert (np.abs(z[fine] - ref[fine]) <= _bound(np.where(np.isfinite(x), x, 0), w, stride, pad)[fine]).all()
    out = torch.empty_like(y)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        B.conv_direct(xd, wd, stride, pad, y=out)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, y)


def test_more_blocks_than_ids_divided_by_multiplication(gpu):
    """Beyond 32768 workgroups (34816 here, of 112 pixels by 128 kernels) their ids are divided as integers; parts of the batch
    stay below.  Whole numbers: every sum is exact, whatever the block."""
    torch, B = gpu
    N, C, H, W, K, R, S, stride, pad = MANY_BLOCKS
    x = torch.randint(-4, 5, (N, C, H, W), device="cuda", dtype=torch.float32)
    w = torch.randint(-4, 5, (K, C, R, S), device="cuda", dtype=torch.float32)
    y = B.conv_direct(x, w, stride, pad)
    for i in range(0, N, 1088):
        assert torch.equal(y[i:i + 1088], B.conv_direct(x[i:i + 1088].contiguous(), w, 1, 1))


@pytest.mark.parametrize("layer", [(4, 24, 18, 18, 40, 3, 1), (4, 3, 24, 24, 40, 7, 3), (12, 768, 17, 17, 192, 1, 0)])
def test_single_products_have_fp32_precision(gpu, layer):
    """One channel and one tap are not zero, so that every output is one product x w of full 24-bit operands.  Of its nine
    products of parts three are left out: m l and l m, each at most 2^-8 2^-16 of it, and l l: 2^-23.  The other six are
    added in five roundings of at most 2^-23 of the sum (truncation allowed for); the partial sums exceed the product by
    no more than 2^-7 of it.  A product left out beside these, h l, l h or m m, breaks it (computed on the CPU with such a
    split: 0.12 of the bound with the six, 10 to 19 times the bound without one of those).  The third layer runs in two fp16
    parts: each operand is held to 2^-23 of it, l l, at most 2^-22, is left out, and the sum is rounded once beside what is far smaller: 4.5 of
    the six 2^-23; 0.8 * 2^-24 in the mean."""
    torch, B = gpu
    N, C, H, W, K, R, pad = layer
    assert B.iolb_route(B.make_shape(N, C, H, W, K, R, R, 1, pad))[0] == B.ROUTE_SPLIT
    g = torch.Generator(device="cuda").manual_seed(C)
    x = torch.zeros((N, C, H, W), device="cuda")
    w = torch.zeros((K, C, R, R), device="cuda")
    x[:, C - 1] = (torch.rand((N, H, W), generator=g, device="cuda") + 1) * torch.where(torch.rand((N, H, W), generator=g, device="cuda") < 0.5, -1.0, 1.0)
    w[:, C - 1, R // 2, R // 2] = torch.rand(K, generator=g, device="cuda") + 1
    exact = x[:, C - 1].double()[:, None] * w[:, C - 1, R // 2, R // 2].double()[None, :, None, None]
    err = ((B.conv_direct(x, w, 1, pad).double() - exact) / exact).abs()
    assert float(err.max()) <= 2.0 ** -23 * (1 + 5 * (1 + 2.0 ** -7)) and float(err.mean()) <= 2.0 ** -24


@pytest.mark.parametrize("offset", [1, 2, 3])
def test_split_direct_takes_tensors_off_16_byte_boundaries(gpu, offset):
    torch, B = gpu
    x, w = make_inputs(2, 20, 9, 10, 24, 3, 3, "u11", "he", seed=offset)
    xh = np.ascontiguousarray(x.transpose(0, 2, 3, 1))
    buf = torch.zeros(xh.size + 4, device="cuda")
    xd = buf[offset:offset + xh.size].view(xh.shape)
    xd.copy_(torch.from_numpy(xh))
    out = torch.full((2 * 9 * 10 * 24 + 8,), 7.0, device="cuda")
    yd = out[offset:offset + 2 * 9 * 10 * 24].view(2, 9, 10, 24)
    B.conv_direct_layout(xd, torch.from_numpy(w).cuda(), 1, 1, B.LAYOUT_HWC, y=yd)
    ref = conv_ref_hwc(xh, w, 1, 1)
    assert (np.abs(yd.cpu().numpy() - ref) <= _bound(xh, w, 1, 1, conv_ref_hwc)).all()
    flat = out.cpu().numpy()
    assert (flat[:offset] == 7).all() and (flat[offset + 2 * 9 * 10 * 24:] == 7).all()


# large enough for the split 1 x 1 kernel (at least 160 channels, 1 GFLOP, 48 flop per byte)
POINT_CASES = [
    # N, C, H, W, K, stride, layout
    (12, 768, 17, 17, 192, 1, "chw"),       # 289 pixels: blocks that end inside an image, pairs over its end
    (2, 161, 64, 65, 400, 1, "chw"),        # ragged channels, K not a multiple of a block
    (60, 515, 6, 6, 500, 1, "chw"),         # blocks over several images
    (70, 515, 7, 5, 500, 1, "chw"),         # the same with an odd number of pixels
    (4, 300, 61, 61, 450, 2, "chw"),        # stride 2: single pixels
    (12, 768, 17, 17, 192, 1, "hwc"),
    (12, 770, 17, 17, 191, 1, "hwc"),       # no vector loads or stores
    (4, 300, 61, 61, 452, 2, "hwc"),
]


@pytest.mark.parametrize("case", POINT_CASES)
def test_split_pointwise_within_the_bound(gpu, case):
    torch, B = gpu
    N, C, H, W, K, stride, layout = case
    assert B.iolb_route(B.make_shape(N, C, H, W, K, 1, 1, stride, 0), B.LAYOUT_HWC if layout == "hwc" else B.LAYOUT_CHW)[0] == B.ROUTE_SPLIT
    x, w = make_inputs(N, C, H, W, K, 1, 1, "u11", "he", seed=N + C)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    xs = xd[:, :, ::stride, ::stride].double().flatten(2).contiguous()
    wk = wd.double().view(1, K, C).expand(N, K, C).contiguous()
    P, Q = (H - 1) // stride + 1, (W - 1) // stride + 1
    ref = torch.bmm(wk, xs).view(N, K, P, Q)
    lim = (12 * -(-C // 8) + 16) * 2.0 ** -23 * torch.bmm(wk.abs(), xs.abs()).view(N, K, P, Q)
    if layout == "chw":
        y = B.conv_direct(xd, wd, stride, 0)
    else:
        y = B.conv_direct_layout(xd.permute(0, 2, 3, 1).contiguous(), wd, stride, 0, B.LAYOUT_HWC).permute(0, 3, 1, 2)
    assert bool(((y.double() - ref).abs() <= lim).all())


@pytest.mark.parametrize("shape", [(2, 24, 12, 13, 20, 3, 1), (2, 3, 40, 40, 16, 11, 0), (12, 768, 17, 17, 192, 1, 0)])
def test_values_whose_parts_are_not_finite_bf16(gpu, shape):
    """Infinities and NaN spread as in plain fp32 sums (0 * inf only where an operand is 0); finite values that round
    to an infinite bf16 and very small sums keep fp32 precision."""
    torch, B = gpu
    N, C, H, W, K, R, pad = shape
    assert B.iolb_route(B.make_shape(N, C, H, W, K, R, R, 1 if R < 11 else 4, pad))[0] == B.ROUTE_SPLIT
    x, w = make_inputs(N, C, H, W, K, R, R, "u11", "he", seed=5)
    w[np.abs(w) < 1e-3] = 1e-3
    x[np.abs(x) < 1e-3] = 1e-3
    wd = torch.from_numpy(w).cuda()
    run = lambda a: B.conv_direct(torch.from_numpy(a).cuda(), wd, 1 if R < 11 else 4, pad).cpu().numpy()
    cpu = lambda a: torch.nn.functional.conv2d(torch.from_numpy(a).double(), torch.from_numpy(w).double(), stride=1 if R < 11 else 4, padding=pad).numpy()
    a = x.copy()
    a[0, 1, 3, 4], a[0, 2, 3, 5], a[N - 1, 0, H - 1, W - 1] = np.inf, -np.inf, np.nan
    got, ref = run(a), cpu(a)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert (np.sign(got[np.isinf(ref)]) == np.sign(ref[np.isinf(ref)])).all()
    ok = np.isfinite(ref)
    assert ok.any() and rel_err(got[ok], ref[ok]) <= 3e-5
    a = x.copy()
    a[0, 0, :2, :2] = 3.4e38                                # above the largest bf16
    w[:] *= 1e-3
    wd = torch.from_numpy(w).cuda()
    got, ref = run(a), cpu(a)
    assert np.isfinite(ref).all() and np.abs(ref).max() < 3e38
    assert np.array_equal(np.isfinite(got), np.isfinite(ref.astype(np.float32)))
    assert rel_err(got, ref) <= 3e-5
    a = (x * np.float32(1e-31)).astype(np.float32)
    got, ref = run(a), cpu(a)
    assert rel_err(got, ref) <= 3e-5


# (operand scales of x and w): each operand near or below the smallest normal number against a large partner, both ways;
# denormal operands; denormal results; operands and sums beyond what the scaled parts hold (2^105, 2^82)
SCALES = [(1e-38, 1e30), (1e30, 1e-38), (1e-41, 1e25), (1e25, 1e-41), (1e-30, 1e-11), (1e33, 1e-10), (1e-10, 1e33), (1e15, 1e12)]


@pytest.mark.parametrize("scales", SCALES)
@pytest.mark.parametrize("shape", [(2, 24, 12, 13, 20, 3, 1, 1), (2, 3, 40, 40, 16, 11, 4, 0), (12, 768, 17, 17, 192, 1, 1, 0)])
def test_operands_over_the_whole_range_keep_fp32_precision(gpu, shape, scales):
    torch, B = gpu
    N, C, H, W, K, R, stride, pad = shape
    assert B.iolb_route(B.make_shape(N, C, H, W, K, R, R, stride, pad))[0] == B.ROUTE_SPLIT
    x, w = make_inputs(N, C, H, W, K, R, R, "u11", "he", seed=31)
    x, w = x * np.float32(scales[0]), w * np.float32(scales[1])
    y = B.conv_direct(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), stride, pad).cpu().numpy()
    # results below the smallest normal number are multiples of 2^-149: one rounding
    assert (np.abs(y - conv_ref(x, w, stride, pad)) <= _bound(x, w, stride, pad) + 2.0 ** -149).all()


@pytest.mark.parametrize("scales", [(1e-38, 1e30), (1e30, 1e-38), (1e33, 1e-10), (1e-10, 1e33)])
def test_winograd_product_over_the_whole_range(gpu, scales):
    torch, B = gpu
    N, C, H, W, K = 64, 512, 7, 7, 512
    assert B.iolb_route(B.make_shape(N, C, H, W, K, algo=B.WINO_F2))[0] == B.ROUTE_SPLIT
    x, w = make_inputs(N, C, H, W, K, 3, 3, "u11", "he", seed=32)
    x, w = x * np.float32(scales[0]), w * np.float32(scales[1])
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    # the fp32 product of the tuned tile, asked for by name
    tile = B.iolb_tune(B.make_shape(N, C, H, W, K, algo=B.WINO_F2))
    ref = B.conv_winograd(xd, wd, 2, cfg=tile).cpu().numpy()
    assert rel_err(B.conv_winograd(xd, wd, 2).cpu().numpy(), ref) <= GUARD_WINO[2]
    U = B.winograd_transform_kernels(wd, 2)[0]
    assert rel_err(B.conv_winograd_pre(xd, U, K, 2).cpu().numpy(), ref) <= GUARD_WINO[2]


@pytest.mark.parametrize("case", CASES)
def test_sums_taken_again_in_every_shape_and_layout(gpu, case):
    """Operands beyond what the parts hold: every output comes from the second, plain fp32, pass over its block."""
    torch, B = gpu
    N, C, H, W, K, R, S, stride, pad = case
    x, w = make_inputs(N, C, H, W, K, R, S, "u11", "he", seed=sum(case) + 1)
    x = (x + np.copysign(np.float32(0.5), x)) * np.float32(1e32)
    ref, lim = conv_ref(x, w, stride, pad), _bound(x, w, stride, pad)
    wd = torch.from_numpy(w).cuda()
    y = B.conv_direct(torch.from_numpy(x).cuda(), wd, stride, pad).cpu().numpy()
    assert (np.abs(y - ref) <= lim).all()
    xh = np.ascontiguousarray(x.transpose(0, 2, 3, 1))
    yh = B.conv_direct_layout(torch.from_numpy(xh).cuda(), wd, stride, pad, B.LAYOUT_HWC).cpu().numpy()
    assert np.array_equal(yh, y.transpose(0, 2, 3, 1))
    xt = np.ascontiguousarray(x.transpose(0, 1, 3, 2))
    yt = B.conv_direct_layout(torch.from_numpy(xt).cuda(), wd, stride, pad, B.LAYOUT_CWH).cpu().numpy()
    assert (np.abs(yt - conv_ref_cwh(xt, w, stride, pad)) <= lim.transpose(0, 1, 3, 2)).all()


@pytest.mark.parametrize("case", [(12, 768, 17, 17, 192, 1, "chw"), (2, 161, 64, 65, 400, 1, "chw"), (70, 515, 7, 5, 500, 1, "chw"),
                                  (4, 300, 61, 61, 450, 2, "chw"), (12, 770, 17, 17, 191, 1, "hwc"), (4, 300, 61, 61, 452, 2, "hwc")])
def test_pointwise_sums_taken_again(gpu, case):
    """One image with operands beyond the parts' range: its outputs are taken again, those of its neighbours keep their bits."""
    torch, B = gpu
    N, C, H, W, K, stride, layout = case
    lay = B.LAYOUT_HWC if layout == "hwc" else B.LAYOUT_CHW
    assert B.iolb_route(B.make_shape(N, C, H, W, K, 1, 1, stride, 0), lay)[0] == B.ROUTE_SPLIT
    x, w = make_inputs(N, C, H, W, K, 1, 1, "u11", "he", seed=N + C + 1)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    big = xd.clone()
    big[1] = (big[1] + torch.copysign(torch.full_like(big[1], 0.5), big[1])) * 1e32
    P, Q = (H - 1) // stride + 1, (W - 1) // stride + 1
    run = lambda a: (B.conv_direct(a, wd, stride, 0) if layout == "chw" else
                     B.conv_direct_layout(a.permute(0, 2, 3, 1).contiguous(), wd, stride, 0, lay).permute(0, 3, 1, 2))
    y, z = run(xd), run(big)
    assert torch.equal(y[0], z[0]) and torch.equal(y[2:], z[2:])
    xs, wk = big[1, :, ::stride, ::stride].double().flatten(1), wd.double().view(K, C)
    lim = (12 * -(-C // 8) + 16) * 2.0 ** -23 * (wk.abs() @ xs.abs())
    assert bool(((z[1].double().flatten(1) - wk @ xs).abs() <= lim).all())


def _framed(torch, values, at):
    """The same values `at` floats after the start of a buffer that is NaN before and after them."""
    frame = torch.full((values.numel() + 80,), float("nan"), device="cuda")
    inside = frame[at:at + values.numel()].view(values.shape)
    inside.copy_(values)
    return frame, inside


def _outside_is_untouched(torch, frame, at, n):
    return bool(torch.isnan(frame[:at]).all()) and bool(torch.isnan(frame[at + n:]).all())


@pytest.mark.parametrize("case", [(64, 256, 14, 14, 256), (50, 260, 12, 15, 261), (50, 300, 10, 13, 300), (12, 768, 17, 17, 192), (9, 256, 30, 34, 250)])
@pytest.mark.parametrize("at", [4, 5, 6])
def test_pointwise_stores_of_several_pixels(gpu, case, at):
    """Neighbouring pixels leave in one store, at any alignment of y, where they cannot run on into another image (planes of a multiple
    of the pixels per lane, or one image per group); the last ones of a plane may be fewer.  Nothing is written beyond y."""
    torch, B = gpu
    N, C, H, W, K = case
    assert B.iolb_route(B.make_shape(N, C, H, W, K, 1, 1, 1, 0))[0] == B.ROUTE_SPLIT
    x, w = make_inputs(N, C, H, W, K, 1, 1, "u11", "he", seed=N + K)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    frame, y = _framed(torch, torch.zeros((N, K, H, W), device="cuda"), at)
    B.conv_direct(xd, wd, 1, 0, y=y)
    assert _outside_is_untouched(torch, frame, at, y.numel())
    xs, wk = xd.double().flatten(2), wd.double().view(1, K, C).expand(N, K, C).contiguous()
    lim = (12 * -(-C // 8) + 16) * 2.0 ** -23 * torch.bmm(wk.abs(), xs.abs())
    assert bool(((y.double().flatten(2) - torch.bmm(wk, xs)).abs() <= lim).all())


def test_what_lies_beyond_the_pixels_is_no_reason_to_take_sums_again(gpu):
    """An odd number of sub-domains: a pair of pixels is read where the plane of inputs ends, and the other half is what the workspace
    held before.  With NaN there the result has the same bits, and no wave takes its block a second time (73 us, 33 without)."""
    torch, B = gpu
    m, N, C, H, W, K = 2, 9, 512, 10, 10, 512                     # 225 sub-domains
    route, need = B.iolb_route(B.make_shape(N, C, H, W, K, algo=B.WINO_ALGO[m]))
    assert route == B.ROUTE_SPLIT and need > 16 * 4 * (C + K) * 225         # (V and M in the workspace: the product)
    x, w = torch.rand((N, C, H, W), device="cuda"), torch.randn((K, C, 3, 3), device="cuda")
    took, out = [], []
    for fill in (0, 255):
        ws = torch.full((need,), fill, dtype=torch.uint8, device="cuda")
        out.append(B.conv_winograd(x, w, m, workspace=ws))
        took.append(1e9)
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                B.conv_winograd(x, w, m, y=out[-1], workspace=ws)
            b.record()
            b.synchronize()
            took[-1] = min(took[-1], a.elapsed_time(b))
    assert torch.equal(out[0], out[1])
    assert took[1] < 1.5 * took[0], took


def test_zeros_around_the_image_meet_infinite_weights(gpu):
    """The border is made of zeros that are multiplied like other operands: 0 times an infinite weight is NaN."""
    torch, B = gpu
    x, w = make_inputs(1, 24, 9, 9, 20, 3, 3, "u11", "he", seed=33)
    x = np.abs(x) + np.float32(0.1)
    w[3, 5, 0, 1], w[7, 2, 2, 2] = np.inf, -np.inf
    y = B.conv_direct(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 1).cpu().numpy()
    assert np.isnan(y[0, 3, 0, :]).all() and (y[0, 3, 1:, :] == np.inf).all()
    assert np.isnan(y[0, 7, 8, :]).all() and np.isnan(y[0, 7, :, 8]).all() and (y[0, 7, :8, :8] == -np.inf).all()
    rest = [k for k in range(20) if k not in (3, 7)]
    assert np.isfinite(y[:, rest]).all()
    tile = B.iolb_tune(B.make_shape(1, 24, 9, 9, 20))
    z = B.conv_direct(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), 1, 1, cfg=tile).cpu().numpy()
    assert np.array_equal(np.isnan(y), np.isnan(z)) and np.array_equal(y[np.isinf(z)], z[np.isinf(z)])


# m, N, C, H, W, K, whether the product is a split one.  Split: ragged channels, kernels and sub-domain counts (not
# multiples of 32, 16, 4) for every m
WINO_CASES = [
    (2, 64, 512, 7, 7, 512, True), (2, 33, 342, 9, 11, 235, True), (2, 9, 179, 21, 20, 510, True), (3, 33, 525, 7, 8, 485, True),
    (4, 5, 187, 35, 34, 489, True), (4, 9, 277, 35, 37, 233, True), (6, 5, 284, 29, 30, 497, True),
    (2, 5, 131, 30, 29, 130, False), (2, 33, 261, 15, 15, 300, False), (4, 2, 290, 75, 73, 384, False),
]


@pytest.mark.parametrize("m,N,C,H,W,K,split", WINO_CASES)
def test_winograd_with_the_split_product(gpu, m, N, C, H, W, K, split):
    """On the fly, pre-transformed, with the least workspace that takes the split product and with the next smaller one,
    which keeps the tuned tile."""
    torch, B = gpu
    shape = B.make_shape(N, C, H, W, K, algo=B.WINO_ALGO[m])
    route, need = B.iolb_route(shape)
    assert route == (B.ROUTE_SPLIT if split else B.ROUTE_TILE)
    needs_as_much = (m, N) == (4, 9)                        # the tuned tile has the larger workspace there
    x, w = make_inputs(N, C, H, W, K, 3, 3, "u01", "he", seed=m + C)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    ref = torch.zeros(N, K, H, W, dtype=torch.float64, device="cuda")
    xp = torch.nn.functional.pad(xd.double(), (1, 1, 1, 1))
    for r in range(3):
        for s in range(3):
            win = xp[:, :, r:r + H, s:s + W].reshape(N, C, H * W).contiguous()
            wk = wd[:, :, r, s].double().view(1, K, C).expand(N, K, C).contiguous()
            ref += torch.bmm(wk, win).view(N, K, H, W)
    ref = ref.cpu().numpy()
    y = B.conv_winograd(xd, wd, m)
    assert rel_err(y.cpu().numpy(), ref) <= GUARD_WINO[m]
    U = B.winograd_transform_kernels(wd, m)[0]
    ws = torch.full((B.winograd_workspace_bytes(N, C, H, W, K, m),), 255, dtype=torch.uint8, device="cuda")    # NaN bits
    yp = B.conv_winograd_pre(xd, U, K, m, workspace=ws)
    assert torch.equal(y, yp)
    ws.fill_(255)
    assert torch.equal(B.conv_winograd(xd, wd, m, workspace=ws), y)
    if split:
        ws.fill_(255)
        assert torch.equal(B.conv_winograd(xd, wd, m, workspace=ws[:need]), y)
        on_tile = B.conv_winograd(xd, wd, m, cfg=B.iolb_tune(shape))
        assert not torch.equal(on_tile, y)
        if not needs_as_much:
            assert torch.equal(B.conv_winograd(xd, wd, m, workspace=ws[:need - 256]), on_tile)


# m, N, C, H, W, K, pad: both block shapes of each m, with columns read whole, cut at the image's edge and one by one;
# sub-domains, kernels and channels that are no multiple of a block's
FUSED_CASES = [
    (2, 8, 64, 28, 28, 64, 1), (2, 5, 20, 41, 39, 70, 1), (2, 12, 36, 60, 61, 66, 2), (2, 16, 128, 14, 14, 96, 1),
    (2, 8, 128, 56, 56, 128, 1), (2, 2, 182, 125, 125, 102, 1), (2, 30, 128, 40, 41, 128, 3),
    (4, 16, 64, 64, 64, 64, 1), (4, 64, 256, 14, 14, 256, 1), (4, 20, 16, 100, 99, 17, 2), (4, 30, 30, 59, 58, 40, 1),
    (4, 8, 80, 128, 128, 144, 1), (4, 12, 36, 60, 61, 66, 1), (4, 1, 48, 300, 301, 34, 2),
    # images of fewer rows than a window has, channels no multiple of the four that are loaded together
    (4, 4, 5, 3, 100, 512, 1), (4, 16, 17, 1, 224, 128, 1), (4, 64, 23, 2, 224, 64, 1), (4, 30, 33, 1, 225, 40, 3),
    (2, 64, 17, 1, 120, 64, 1), (2, 64, 21, 1, 33, 40, 2),
]


def _winograd_ref(torch, xd, wd, pad):
    N, C, H, W = xd.shape
    K, P, Q = wd.shape[0], H + 2 * pad - 2, W + 2 * pad - 2
    ref = torch.zeros(N, K, P * Q, dtype=torch.float64, device="cuda")
    xp = torch.nn.functional.pad(xd.double(), (pad,) * 4)
    for r in range(3):
        for s in range(3):
            win = xp[:, :, r:r + P, s:s + Q].reshape(N, C, P * Q).contiguous()
            ref += torch.bmm(wd[:, :, r, s].double().unsqueeze(0).expand(N, K, C).contiguous(), win)
    return ref.view(N, K, P, Q)


def _runs_fused(B, call):
    """The result of the call, which has to run one Winograd kernel on the bf16 matrix cores."""
    B.timing_enable()
    try:
        B.timing_read(B.TIME_WINO_FUSED)
        y = call()
        launches = B.timing_read(B.TIME_WINO_FUSED)[0]
    finally:
        B.timing_enable(False)
    assert launches == 1
    return y


@pytest.mark.parametrize("m,N,C,H,W,K,pad", FUSED_CASES)
@pytest.mark.parametrize("at", [4, 5])
def test_fused_winograd_in_every_shape(gpu, m, N, C, H, W, K, pad, at):
    torch, B = gpu
    assert B.iolb_route(B.make_shape(N, C, H, W, K, 3, 3, 1, pad, algo=B.WINO_ALGO[m]))[0] == B.ROUTE_SPLIT
    x, w = make_inputs(N, C, H, W, K, 3, 3, "u11", "he", seed=m + C + pad)
    xf, xd = _framed(torch, torch.from_numpy(x).cuda(), at)
    wd = torch.from_numpy(w).cuda()
    yf, y = _framed(torch, torch.zeros((N, K, H + 2 * pad - 2, W + 2 * pad - 2), device="cuda"), at)
    _runs_fused(B, lambda: B.conv_winograd(xd, wd, m, y=y, pad=pad))
    assert _outside_is_untouched(torch, yf, at, y.numel())
    ref = _winograd_ref(torch, xd, wd, pad)
    assert rel_err(y.cpu().numpy(), ref.cpu().numpy()) <= GUARD_WINO[m]
    if pad == 1:
        U = B.winograd_transform_kernels(wd, m)[0]
        ws = torch.full((B.winograd_workspace_bytes(N, C, H, W, K, m),), 255, dtype=torch.uint8, device="cuda")    # NaN bits
        assert torch.equal(_runs_fused(B, lambda: B.conv_winograd_pre(xd, U, K, m, workspace=ws)), y)


@pytest.mark.parametrize("m,N,C,H,W,K,pad", FUSED_CASES)
def test_fused_winograd_sums_taken_again(gpu, m, N, C, H, W, K, pad):
    """One image with operands beyond the parts' range: its outputs are taken again in fp32, all others keep their bits;
    then infinite and NaN kernels, which spoil their own outputs only."""
    torch, B = gpu
    x, w = make_inputs(N, C, H, W, K, 3, 3, "u11", "he", seed=m + C + pad + 1)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    big, i = xd.clone(), N - 1
    big[i] = (big[i] + torch.copysign(torch.full_like(big[i], 0.5), big[i])) * 1e32
    y, z = (_runs_fused(B, lambda: B.conv_winograd(a, wd, m, pad=pad)) for a in (xd, big))
    assert torch.equal(y[:i], z[:i])
    assert rel_err(z[i].cpu().numpy(), _winograd_ref(torch, big[i:], wd, pad)[0].cpu().numpy()) <= GUARD_WINO[m]
    odd = wd.clone()
    odd[1, C - 1, 2, 2], odd[K - 1, 0, 0, 1] = float("inf"), float("nan")
    z = B.conv_winograd(xd, odd, m, pad=pad)
    assert not bool(torch.isfinite(z[:, [1, K - 1]]).any())
    rest = [k for k in range(K) if k not in (1, K - 1)]
    assert torch.equal(z[:, rest], y[:, rest])


@pytest.mark.parametrize("scales", [(1e-38, 1e30), (1e30, 1e-38), (1e33, 1e-10), (1e-10, 1e33)])
@pytest.mark.parametrize("m,N,C,H,W,K,pad", [FUSED_CASES[0], FUSED_CASES[5], FUSED_CASES[8], FUSED_CASES[12]])
def test_fused_winograd_over_the_whole_range(gpu, m, N, C, H, W, K, pad, scales):
    torch, B = gpu
    x, w = make_inputs(N, C, H, W, K, 3, 3, "u11", "he", seed=32)
    xd, wd = torch.from_numpy(x * np.float32(scales[0])).cuda(), torch.from_numpy(w * np.float32(scales[1])).cuda()
    # the fp32 kernels of the tuned tile, asked for by name
    ref = B.conv_winograd(xd, wd, m, cfg=B.iolb_tune(B.make_shape(N, C, H, W, K, algo=B.WINO_ALGO[m]))).cpu().numpy()
    assert rel_err(_runs_fused(B, lambda: B.conv_winograd(xd, wd, m)).cpu().numpy(), ref) <= GUARD_WINO[m]


def test_fused_winograd_in_a_graph_and_on_little_workspace(gpu):
    torch, B = gpu
    m, N, C, H, W, K = 4, 16, 64, 64, 64, 64
    shape = B.make_shape(N, C, H, W, K, algo=B.WINO_ALGO[m])
    need = B.iolb_route(shape)[1]
    x, w = torch.rand((N, C, H, W), device="cuda"), torch.randn((K, C, 3, 3), device="cuda")
    ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
    y = _runs_fused(B, lambda: B.conv_winograd(x, w, m, workspace=ws))
    # (fewer bytes than the split kernels take, but enough for the tile)
    on_tile = B.conv_winograd(x, w, m, cfg=B.iolb_tune(shape))
    assert not torch.equal(on_tile, y)
    with pytest.raises(B.IolbError):
        B.conv_winograd(x, w, m, workspace=ws[:256])
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        B.conv_winograd(x, w, m, y=y, workspace=ws)
    for rep in range(3):
        x.copy_(torch.rand(x.shape, device="cuda"))
        y.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, B.conv_winograd(x, w, m)), rep
        torch.cuda.synchronize()


def test_split_layers_through_the_call_that_allocates_nothing(gpu):
    """The same bits as conv_direct up to its limit on the kernels, in three parts too; beyond it the error stays."""
    torch, B = gpu
    # (641 channels: the kernels fit in fp32, but not their parts, which take whole chunks of 32)
    for (N, C, H, W, K, R, split) in ((1, 640, 5, 5, 704, 3, 1), (1, 641, 9, 9, 704, 3, 0), (2, 20, 12, 12, 40, 5, 1), (12, 768, 17, 17, 192, 1, 1)):
        assert B.iolb_route(B.make_shape(N, C, H, W, K, R, R, 1, R // 2))[0] == split
        x, w = make_inputs(N, C, H, W, K, R, R, "u01", "he", seed=C)
        xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
        y = B.conv_direct(xd, wd, 1, R // 2)
        z = B.conv_direct_noalloc(xd, wd, 1, R // 2, torch.empty_like(y))
        assert torch.equal(y, z)
    x, w = make_inputs(1, 704, 9, 9, 704, 3, 3, "u01", "he", seed=1)      # (4 x 4 would take a tile that needs no room)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    y = torch.full((1, 704, 9, 9), 3.0, device="cuda")
    with pytest.raises(B.IolbError) as e:
        B.conv_direct_noalloc(xd, wd, 1, 1, y)
    assert e.value.code == -4 and bool((y == 3.0).all())
    B.conv_direct(xd, wd, 1, 1, y=y)
    assert rel_err(y.cpu().numpy(), conv_ref(x, w, 1, 1)) <= 3e-5


def test_first_call_of_a_pointwise_layer_may_be_a_captured_one(gpu):
    """A 1 x 1 layer whose fp32 kernel reads the weights in place could always be captured without an eager call before
    it on the stream; its split kernel needs scratch."""
    torch, B = gpu
    N, C, H, K = 12, 768, 17, 192
    assert B.iolb_route(B.make_shape(N, C, H, H, K, 1, 1, 1, 0))[0] == B.ROUTE_SPLIT
    x, w = make_inputs(N, C, H, H, K, 1, 1, "u01", "he", seed=8)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    y = torch.empty((N, K, H, H), device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    B.release_workspace()                                   # no stream has any
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        B.conv_direct(xd, wd, 1, 0, y=y)
    for rep in range(3):
        xd.copy_(torch.rand(xd.shape, device="cuda"))
        y.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, B.conv_direct(xd, wd, 1, 0)), rep
        torch.cuda.synchronize()


@pytest.mark.parametrize("m,N,C,H,W,K", [(4, 9, 277, 35, 37, 233), (2, 64, 512, 7, 7, 512), (6, 5, 284, 29, 30, 497)])
def test_a_workspace_too_small_for_the_tuned_tile_stays_refused(gpu, m, N, C, H, W, K):
    torch, B = gpu
    shape = B.make_shape(N, C, H, W, K, algo=B.WINO_ALGO[m])
    route, need = B.iolb_route(shape)
    assert route == B.ROUTE_SPLIT
    x, w = torch.rand((N, C, H, W), device="cuda"), torch.randn((K, C, 3, 3), device="cuda")
    tile = B.iolb_tune(shape)
    ws = torch.empty(B.winograd_workspace_bytes(N, C, H, W, K, m), dtype=torch.uint8, device="cuda")

    def taken(size, **kw):
        try:
            B.conv_winograd(x, w, m, workspace=ws[:size], **kw)
        except B.IolbError as e:
            assert e.code == -4
            return False
        return True

    # the tile's own size, to 256 bytes
    lo, hi = 0, ws.numel() // 256
    while lo + 1 < hi:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if taken(256 * mid, cfg=tile) else (mid, hi)
    assert taken(256 * hi) and not taken(256 * lo)
    assert need >= 256 * hi and taken(need)
