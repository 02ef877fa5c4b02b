"""Which kernel a call without a tile runs on (iolb_route): a property of the layer, whatever was asked before, and within
the fixed room of conv_direct_noalloc.  Host only, except where marked."""
import ctypes
import json
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2012_15667_amd import binding as B
from tests import plan_host
from tests.test_split_kernels import MANY_BLOCKS, NOT_OWN_LAYERS, OWN_LAYERS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SCRATCH_BYTES = 6 * 4194304              # conv_direct_noalloc's array: 4 Mi weights in three bf16 parts

# 1 x 1 layers with more kernels than that array holds: (N, C, H, W, K)
LARGE_POINT = [(8, 2304, 14, 14, 2304), (8, 2048, 17, 17, 2304), (4, 2560, 16, 16, 2560)]


def _routes(order):
    """iolb_route of every layer in the given layout order, asked in a process of its own (the library remembers)."""
    code = ("import json; from paper_2012_15667_amd import binding as B\n"
            "out = {}\n"
            "for l in %r:\n"
            "    for lay in %r:\n"
            "        out['%%s %%s' %% (l, lay)] = B.iolb_route(B.make_shape(*l, 1, 1, 1, 0), lay)\n"
            "print(json.dumps(out))" % (LARGE_POINT, order))
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, stdout=subprocess.PIPE, text=True, check=True, timeout=100)
    return json.loads(r.stdout)


def test_the_route_does_not_depend_on_what_was_asked_before():
    a = _routes([B.LAYOUT_CWH, B.LAYOUT_CHW, B.LAYOUT_HWC])
    assert a == _routes([B.LAYOUT_CHW, B.LAYOUT_HWC, B.LAYOUT_CWH])


def _noalloc_takes(shape):
    """The limit conv_direct_noalloc states, on the tile of conv_direct."""
    t = B.iolb_tune(shape)
    padded = -(-shape.K // 32) * 32 * -(-shape.C // t["alpha"]) * t["alpha"] * shape.R * shape.S
    return t["path"] != B.PATH_MFMA or padded <= 4194304


@pytest.mark.parametrize("layer", LARGE_POINT + [(1, 704, 9, 9, 640), (1, 704, 9, 9, 704), (1, 640, 5, 5, 704), (2, 1024, 8, 8, 1024)])
def test_layers_the_call_without_allocation_takes_fit_its_room(layer):
    R = 1 if layer in LARGE_POINT else 3
    shape = B.make_shape(*layer, R, R, 1, R // 2)
    for layout in (B.LAYOUT_CWH, B.LAYOUT_CHW):                 # another layout's tile first
        route, need = B.iolb_route(shape, layout)
        if _noalloc_takes(shape):
            assert need <= SCRATCH_BYTES, layout
        if need > SCRATCH_BYTES:
            assert route == B.ROUTE_SPLIT


def test_division_by_multiplication_is_exact_in_its_range():
    """The library's Divisor for every n d < 2^31: around the multiples of d and at the largest n, where it would be wrong first."""
    rng = np.random.default_rng(0)
    for d in list(range(1, 600)) + rng.integers(600, 1 << 20, 400).tolist() + [32767, 32768, 32769, (1 << 30) + 1, (1 << 31) - 1]:
        most = ((1 << 31) - 1) // d
        k = np.unique(np.concatenate([np.arange(0, 200), rng.integers(0, most // d + 1, 200), [most // d]]))
        n = np.unique(np.concatenate([k * d - 1, k * d, k * d + 1, [most]]))
        n = np.ascontiguousarray(n[(n >= 0) & (n <= most)].astype(np.int32))
        q = np.empty_like(n)
        plan_host.lib().divide(n.ctypes.data, len(n), d, q.ctypes.data)
        assert np.array_equal(q, n // d), d


@pytest.mark.parametrize("layer", [
    # N, C, H, W, K, R, S, stride, pad
    (1, 16, 14, 14, 16, 3, 3, 1, 1), (64, 256, 56, 56, 256, 3, 3, 1, 1), (2, 3, 60, 60, 7, 7, 7, 2, 3), (1, 8, 224, 224, 64, 11, 11, 4, 0),
    (3, 17, 40, 300, 40, 1, 65, 1, 0), (2, 9, 33, 35, 17, 2, 2, 5, 0), (600, 40, 14, 14, 2000, 3, 3, 1, 1), (4352, 9, 14, 14, 512, 3, 3, 1, 1),
    (64, 64, 224, 224, 512, 3, 3, 1, 1), (8192, 9, 7, 7, 512, 3, 3, 1, 1),
])
def test_what_the_direct_kernel_divides_is_in_that_range(layer):
    facts = (ctypes.c_int * 4)()
    assert plan_host.lib().split_facts(*layer, facts) == 1
    assert facts[3] == 1 and facts[2] == (facts[0] <= 32768), list(facts)


@pytest.mark.parametrize("layer,own", [(l, 1) for l in OWN_LAYERS] + [(l, 0) for l in NOT_OWN_LAYERS] + [(MANY_BLOCKS, 0)])
def test_which_layers_prepare_their_own_kernels(layer, own):
    facts = (ctypes.c_int * 4)()
    assert plan_host.lib().split_facts(*layer, facts) == 1 and facts[3] == 1
    assert facts[1] == own
    assert (facts[0] > 32768) == (layer == MANY_BLOCKS)         # workgroups: where ids are divided as integers


@pytest.mark.parametrize("layer", [
    # N, C, H, W, K, m, pad: tiles times the tiles of an image on both sides of 2^31
    (1, 8, 180, 180, 8, 2, 1), (1, 5, 430, 430, 32, 2, 1), (1, 5, 432, 432, 32, 2, 1), (64, 16, 99, 101, 64, 4, 1), (200, 5, 129, 131, 40, 4, 2),
    (1, 5, 4000, 4001, 32, 2, 1), (20000, 5, 7, 7, 100, 2, 1),
])
def test_what_the_fused_winograd_kernel_divides_is_in_that_range(layer):
    N, C, H, W, K, m, pad = layer
    facts = (ctypes.c_int * 3)()
    assert plan_host.lib().wino_split_facts(*layer, facts) == 1
    per = -(-(H + 2 * pad - 2) // m) * -(-(W + 2 * pad - 2) // m)
    assert facts[2] == 1 and (facts[1] == 1 or (N * per + 64) * per >= 1 << 31 or facts[0] ** 2 >= 1 << 31)


@pytest.mark.parametrize("m,layer", [
    (3, (8, 128, 77, 77, 304)), (3, (23, 128, 47, 65, 336)), (6, (4, 128, 128, 128, 176)), (6, (14, 256, 104, 104, 160)),
])
def test_winograd_layers_of_many_channels_keep_the_product(m, layer):
    """It is 1.1 - 1.35 times as fast there as the tile, to which its modelled time sends them."""
    N, C, H, W, K = layer
    route, need = B.iolb_route(B.make_shape(*layer, algo=B.WINO_ALGO[m]))
    assert route == B.ROUTE_SPLIT and need > 4 * (m + 2) ** 2 * (C + K) * N * -(-H // m) * -(-W // m)      # V and M in the workspace



@pytest.mark.parametrize("m", [2, 4])
@pytest.mark.parametrize("pad", [1, 2, 3])
def test_scalar_offsets_of_the_fused_winograd_loads_stay_inside_one_image(m, pad):
    """The hardware checks a lane's offset against the buffer's range less the scalar offset: that must not wrap, whatever
    the lanes' masks say.  Images of fewer rows than a window has, every remainder of C by the four channels loaded together."""
    for H in range(1, 8):
        for W in (1, 2, 3, 5, 100, 224):
            for C in list(range(5, 36)) + [100, 101, 102, 103]:
                for N, K in ((1, 64), (4, 512)):
                    beyond = plan_host.lib().wino_split_beyond_range(N, C, H, W, K, m, pad)
                    assert beyond <= 0, (N, C, H, W, K, beyond)


@pytest.mark.gpu
@pytest.mark.parametrize("first", [B.LAYOUT_CWH, B.LAYOUT_CHW])
def test_large_pointwise_layers_give_the_same_bits_whatever_ran_before(first):
    """Another layout first, then conv_direct_noalloc: the result of conv_direct, nothing written beside the scratch."""
    import torch
    N, C, H, K = (8, 2304, 14, 2304) if first == B.LAYOUT_CWH else (4, 2304, 14, 2304)
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.rand((N, C, H, H), generator=g, device="cuda") - 0.5
    w = torch.randn((K, C, 1, 1), generator=g, device="cuda") * C ** -0.5
    B.conv_direct_layout(x, w, 1, 0, first)
    y = torch.full((N, K, H, H), 7.0, device="cuda")
    B.conv_direct_noalloc(x, w, 1, 0, y)
    assert torch.equal(y, B.conv_direct(x, w, 1, 0))
    ref = torch.bmm(w.double().view(1, K, C).expand(N, K, C).contiguous(), x.double().flatten(2).contiguous()).view(N, K, H, H)
    # sums of C fp32 products: every rounding at most 2^-23 of the magnitudes
    lim = 2 * C * 2.0 ** -23 * torch.bmm(w.double().abs().view(1, K, C).expand(N, K, C).contiguous(), x.double().abs().flatten(2).contiguous()).view(N, K, H, H)
    assert bool(((y.double() - ref).abs() <= lim).all())


@pytest.mark.gpu
def test_calls_follow_the_current_stream_with_and_without_the_raw_handle(monkeypatch):
    """Graphs record what is enqueued on the capture's stream: a call on another one would leave y as it was."""
    import torch
    x, w = torch.rand((2, 24, 9, 9), device="cuda"), torch.randn((20, 24, 3, 3), device="cuda")
    want = B.conv_direct(x, w, 1, 1)
    for without in (False, True):
        if without:
            monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
        y = torch.zeros_like(want)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            B.conv_direct(x, w, 1, 1, y=y)
        for _ in range(2):
            y.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, want), without
