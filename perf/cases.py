"""Layers on which the speed of the library is measured: one convolution layer per case, through the Python entry
points, over the range of sizes that the networks named in inputs.py and layersets.py use.

A case names the entry point (`call`), the layer and, for Winograd, the output tile edge m:
  direct      binding.conv_direct               x [N][C][H][W], one stride, `pad` or (pad_h, pad_w)
  hwc         binding.conv_direct_layout        the same layer with channels innermost
  winograd    binding.conv_winograd             F(m x m, 3 x 3), kernels transformed in every call
  pre         binding.conv_winograd_pre         kernels transformed once, workspace kept: inference
"""
import math

import torch

from paper_2012_15667_amd import binding as B


def _case(name, call, N, C, H, W, K, R=3, S=3, stride=1, pad_h=1, pad_w=1, m=0, x="u01"):
    return {"name": name, "call": call, "N": N, "C": C, "H": H, "W": W, "K": K, "R": R, "S": S, "stride": stride,
            "pad_h": pad_h, "pad_w": pad_w, "m": m, "x": x}


def listed():
    return [
        # one small image, as in a latency-bound service or a unit test: launches and host work count
        _case("direct_one_image", "direct", 1, 16, 14, 14, 16, x="u11"),
        # a small batch of a mid-network layer in Winograd form: still bound by launches and half-empty grids
        _case("wino2_small_batch", "winograd", 8, 64, 28, 28, 64, m=2, x="u11"),
        # first residual stage of a ResNet at a training batch
        _case("direct_resnet_stage1", "direct", 32, 64, 56, 56, 64),
        # deep, narrow residual stage in the larger Winograd tile; 14 is not a multiple of 4: ragged sub-domains
        _case("wino4_resnet_stage3", "winograd", 64, 256, 14, 14, 256, m=4),
        # last residual stage at inference: 7 x 7 images, kernels transformed beforehand
        _case("wino2_resnet_stage4_pre", "pre", 64, 512, 7, 7, 512, m=2),
        # first layer of a VGG: three channels in, large output, bound by its stores
        _case("direct_vgg_first", "direct", 64, 3, 224, 224, 64),
        # the bulk of a VGG's work, direct and in both Winograd tiles
        _case("direct_vgg_256", "direct", 64, 256, 56, 56, 256),
        _case("wino4_vgg_128", "winograd", 64, 128, 112, 112, 128, m=4),
        _case("wino2_vgg_512", "winograd", 64, 512, 28, 28, 512, m=2),
        # 1 x 1 reduction of an Inception block on odd 17 x 17 images
        _case("direct_pointwise_17", "direct", 64, 768, 17, 17, 192, 1, 1, 1, 0, 0),
        # downsampling layer between two residual stages: stride 2
        _case("direct_stride2", "direct", 64, 128, 28, 28, 256, 3, 3, 2, 1, 1),
        # 5 x 5 layer with channels innermost (second layer of an AlexNet), odd 27 x 27 images
        _case("hwc_5x5_27", "hwc", 16, 96, 27, 27, 256, 5, 5, 1, 2, 2),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# direct-equivalent flop and elements of one tensor that a drawn case stays below (the largest listed layers)
MOST_FLOP = 1.2e11
MOST_ELEMS = 64 * 64 * 224 * 224


def draw(rng):
    """One more layer: kinds as networks use them; batch, image, channels over the whole range, odd sizes included."""
    kind = rng.choice(["3x3", "3x3", "3x3_stride2", "1x1", "1x1", "factorised", "5x5", "first", "hwc", "winograd", "winograd",
                       "winograd", "pre"])
    C, K = _log_int(rng, 16, 512), _log_int(rng, 16, 512)
    if rng.random() < 0.6:                       # most networks' channel counts are multiples of 16
        C, K = (C + 8) // 16 * 16, (K + 8) // 16 * 16
    H = _log_int(rng, 7, 224)
    W = H if rng.random() < 0.7 else max(7, min(224, int(H * rng.uniform(0.7, 1.4))))
    call, R, S, stride, m = "direct", 3, 3, 1, 0
    pad_h = pad_w = 1
    if kind == "3x3_stride2":
        stride, pad_h = 2, rng.choice([0, 1])
        pad_w = pad_h
    elif kind == "1x1":
        R = S = 1
        pad_h = pad_w = 0
        stride = rng.choice([1, 1, 1, 2])
        C = min(2048, C * rng.choice([1, 2, 4]))
    elif kind == "factorised":                   # Inception's one-sided kernels, padded along one axis only
        L = rng.choice([3, 7])
        R, S = rng.choice([(1, L), (L, 1)])
        pad_h, pad_w = R // 2, S // 2
        H = W = rng.choice([8, 9, 17, 18, 35])
    elif kind == "5x5":
        R = S = 5
        pad_h = pad_w = 2
    elif kind == "first":                        # layers on RGB images
        C, (R, stride, pad_h) = 3, rng.choice([(3, 1, 1), (3, 2, 0), (7, 2, 3), (11, 4, 0)])
        S, pad_w = R, pad_h
        H = W = _log_int(rng, 64, 299)
    elif kind == "hwc":
        call = "hwc"
        R = S = rng.choice([1, 3, 3, 5])
        pad_h = pad_w = R // 2
        stride = rng.choice([1, 1, 2])
    elif kind in ("winograd", "pre"):
        call, m = kind, rng.choice([2, 2, 4, 4, 4, 3, 6])
    while True:
        P, Q = (H + 2 * pad_h - R) // stride + 1, (W + 2 * pad_w - S) // stride + 1
        most_n = min(MOST_FLOP / (2.0 * K * P * Q * C * R * S), MOST_ELEMS / float(max(C * H * W, K * P * Q)))
        if most_n >= 1:
            break
        H, W = H * 3 // 4, W * 3 // 4
    N = min(_log_int(rng, 1, 64), int(most_n))
    d = _case("", call, N, C, H, W, K, R, S, stride, pad_h, pad_w, m, rng.choice(["u01", "u01", "u11"]))
    del d["name"]
    return d


def _inputs(case, seed):
    """x uniform on [0, 1] (after a ReLU) or [-1, 1] (centred), w normal with the He deviation, from the seed."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    shape = (case["N"], case["H"], case["W"], case["C"]) if case["call"] == "hwc" else (case["N"], case["C"], case["H"], case["W"])
    x = torch.rand(shape, generator=g, device="cuda", dtype=torch.float32)
    if case["x"] == "u11":
        x.mul_(2).sub_(1)
    w = torch.randn((case["K"], case["C"], case["R"], case["S"]), generator=g, device="cuda", dtype=torch.float32)
    w.mul_(math.sqrt(2.0 / (case["C"] * case["R"] * case["S"])))
    return x, w


def prepare(case, seed):
    x, w = _inputs(case, seed)
    state = {"case": case, "x": x, "w": w}
    if case["call"] == "pre":
        state["U"] = B.winograd_transform_kernels(w, case["m"])[0]
        need = B.winograd_workspace_bytes(case["N"], case["C"], case["H"], case["W"], case["K"], case["m"])
        state["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    return state


def run(state):
    c = state["case"]
    if c["call"] == "direct":
        pad = c["pad_h"] if c["pad_h"] == c["pad_w"] else (c["pad_h"], c["pad_w"])
        return B.conv_direct(state["x"], state["w"], c["stride"], pad)
    if c["call"] == "hwc":
        return B.conv_direct_layout(state["x"], state["w"], c["stride"], c["pad_h"], B.LAYOUT_HWC)
    if c["call"] == "winograd":
        return B.conv_winograd(state["x"], state["w"], c["m"])
    return B.conv_winograd_pre(state["x"], state["U"], c["K"], c["m"], workspace=state["workspace"])


def _out(case):
    return ((case["H"] + 2 * case["pad_h"] - case["R"]) // case["stride"] + 1,
            (case["W"] + 2 * case["pad_w"] - case["S"]) // case["stride"] + 1)


def work(case):
    """Each input read once, each output written once; the multiplications and additions of the algorithm the entry
    point names (Winograd: the products of the transformed tiles and their channel sums)."""
    N, C, K, m = case["N"], case["C"], case["K"], case["m"]
    P, Q = _out(case)
    if m:
        tiles = N * -(-P // m) * -(-Q // m)
        flops = 2 * (m + 2) ** 2 * tiles * C * K
    else:
        flops = 2 * N * K * P * Q * C * case["R"] * case["S"]
    weights = K * C * ((m + 2) ** 2 if case["call"] == "pre" else case["R"] * case["S"])
    return {"bytes": 4 * (N * C * case["H"] * case["W"] + weights + N * K * P * Q), "flops": flops}


def tolerance(case):
    """32-bit sums over up to 12800 products; the Winograd transforms amplify rounding with m.  About four times the
    largest distance from `exact` seen over the listed and 30 drawn cases (direct 1.6e-6 / 1.1e-5, m = 2 5.2e-7 / 4.4e-6,
    m = 4 2.9e-6 / 6.6e-5, m = 6 4.4e-6 / 8.4e-5)."""
    rel, most = {0: (6e-6, 5e-5), 2: (4e-6, 4e-5), 3: (1e-5, 2e-4), 4: (1.2e-5, 3e-4), 6: (2e-5, 4e-4)}[case["m"]]
    return {"rel": rel, "max": most}


def exact(case, seed):
    """The layer in 64 bits, as one matrix product per kernel element over the shifted input."""
    x, w = _inputs(case, seed)
    hwc = case["call"] == "hwc"
    x = (x.permute(0, 3, 1, 2) if hwc else x).double()
    w = w.double()
    P, Q = _out(case)
    st = case["stride"]
    x = torch.nn.functional.pad(x, (case["pad_w"], case["pad_w"], case["pad_h"], case["pad_h"]))
    y = torch.zeros((case["N"], case["K"], P * Q), dtype=torch.float64, device=x.device)
    for r in range(case["R"]):
        for s in range(case["S"]):
            win = x[:, :, r:r + st * (P - 1) + 1:st, s:s + st * (Q - 1) + 1:st].reshape(case["N"], case["C"], P * Q).contiguous()
            wrs = w[:, :, r, s].unsqueeze(0).expand(case["N"], -1, -1).contiguous()
            y += torch.bmm(wrs, win)
    y = y.reshape(case["N"], case["K"], P, Q)
    return y.permute(0, 2, 3, 1).contiguous() if hwc else y
