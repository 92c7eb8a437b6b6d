"""Timed cases of the conv2d forward library: what its users run, through its public entry points.

A case is one convolution layer (shape, type, layout, algorithm, entry point).  `prepare` makes
what a program holds before the call (inputs on the GPU, the descriptor, the output tensor), `run`
is one forward call, `exact` is the same layer in float64 with plain torch.
"""
import math

import torch

from paper_2407_10730_amd import binding as B

_ALGOS = {"auto": B.CONV2D_ALGO_AUTO, "im2col": B.CONV2D_ALGO_IM2COL_GEMM,
          "winograd": B.CONV2D_ALGO_WINOGRAD}


def _case(name, n, c, h, w, k, r, s, stride=1, pad=0, dil=1, groups=1, layout="nchw", dtype="f32",
          y_dtype=None, bias=True, algo="auto", entry="fwd"):
    case = {"n": n, "c": c, "h": h, "w": w, "k": k, "r": r, "s": s, "stride": stride, "pad": pad,
            "dil": dil, "groups": groups, "layout": layout, "dtype": dtype, "y_dtype": y_dtype or dtype,
            "bias": bias, "algo": algo, "entry": entry}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # batch-1 stem of a small image: one call is all launch and start-up latency
        _case("stem_n1_f32", 1, 3, 32, 32, 16, 3, 3, pad=1),
        # the square-channel 3x3 layer of a residual network's first stage (the bench's headline)
        _case("conv3x3_f32", 32, 64, 56, 56, 64, 3, 3, pad=1),
        # a wide 3x3 layer of its third stage
        _case("wide3x3_f32", 32, 256, 28, 28, 256, 3, 3, pad=1),
        # bottleneck reduction, 1x1
        _case("pointwise_f32", 32, 256, 56, 56, 64, 1, 1),
        # strided 1x1 shortcut between stages
        _case("downsample_f32", 32, 256, 56, 56, 512, 1, 1, stride=2),
        # 7x7 stride-2 stem on full-size images, both types
        _case("stem7x7_f32", 32, 3, 224, 224, 64, 7, 7, stride=2, pad=3),
        _case("stem7x7_bf16", 32, 3, 224, 224, 64, 7, 7, stride=2, pad=3, dtype="bf16"),
        # depthwise 3x3 on channels-last activations, as mobile networks run it in bf16
        _case("depthwise_nhwc_bf16", 32, 256, 56, 56, 256, 3, 3, pad=1, groups=256, layout="nhwc",
              dtype="bf16"),
        # grouped 3x3 with cardinality 32
        _case("grouped_f32", 32, 256, 56, 56, 256, 3, 3, pad=1, groups=32),
        # the largest: a contraction-bound bf16 layer
        _case("conv3x3_bf16", 32, 256, 56, 56, 256, 3, 3, pad=1, dtype="bf16"),
        # serving at batch 1 on an odd plane through the entry point that never allocates
        _case("batch1_noalloc_bf16", 1, 512, 13, 19, 512, 3, 3, pad=1, dtype="bf16", entry="noalloc"),
        # the baseline algorithm of the comparison (explicit im2col and GEMM) on ragged sizes
        _case("baseline_ragged_f32", 6, 65, 27, 35, 130, 3, 3, pad=2, dil=2, algo="im2col"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost_us(case):
    """A rough time, only to keep drawn cases below the largest listed one."""
    w = work(case)
    if case["groups"] > 1:
        rate = 12e12
    else:
        rate = 70e12 if case["dtype"] == "f32" else 250e12
    moved = w["bytes"]
    if case["algo"] == "im2col":
        ho, wo = _out_hw(case)
        col = case["n"] * ho * wo * case["c"] * case["r"] * case["s"]
        moved += 6 * col * (2 if case["dtype"] == "bf16" else 4)
    return 1e6 * (w["flops"] / rate + moved / 3e12)


def draw(rng):
    while True:
        kind = rng.choice(("regular", "regular", "regular", "pointwise", "pointwise", "depthwise",
                           "grouped", "stem"))
        n = _log_int(rng, 1, 32)
        h = _log_int(rng, 7, 224)
        w = h if rng.random() < 0.6 else _log_int(rng, 7, 224)
        if rng.random() < 0.5:  # common channel counts are multiples of 16, others are anything
            c, k = 16 * _log_int(rng, 1, 128), 16 * _log_int(rng, 1, 128)
        else:
            c, k = _log_int(rng, 3, 1024), _log_int(rng, 3, 1024)
        r = rng.choice((3, 3, 5, 7))
        s = r if rng.random() < 0.9 else rng.choice((1, 3, 5))
        stride, dil, groups = rng.choice((1, 1, 2)), rng.choice((1, 1, 1, 2)), 1
        if kind == "pointwise":
            r = s = dil = 1
        elif kind == "depthwise":
            k = groups = c
            s = r
        elif kind == "grouped":
            groups = rng.choice((2, 4, 8, 16, 32))
            c, k = groups * _log_int(rng, 2, 32), groups * _log_int(rng, 2, 32)
        elif kind == "stem":
            c, k, dil = 3, rng.choice((16, 24, 32, 48, 64, 96)), 1
        dtype = rng.choice(("f32", "bf16"))
        y_dtype = "f32" if dtype == "bf16" and rng.random() < 0.15 else dtype
        algo = rng.choice(("auto", "auto", "auto", "auto", "auto", "im2col"))
        if kind == "regular" and r == s == 3 and stride == dil == 1 and dtype == "f32" and rng.random() < 0.2:
            algo = "winograd"
        pad = dil * (r - 1) // 2
        case = _case(None, n, c, h, w, k, r, s, stride, pad, dil, groups,
                     rng.choice(("nchw", "nchw", "nhwc")), dtype, y_dtype, rng.random() < 0.8, algo, "fwd")
        if w < dil * (s - 1) + 1 or h < dil * (r - 1) + 1:
            continue
        while case["n"] > 1 and _cost_us(case) > 100:
            case["n"] = (case["n"] + 1) // 2
        if _cost_us(case) <= 100:
            return case


def _out_hw(case):
    ho = (case["h"] + 2 * case["pad"] - case["dil"] * (case["r"] - 1) - 1) // case["stride"] + 1
    wo = (case["w"] + 2 * case["pad"] - case["dil"] * (case["s"] - 1) - 1) // case["stride"] + 1
    return ho, wo


def _torch_type(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _tensors(case, seed):
    """x (N, C, H, W), w (K, C/g, R, S) and bias, as a network in use has them: normal activations,
    weights scaled by the fan-in."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    cg = case["c"] // case["groups"]

    def normal(shape, scale):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(scale)

    dt = _torch_type(case["dtype"])
    x = normal((case["n"], case["c"], case["h"], case["w"]), 1.0).to(dt)
    w = normal((case["k"], cg, case["r"], case["s"]), math.sqrt(2.0 / (cg * case["r"] * case["s"]))).to(dt)
    b = normal((case["k"],), 0.1) if case["bias"] else None
    return x, w, b


class _State:
    def __del__(self):
        # work queued on the descriptor must be done before it goes
        if getattr(self, "desc", None):
            torch.cuda.synchronize()
            B.conv2d_desc_destroy(self.desc)
            self.desc = None


def prepare(case, seed):
    st = _State()
    x, w, b = _tensors(case, seed)
    if case["layout"] == "nhwc":
        x = x.permute(0, 2, 3, 1).contiguous()
    st.x, st.w, st.b = x, w, b
    bf = {"f32": B.CONV2D_F32, "bf16": B.CONV2D_BF16}
    st.desc = B.conv2d_desc_create(B.conv2d_params(
        n=case["n"], c=case["c"], h=case["h"], w=case["w"], k=case["k"], r=case["r"], s=case["s"],
        stride_h=case["stride"], stride_w=case["stride"], pad_h=case["pad"], pad_w=case["pad"],
        dil_h=case["dil"], dil_w=case["dil"], groups=case["groups"],
        layout=B.CONV2D_NHWC if case["layout"] == "nhwc" else B.CONV2D_NCHW,
        x_dtype=bf[case["dtype"]], y_dtype=bf[case["y_dtype"]], has_bias=1 if case["bias"] else 0))
    n, k, ho, wo = B.conv2d_output_shape(st.desc)
    shape = (n, ho, wo, k) if case["layout"] == "nhwc" else (n, k, ho, wo)
    st.y = torch.empty(shape, device="cuda", dtype=_torch_type(case["y_dtype"]))
    st.algo = _ALGOS[case["algo"]]
    st.call = B.conv2d_fwd_noalloc if case["entry"] == "noalloc" else B.conv2d_fwd
    return st


def run(st):
    st.call(st.desc, st.x, st.w, st.b, st.y, st.algo, torch.cuda.current_stream())
    return st.y


def work(case):
    """Every input pixel that a window touches, the weights and the bias read once, y written once;
    2 flops per multiply-add of the direct convolution."""
    ho, wo = _out_hw(case)
    es = 2 if case["dtype"] == "bf16" else 4
    ys = 2 if case["y_dtype"] == "bf16" else 4

    def touched(out, size, taps):
        at = {o * case["stride"] - case["pad"] + t * case["dil"] for o in range(out) for t in range(taps)}
        return sum(1 for i in at if 0 <= i < size)

    cg = case["c"] // case["groups"]
    px = touched(ho, case["h"], case["r"]) * touched(wo, case["w"], case["s"])
    y = case["n"] * case["k"] * ho * wo
    weights = case["k"] * cg * case["r"] * case["s"]
    return {"bytes": case["n"] * case["c"] * px * es + weights * es + (case["k"] * 4 if case["bias"] else 0) + y * ys,
            "flops": 2 * y * cg * case["r"] * case["s"]}


def tolerance(case):
    # about four times the error against float64: bf16 outputs show their rounding (1.7e-3), fp32
    # sums 1.5e-7 to 4e-7 and up to 8e-7 on long reductions, fp32 Winograd F(4x4) 3.2e-6
    if case["y_dtype"] == "bf16":
        return {"rel": 7e-3}
    if case["r"] == case["s"] == 3 and case["stride"] == case["dil"] == case["groups"] == 1:
        return {"rel": 1.3e-5}
    long = case["c"] // case["groups"] * case["r"] * case["s"] > 1024
    return {"rel": 4e-6 if long else 2e-6}


def exact(case, seed):
    x, w, b = _tensors(case, seed)
    n, c, g, k = case["n"], case["c"], case["groups"], case["k"]
    ho, wo = _out_hw(case)
    p, st, dl = case["pad"], case["stride"], case["dil"]
    x = torch.nn.functional.pad(x.double(), (p, p, p, p)).reshape(n, g, c // g, case["h"] + 2 * p, case["w"] + 2 * p)
    w = w.double().reshape(1, g, k // g, c // g, case["r"], case["s"])
    y = torch.zeros((n, g, k // g, ho * wo), device="cuda", dtype=torch.float64)
    for r in range(case["r"]):
        for s in range(case["s"]):
            win = x[..., r * dl:r * dl + (ho - 1) * st + 1:st, s * dl:s * dl + (wo - 1) * st + 1:st]
            win = win.reshape(n, g, c // g, ho * wo)
            tap = w[..., r, s].contiguous()
            if c == g:  # one channel per group
                y += tap * win
            else:
                for i in range(n):
                    y[i] += torch.matmul(tap[0], win[i])
    y = y.reshape(n, k, ho, wo)
    if b is not None:
        y += b.double().reshape(1, k, 1, 1)
    return y.permute(0, 2, 3, 1).contiguous() if case["layout"] == "nhwc" else y
