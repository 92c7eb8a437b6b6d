"""The patch convolution (AUTO's implicit kernel on an input patch in LDS) against the fp64 oracle.

Every test checks in the plan that the patch kernel is what runs.

Every tile config is forced (CONV2D_PATCH_CFG) on shapes that sit on its edges: partial pixel,
channel and row tiles, image borders inside a tile, column blocks, stride, dilation, odd rows (no
pixel pairs), groups, the split reduction and the tail split.  Gates as everywhere: fp32 1e-5 and
bf16 1e-2 per output; integer data is exact (small integers are exact in bf16, so their fp32 split
has no remainder, and every partial sum is an integer below 2^24).
"""

import numpy as np
import pytest

import datagen
import oracle
from paper_2407_10730_amd import binding as B
from paper_2407_10730_amd.runner import DeviceConv

pytestmark = pytest.mark.gpu

GATE = {"f32": 1e-5, "bf16": 1e-2}
TILES = {0: (64, 128), 1: (64, 256), 2: (128, 128), 3: (32, 256), 4: (256, 128)}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load()
    yield
    torch.cuda.synchronize()


def _shape(n, c, h, w, k, r, s, st=1, pd=None, dl=1, g=1, layout="nchw", seed=31):
    pd = dl * (r - 1) // 2 if pd is None else pd
    return datagen.ConvShape(n=n, c=c, h=h, w=w, k=k, r=r, s=s, stride=(st, st), pad=(pd, pd), dil=(dl, dl),
                             groups=g, layout=layout, seed=seed)


# (shape, column blocks)
SHAPES = [
    (_shape(1, 8, 1, 1, 1, 1, 1), 1),                       # one pixel, one row of the tile
    (_shape(2, 17, 9, 11, 33, 3, 3), 1),                    # odd rows, partial chunk, partial row tile
    (_shape(2, 17, 9, 19, 33, 3, 3), 2),                    # ... in column blocks, the last one partial
    (_shape(3, 40, 7, 7, 70, 3, 3, layout="nhwc"), 1),      # several images per tile, 16-byte loads
    (_shape(3, 33, 14, 14, 65, 3, 3), 1),                   # even rows, odd padding (pairs shifted by one)
    (_shape(3, 33, 14, 18, 65, 3, 3), 2),                   # ... and blocks of odd width
    (_shape(2, 24, 16, 18, 48, 3, 3, st=2, dl=2), 1),
    (_shape(1, 16, 5, 130, 32, 5, 5, pd=0), 2),             # one output row, wider than a tile
    # groups: a partial last chunk beside the next group's channels, K/g a multiple of 4 and not
    (_shape(2, 60, 12, 12, 40, 3, 3, g=2), 1),
    (_shape(2, 60, 12, 12, 40, 3, 3, g=2, layout="nhwc"), 1),
    (_shape(2, 66, 11, 26, 42, 3, 3, st=2, g=3), 1),
    (_shape(2, 66, 11, 33, 42, 3, 3, st=2, g=3, layout="nhwc"), 2),
    (_shape(2, 80, 9, 10, 48, 3, 3, g=2, layout="nhwc"), 1),
    (_shape(1, 48, 12, 12, 70, 7, 7, g=2), 1),
    (_shape(2, 72, 10, 12, 66, 1, 1, g=3, layout="nhwc"), 1),
    (_shape(2, 72, 10, 12, 66, 1, 1, g=3), 1),
    (_shape(4, 24, 10, 30, 48, 1, 1), 1),
    (_shape(2, 24, 11, 13, 40, 1, 1, st=2), 1),
    (_shape(2, 72, 10, 12, 130, 1, 1, layout="nhwc"), 1),
    (_shape(2, 12, 9, 10, 20, 1, 3, pd=1), 1),
]
# tiles whose patch needs more staging units than a block has
UNFIT = {("f32", 6): {0, 3}, ("bf16", 6): {0, 4}, ("f32", 10): {0, 3}, ("bf16", 10): {0, 4}, ("bf16", 11): {0, 4}}
TILE_CASES = [(i, dt, cfg) for i in range(len(SHAPES)) for dt in ("f32", "bf16", "bf16-f32") for cfg in TILES
              if not (dt == "f32" and cfg == 4) and cfg not in UNFIT.get((dt.split("-")[0], i), ())]


def _run(monkeypatch, cs, mode, env, calls=1):
    import torch
    monkeypatch.setenv("CONV2D_PATCH", "1")
    for k, v in env.items():
        monkeypatch.setenv("CONV2D_PATCH_" + k, str(v))
    print(f"\n[case] patch {cs} {env} {mode}", flush=True)
    dc = DeviceConv(cs, mode)
    try:
        plan = dc.plan()
        assert plan.algo == B.CONV2D_ALGO_IMPLICIT_GEMM and plan.kernel == B.CONV2D_KERNEL_PATCH
        assert (plan.tile_m, plan.tile_n) == TILES[env["CFG"]]
        ys = []
        for _ in range(calls):
            dc.y.fill_(float("nan"))
            dc.run()
            torch.cuda.synchronize()
            ys.append(dc.y.clone())
        assert all(torch.equal(ys[0], y) for y in ys)
        return dc.y_nchw(), (dc.x_host, dc.w_host, dc.b_host), plan
    finally:
        dc.close()


def _check(monkeypatch, cs, mode, env, calls=1):
    y, (x, w, b), plan = _run(monkeypatch, cs, mode, env, calls)
    ref, a = oracle.conv2d(x, w, b if cs.has_bias else None, cs.stride, cs.pad, cs.dil, cs.groups)
    if mode == "integer" and cs.y_dtype == "f32":
        assert np.array_equal(y, ref)
    else:
        _, pt = oracle.normalised_errors(y, ref, a)
        assert pt <= GATE[cs.x_dtype], pt
    return plan


@pytest.mark.parametrize("i,dt,cfg", TILE_CASES)
def test_patch_tiles(monkeypatch, i, dt, cfg):
    cs, cb = SHAPES[i]
    cs = cs.with_(x_dtype=dt.split("-")[0], y_dtype=dt.split("-")[-1])
    _check(monkeypatch, cs, "integer", {"CFG": cfg, "CB": cb})


@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("c,r", [(60, 3), (80, 3), (72, 1)])
def test_patch_groups_do_not_meet(monkeypatch, layout, dt, c, r):
    """A group whose input is all NaN or infinite leaves the other group's outputs as they are, its
    partial last chunk included, and only its own outputs are not finite."""
    import torch
    monkeypatch.setenv("CONV2D_PATCH", "1")
    cs = _shape(2, c, 9, 10, 48, r, r, g=2, layout=layout).with_(x_dtype=dt, y_dtype="f32")
    x, w, b = datagen.make_inputs(cs, "integer")
    x = x.copy()
    x[0, c // 2:], x[1, c // 2:] = np.nan, np.inf
    dc = DeviceConv(cs, "integer")
    try:
        assert dc.plan().kernel == B.CONV2D_KERNEL_PATCH
        xt = torch.from_numpy(x if layout == "nchw" else np.ascontiguousarray(x.transpose(0, 2, 3, 1))).to(dc.x.dtype)
        dc.x.copy_(xt)
        dc.run()
        torch.cuda.synchronize()
        y = dc.y_nchw()
    finally:
        dc.close()
    ref, _ = oracle.conv2d(np.nan_to_num(x, nan=0.0, posinf=0.0), w, b, cs.stride, cs.pad, cs.dil, cs.groups)
    assert np.array_equal(y[:, :24], ref[:, :24])
    assert not np.isfinite(y[0, 24:]).any()


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("env", [{"CFG": 0, "KSPLIT": 3}, {"CFG": 2, "KSPLIT": 5}, {"CFG": 1, "TAIL": 2},
                                 {"CFG": 0, "TAIL": 4}, {"CFG": 3, "TAIL": 16}], ids=str)
@pytest.mark.parametrize("layout", ["nchw", "nhwc"])
def test_patch_splits(monkeypatch, dt, env, layout):
    """Split reduction (partials added by the unpack) and tail split (added by a tile's last
    piece), partial last chunk; the same bits on every call."""
    cs = _shape(2, 200, 10, 12, 72, 3, 3, layout=layout).with_(x_dtype=dt, y_dtype=dt)
    plan = _check(monkeypatch, cs, "random", env, calls=4)
    assert (plan.ksplit > 1) == ("KSPLIT" in env) and (plan.tail_pieces > 1) == ("TAIL" in env)


@pytest.mark.parametrize("r", [1, 3, 5])
@pytest.mark.parametrize("split", [0, 2])
def test_patch_f32_nonfinite_and_huge(monkeypatch, r, split):
    """fp32 values whose three-way split is not finite (infinities, NaN, values past the largest
    bf16) give what plain fp32 sums give; outputs without them keep the fp32 gate."""
    import torch
    cs = _shape(2, 40, 9, 10, 48, r, r)
    monkeypatch.setenv("CONV2D_PATCH", "1")
    monkeypatch.setenv("CONV2D_PATCH_TAIL", str(split))
    x, w, b = datagen.make_inputs(cs, "random")
    x, w = x.copy(), (w * 1e-3).astype(np.float32)
    x[0, 3, 2, 2], x[0, 7, 6, 5], x[1, 1, 4, 4], x[1, 30, 8, 9] = np.inf, -np.inf, np.nan, 3.4e38
    dc = DeviceConv(cs, inputs=(x, w, b))
    try:
        assert dc.plan().kernel == B.CONV2D_KERNEL_PATCH
        dc.run()
        torch.cuda.synchronize()
        y = dc.y_nchw()
    finally:
        dc.close()
    with np.errstate(all="ignore"):
        ref, a = oracle.conv2d(x, w, b, cs.stride, cs.pad, cs.dil, cs.groups)
    assert np.array_equal(np.isnan(y), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(y[inf], ref[inf])
    ok = np.isfinite(ref)
    assert ok.any() and inf.any() and np.isnan(ref).any()
    assert np.max(np.abs(y[ok] - ref[ok]) / a[ok]) <= GATE["f32"]


def _dense_run(cs, inputs, algo):
    import torch
    dc = DeviceConv(cs, inputs=inputs)
    try:
        assert dc.plan(algo).kernel == B.CONV2D_KERNEL_PATCH
        dc.run(algo)
        torch.cuda.synchronize()
        return dc.y_nchw()
    finally:
        dc.close()


# powers of two of (x, w): plain values; values whose bf16 remainders would be subnormal or vanish
# (below 2^-110), down to the smallest normal and below it; values whose scaled form overflows
EXPONENTS = [(0, 0), (-108, 0), (-112, 0), (-126, 0), (-140, 0), (0, -112), (0, -126), (0, -140), (-60, -60),
             (110, 0), (0, 110), (60, 60)]


@pytest.mark.parametrize("e", EXPONENTS, ids=lambda e: f"x{e[0]}w{e[1]}")
@pytest.mark.parametrize("algo", [B.CONV2D_ALGO_AUTO, B.CONV2D_ALGO_IM2COL_GEMM], ids=["auto", "im2col"])
@pytest.mark.parametrize("r", [1, 3])
@pytest.mark.parametrize("side", ["x", "w"])
def test_patch_f32_keeps_every_bit(monkeypatch, side, r, algo, e):
    """One operand holds 24 significant bits, the other is one-hot (a power of two, the rest zero), so
    every output is one product of 24 bits: exact where it is a normal number, and it needs all three
    planes of the split."""
    monkeypatch.setenv("CONV2D_PATCH", "1")
    monkeypatch.setenv("CONV2D_PATCH_DENSE", "1")
    cs = _shape(2, 40, 9, 10, 48, r, r).with_(has_bias=False)
    rng = np.random.default_rng(5)
    odd = lambda shape: (1 + (2 * rng.integers(0, 1 << 22, shape) + 1) / 2.0 ** 23) * rng.choice([-1.0, 1.0], shape)
    if side == "x":
        x = odd((cs.n, cs.c, cs.h, cs.w))
        w = np.zeros((cs.k, cs.c, r, r))
        for k in range(cs.k):
            w[k, (7 * k) % cs.c, k % r, (k // r) % r] = 1.0
    else:
        x = np.zeros((cs.n, cs.c, cs.h, cs.w))
        for i in range(cs.n):  # windows of different ones do not overlap
            for h in range(1, cs.h, 4):
                for v in range(1, cs.w, 4):
                    x[i, (5 * h + v + 11 * i) % cs.c, h, v] = 1.0
        w = odd((cs.k, cs.c, r, r))
    x, w = np.ldexp(x, e[0]).astype(np.float32), np.ldexp(w, e[1]).astype(np.float32)
    y = _dense_run(cs, (x, w, np.zeros(cs.k, np.float32)), algo)
    ref, _ = oracle.conv2d(x, w, None, cs.stride, cs.pad, cs.dil, cs.groups)
    assert np.count_nonzero(ref) > 500
    assert np.array_equal(y, ref.astype(np.float32))  # (a subnormal product rounds once)


@pytest.mark.parametrize("scale", [(1e-33, 1.0), (1e-36, 1.0), (1.0, 1e-36), (1e-18, 1e-18)], ids=str)
@pytest.mark.parametrize("algo", [B.CONV2D_ALGO_AUTO, B.CONV2D_ALGO_IM2COL_GEMM, B.CONV2D_ALGO_WINOGRAD],
                         ids=["auto", "im2col", "winograd"])
def test_patch_f32_small_magnitudes(monkeypatch, algo, scale):
    """Tensors of small normal values keep the fp32 gate (each output is a normal number; its own
    rounding there is below 2^-24)."""
    monkeypatch.setenv("CONV2D_PATCH", "1")
    monkeypatch.setenv("CONV2D_PATCH_DENSE", "1")
    cs = _shape(2, 64, 14, 14, 64, 3, 3).with_(has_bias=False)
    x, w, b = datagen.make_inputs(cs, "random")
    x, w = (x * scale[0]).astype(np.float32), (w * scale[1]).astype(np.float32)
    y = _dense_run(cs, (x, w, b), algo)
    ref, a = oracle.conv2d(x, w, None, cs.stride, cs.pad, cs.dil, cs.groups)
    assert np.max(np.abs(y - ref) / a) <= GATE["f32"]


@pytest.mark.parametrize("env", [{"KSPLIT": 1, "TAIL": 0}, {"KSPLIT": 1, "TAIL": 2}, {"KSPLIT": 2}], ids=str)
def test_patch_probes(monkeypatch, env):
    """After an AUTO call that ran the patch kernel the probes launch it: the loader probe writes
    nothing, the kernel probe the whole output (a split reduction's goes to its partials)."""
    import torch
    monkeypatch.setenv("CONV2D_PATCH", "1")
    for k, v in env.items():
        monkeypatch.setenv("CONV2D_PATCH_" + k, str(v))
    dc = DeviceConv(_shape(2, 64, 14, 14, 64, 3, 3), "random")
    try:
        plan = dc.plan()
        assert plan.kernel == B.CONV2D_KERNEL_PATCH and plan.ksplit == env["KSPLIT"]
        assert (plan.tail_pieces > 1) == (env.get("TAIL") == 2)
        dc.run()
        torch.cuda.synchronize()
        y0 = dc.y.clone()
        B.conv2d_pack_probe(dc.desc, dc.x, dc.w)
        torch.cuda.synchronize()
        assert torch.equal(dc.y, y0)
        dc.y.zero_()
        for _ in range(2):
            B.conv2d_kernel_probe(dc.desc, dc.x, dc.w, dc.b, dc.y)
        torch.cuda.synchronize()
        assert torch.equal(dc.y, y0) if plan.ksplit == 1 else not dc.y.any()
        dc.run()  # (the tail split's counters are as the kernel left them)
        torch.cuda.synchronize()
        assert torch.equal(dc.y, y0)
    finally:
        dc.close()


@pytest.mark.parametrize("env", [{"KSPLIT": 1, "TAIL": 0}, {"KSPLIT": 1, "TAIL": 2}, {"KSPLIT": 3}], ids=str)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_patch_noalloc(monkeypatch, env, dt):
    """The no-allocation entry point gives the same bits, also after a larger call used its scratch and,
    with the tail split, its shared counters."""
    import torch
    monkeypatch.setenv("CONV2D_PATCH", "1")
    for k, v in env.items():
        monkeypatch.setenv("CONV2D_PATCH_" + k, str(v))
    dcs = [DeviceConv(_shape(n, 96, 14, 14, 64, 3, 3).with_(x_dtype=dt, y_dtype=dt), "random") for n in (5, 2)]
    try:
        for dc in dcs:
            plan = dc.plan()
            assert plan.kernel == B.CONV2D_KERNEL_PATCH and plan.ksplit == env["KSPLIT"]
            assert (plan.tail_pieces > 1) == (env.get("TAIL") == 2)
            dc.run()
        torch.cuda.synchronize()
        s = torch.cuda.current_stream()
        for dc in dcs + dcs[::-1] + dcs:
            y = torch.full_like(dc.y, float("nan"))
            B.conv2d_fwd_noalloc(dc.desc, dc.x, dc.w, dc.b, y, B.CONV2D_ALGO_AUTO, s)
            torch.cuda.synchronize()
            assert torch.equal(y, dc.y)
    finally:
        for dc in dcs:
            dc.close()


@pytest.mark.parametrize("env", [{"KSPLIT": 1, "TAIL": 0}, {"KSPLIT": 1, "TAIL": 2}, {"KSPLIT": 3}], ids=str)
@pytest.mark.parametrize("entry", ["fwd", "noalloc"])
def test_patch_in_a_graph(monkeypatch, entry, env):
    """A captured call replays with new inputs, eager calls and synchronisations between the replays (the
    tail split's counters are left at zero by every launch)."""
    import torch
    monkeypatch.setenv("CONV2D_PATCH", "1")
    for k, v in env.items():
        monkeypatch.setenv("CONV2D_PATCH_" + k, str(v))
    dc = DeviceConv(_shape(2, 96, 14, 14, 64, 3, 3), "random")
    call = B.conv2d_fwd if entry == "fwd" else B.conv2d_fwd_noalloc
    try:
        assert dc.plan().kernel == B.CONV2D_KERNEL_PATCH
        y = torch.empty_like(dc.y)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            for _ in range(2):  # workspaces exist before the capture, on its stream
                call(dc.desc, dc.x, dc.w, dc.b, y, B.CONV2D_ALGO_AUTO, s)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            call(dc.desc, dc.x, dc.w, dc.b, y, B.CONV2D_ALGO_AUTO, s)
        for i in range(4):
            dc.x.mul_(-1.0 if i % 2 else 0.5)
            y.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            call(dc.desc, dc.x, dc.w, dc.b, dc.y, B.CONV2D_ALGO_AUTO, s)
            torch.cuda.synchronize()
            assert y.any() and torch.equal(y, dc.y)
    finally:
        dc.close()


def test_patch_breakdown_does_not_depend_on_the_last_call(monkeypatch):
    """IMPLICIT_GEMM's account holds named calls (here with an unpack) and AUTO's patch calls (without):
    its totals and its fused phases are the same whichever ran last."""
    import torch
    monkeypatch.setenv("CONV2D_PATCH", "1")
    monkeypatch.setenv("CONV2D_PATCH_KSPLIT", "1")
    monkeypatch.setenv("CONV2D_KSPLIT", "2")
    dc = DeviceConv(_shape(2, 64, 14, 14, 64, 3, 3), "random")
    named = B.CONV2D_ALGO_IMPLICIT_GEMM
    try:
        assert dc.plan().kernel == B.CONV2D_KERNEL_PATCH and dc.plan().ksplit == 1
        assert dc.plan(named).kernel == B.CONV2D_KERNEL_GEMM and dc.plan(named).ksplit == 2
        for order in ((B.CONV2D_ALGO_AUTO,), (named, B.CONV2D_ALGO_AUTO), (B.CONV2D_ALGO_AUTO, named)):
            B.conv2d_breakdown_reset(dc.desc)
            for algo in order:
                dc.run(algo)
            torch.cuda.synchronize()
            bd = dc.breakdown(named)
            assert bd["fwd_calls"] == len(order)
            assert ("in_unpacking" in bd["fused"]) == (named not in order)
    finally:
        dc.close()


@pytest.mark.parametrize("layout,dt", [("nhwc", "f32"), ("nchw", "bf16"), ("nhwc", "bf16")])
def test_patch_needs_its_alignment(monkeypatch, layout, dt):
    """An AUTO call whose x is not aligned for the plan's loads runs what a named IMPLICIT_GEMM runs."""
    import torch
    monkeypatch.setenv("CONV2D_PATCH", "1")
    cs = _shape(2, 32, 10, 12, 32, 3, 3, layout=layout).with_(x_dtype=dt, y_dtype=dt)
    dc = DeviceConv(cs, "random")
    try:
        assert dc.plan().kernel == B.CONV2D_KERNEL_PATCH
        buf = torch.empty(dc.x.numel() + 1, dtype=dc.x.dtype, device=dc.x.device)
        xs = buf[1:].view(dc.x.shape)
        xs.copy_(dc.x)
        ys = []
        for algo in (B.CONV2D_ALGO_AUTO, B.CONV2D_ALGO_IMPLICIT_GEMM):
            y = torch.full_like(dc.y, float("nan"))
            B.conv2d_fwd(dc.desc, xs, dc.w, dc.b, y, algo, torch.cuda.current_stream())
            torch.cuda.synchronize()
            ys.append(y)
        assert torch.equal(ys[0], ys[1])
        dc.y.copy_(ys[0])
        ref, a = oracle.conv2d(dc.x_host, dc.w_host, dc.b_host, cs.stride, cs.pad, cs.dil, cs.groups)
        assert oracle.normalised_errors(dc.y_nchw(), ref, a)[1] <= GATE[dt]
    finally:
        dc.close()


def _packed(groups, m, kred, dt):
    """Bytes of the packed filters of a dense GEMM."""
    return groups * -(-m // 32) * -(-kred // 32) * (6 if dt == "f32" else 2) * 1024


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("chunked", [False, True])
@pytest.mark.parametrize("cs", [_shape(2, 9, 13, 11, 70, 3, 3, st=2), _shape(2, 48, 8, 10, 24, 5, 5, g=4),
                                _shape(1, 200, 6, 7, 130, 1, 1, layout="nhwc")], ids=["s2", "g4", "nhwc"])
def test_patch_dense_im2col(monkeypatch, cs, chunked, dt):
    """The explicit path's GEMM on the patch kernel: one chunk (its result split where the planner
    splits it) and two chunks, the second one shorter, whose workspace and packed filters fill the
    limit."""
    import torch
    monkeypatch.setenv("CONV2D_PATCH_DENSE", "1")
    kred = cs.c // cs.groups * cs.r * cs.s
    if chunked:
        ho = (cs.h + 2 * cs.pad[0] - cs.r) // cs.stride[0] + 1
        wo = (cs.w + 2 * cs.pad[1] - cs.s) // cs.stride[1] + 1
        row = wo * (cs.groups * kred * (4 if dt == "f32" else 2) + cs.k * 4)
        limit = _packed(cs.groups, cs.k // cs.groups, kred, dt) + 256 + (cs.n * ho // 2 + 1) * row
        monkeypatch.setenv("CONV2D_WORKSPACE_LIMIT_BYTES", str(limit))
    dc = DeviceConv(cs.with_(x_dtype=dt, y_dtype="f32"), "integer")
    try:
        plan = dc.plan(B.CONV2D_ALGO_IM2COL_GEMM)
        assert plan.kernel == B.CONV2D_KERNEL_PATCH and plan.chunks == (2 if chunked else 1)
        dc.run(B.CONV2D_ALGO_IM2COL_GEMM)
        torch.cuda.synchronize()
        y = dc.y_nchw()
    finally:
        dc.close()
    ref, _ = oracle.conv2d(dc.x_host, dc.w_host, dc.b_host, cs.stride, cs.pad, cs.dil, cs.groups)
    assert np.array_equal(y, ref)


@pytest.mark.parametrize("mt", ["2", "4"])
@pytest.mark.parametrize("chunked", [False, True])
def test_patch_dense_winograd(monkeypatch, mt, chunked):
    """The Winograd GEMMs on the patch kernel, one chunk of tiles and two."""
    import torch
    monkeypatch.setenv("CONV2D_PATCH_DENSE", "1")
    monkeypatch.setenv("CONV2D_WINO_TILE", mt)
    cs = _shape(2, 40, 17, 15, 72, 3, 3)
    if chunked:
        m = int(mt)
        tiles, npos = 2 * -(-17 // m) * -(-15 // m), (m + 2) ** 2
        limit = _packed(npos, 72, 40, "f32") + 256 + npos * (40 + 72) * 4 * (tiles * 3 // 5)
        monkeypatch.setenv("CONV2D_WORKSPACE_LIMIT_BYTES", str(limit))
    dc = DeviceConv(cs, "random")
    try:
        plan = dc.plan(B.CONV2D_ALGO_WINOGRAD)
        assert plan.kernel == B.CONV2D_KERNEL_PATCH and plan.chunks == (2 if chunked else 1)
        dc.run(B.CONV2D_ALGO_WINOGRAD)
        torch.cuda.synchronize()
        y = dc.y_nchw()
    finally:
        dc.close()
    ref, a = oracle.conv2d(dc.x_host, dc.w_host, dc.b_host, cs.stride, cs.pad, cs.dil, cs.groups)
    assert oracle.normalised_errors(y, ref, a)[1] <= GATE["f32"]
