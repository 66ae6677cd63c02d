"""GPU parity of the implicit-GEMM families that the launch planner chooses by size: eight-wave tiles, tiles that
keep a 3x3 neighbourhood in LDS and tiles whose waves split the reduction, and of the few-channel and eight-wave weight-gradient kernels.  Every tile is forced on shapes around its edges (rows and channels one below, at and above a tile,
fewer slices than waves or ring stages, strided row classes, a class without taps) and compared with the CPU checker."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2205_10357_amd import binding as B                 # noqa: E402
from paper_2205_10357_amd import workloads as wl              # noqa: E402
from tests import parity_util as pu                           # noqa: E402

SHAPES = {
    "one_slice_few_rows": dict(N=1, H=3, W=5, C_in=64, C_out=64, K=1, stride=1, pad=0, res=True),
    "rows_one_over_a_tile": dict(N=1, H=3, W=43, C_in=64, C_out=136, K=3, stride=1, pad=1, res=True),
    "rows_one_under_a_tile": dict(N=1, H=5, W=51, C_in=128, C_out=264, K=3, stride=1, pad=1),
    "long_reduction_few_rows": dict(N=1, H=4, W=4, C_in=512, C_out=72, K=3, stride=1, pad=1),
    "strided_classes": dict(N=2, H=15, W=13, C_in=64, C_out=128, K=3, stride=2, pad=1),
    "strided_1x1": dict(N=2, H=9, W=11, C_in=192, C_out=320, K=1, stride=2, pad=0, relu=False),
}


KINDS = {"SOL_WIDE": "eight waves", "SOL_HALO": "neighbourhood in LDS", "SOL_KSPLIT": "waves split the reduction", "SOL_FAST_STAGES": "pipelined"}


def halo_serves(tile, W, C, K):
    """Whether a 3x3 / 5x5 "same" launch over C source channels and rows of W pixels fits the neighbourhood tile: two channel
    slices of its pixels (one for 64 channels), a ring of four weight slices and a row of zeros in 160 KiB, and the copies of
    the next slice's pixels done two taps before it, at most two per tap.  (Two per tap occur with 128 x 64 tiles only: eight
    copies of the others do not fit.)"""
    bp, bc, per_copy = {1: (256, 128, 64), 2: (128, 128, 64), 3: (128, 64, 32)}[tile]
    copies = -(-(bp + (K - 1) * (W + 1)) // per_copy)
    lds = 4 * bc * 128 + 128 + (2 if C > 64 else 1) * copies * per_copy * 128
    return lds <= 160 * 1024 and (C == 64 or copies <= 2 * (K * K - 2))


def check_family(family, n, d, kinds):
    """The launch trace names the forced family for the forward launch and, where its channels allow, the data gradient."""
    gemms = [k for k in kinds if k.startswith("implicit GEMM")]
    assert len(gemms) == 2, kinds
    for kind, channels in zip(gemms, (d.C_in, d.C_out)):
        serves = family in ("SOL_KSPLIT", "SOL_FAST_STAGES") or channels % 64 == 0
        if family == "SOL_HALO":
            serves = serves and halo_serves(n, d.W, channels, d.KH)
        assert (f"({KINDS[family]})" in kind) == serves, (kind, channels)
    return gemms


def run_forced(shape, family, n, sol_env, rides=False):
    sol_env(family, n)
    case = pu.make_case(211, **SHAPES[shape])
    r = np.random.default_rng(212)
    dxm = wl.snap_to_bf16(np.maximum(r.standard_normal(case["x"].shape), 0).astype(np.float32))
    ad = wl.snap_to_bf16(r.standard_normal(case["x"].shape).astype(np.float32))
    if rides:
        sol_env("SOL_REDUCE_RIDES", 3)
    print(f"[{family}={n}] {shape}", flush=True)
    B.sol_trace_start(64)
    got = pu.gpu_block(case, addend=ad, dx_mask=dxm, premasked=True)
    kinds = [B.sol_trace_kind_name(k) for k, _, _, _ in B.sol_trace_stop(64)]
    if family in KINDS and int(n) > 0:
        check_family(family, int(n), case["d"], kinds)
    pu.check_block(case, got, addend=ad, dx_mask=dxm, premasked=True)
    return got


@pytest.mark.parametrize("tile", [1, 2, 3])
@pytest.mark.parametrize("shape", list(SHAPES), ids=list(SHAPES))
def test_eight_wave_tiles(shape, tile, sol_env):
    """Also bit for bit against the four-wave 64 x 64 tile (same order of the reduction), with riding reductions."""
    got = run_forced(shape, "SOL_WIDE", tile, sol_env, rides=True)
    sol_env("SOL_WIDE", -1)
    sol_env("SOL_FAST_TILE", 2)
    ref = run_forced(shape, "SOL_KSPLIT", -1, sol_env)
    for key in ("y", "dx"):
        assert np.array_equal(got[key], ref[key]), key


@pytest.mark.parametrize("tile", [1, 2, 3, 4])
@pytest.mark.parametrize("shape", list(SHAPES), ids=list(SHAPES))
def test_tiles_whose_waves_split_the_reduction(shape, tile, sol_env):
    """Twice: the partial tiles are added in a fixed order, so the bits repeat; the second time with riding reductions."""
    a = run_forced(shape, "SOL_KSPLIT", tile, sol_env)
    b = run_forced(shape, "SOL_KSPLIT", tile, sol_env, rides=True)
    for key in ("y", "dx", "dW", "dscale", "dshift"):
        assert np.array_equal(a[key], b[key]), key


HALO_SHAPES = {
    "image_smaller_than_the_filter_reach": dict(N=3, H=1, W=2, C_in=64, C_out=64, K=3, stride=1, pad=1),
    "rows_one_over_a_tile": dict(N=1, H=3, W=43, C_in=64, C_out=136, K=3, stride=1, pad=1, res=True),
    "many_images_in_a_tile": dict(N=11, H=5, W=6, C_in=192, C_out=72, K=3, stride=1, pad=1),
    "two_copies_per_slice": dict(N=1, H=6, W=56, C_in=128, C_out=128, K=3, stride=1, pad=1, res=True),
    "wide_rows": dict(N=1, H=4, W=61, C_in=128, C_out=64, K=3, stride=1, pad=1),
    "5x5": dict(N=2, H=9, W=11, C_in=128, C_out=72, K=5, stride=1, pad=2),
    "widest_rows_of_the_256_pixel_tile": dict(N=2, H=11, W=31, C_in=128, C_out=192, K=3, stride=1, pad=1),
    "one_pixel_too_wide_for_it": dict(N=1, H=9, W=32, C_in=192, C_out=128, K=3, stride=1, pad=1),
}


@pytest.mark.parametrize("tile", [1, 2, 3])
@pytest.mark.parametrize("shape", list(HALO_SHAPES), ids=list(HALO_SHAPES))
def test_tiles_that_keep_the_neighbourhood(shape, tile, sol_env):
    """Forward and data gradient, again with riding reductions; bits repeat.  Rows too wide for a tile take another family."""
    SHAPES[shape] = HALO_SHAPES[shape]
    a = run_forced(shape, "SOL_HALO", tile, sol_env)
    b = run_forced(shape, "SOL_HALO", tile, sol_env, rides=True)
    for key in ("y", "dx", "dW", "dscale", "dshift"):
        assert np.array_equal(a[key], b[key]), key


@pytest.mark.parametrize("shape", [
    dict(N=1, H=4, W=4, C_in=16, C_out=16, K=1, stride=1, pad=0),                 # exactly one tile
    dict(N=3, H=5, W=7, C_in=17, C_out=33, K=3, stride=1, pad=1, res=True),       # one over a tile everywhere
    dict(N=1, H=1, W=1, C_in=1, C_out=1, K=1, stride=1, pad=0),                   # fewer reduction elements than waves
    dict(N=2, H=11, W=9, C_in=5, C_out=3, K=5, stride=3, pad=2),
])
def test_fp32_matrix_kernels(shape):
    case = pu.make_case(231, bf16=False, **shape)
    r = np.random.default_rng(232)
    ad = r.standard_normal(case["x"].shape).astype(np.float32)
    am = r.standard_normal(case["x"].shape).astype(np.float32)
    one = pu.gpu_block(case, addend=ad, addend_mask=am, want_dres=True)
    pu.check_block(case, one, addend=ad, addend_mask=am)
    two = pu.gpu_block(case, addend=ad, addend_mask=am, two_calls=True)           # each branch as a launch of its own
    for key in ("dx", "dW", "dscale", "dshift"):
        assert np.array_equal(one[key], two[key]), key


def _same_class_and_value(name, got, ref, tol):
    """NaN and the two infinities exactly where the checker has them; finite values to `tol` of their norm."""
    kind = lambda a: np.isnan(a) * 1 + np.isposinf(a) * 2 + np.isneginf(a) * 3
    assert np.array_equal(kind(got), kind(ref)), (name, int((kind(got) != kind(ref)).sum()), int((kind(ref) > 0).sum()))
    fin = np.isfinite(ref)
    assert pu.rel_l2(got[fin], ref[fin]) <= tol, name


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("plant", ["w", "dy"])
@pytest.mark.parametrize("shape", [
    dict(N=2, H=9, W=11, C_in=3, C_out=20, K=3, stride=1, pad=1),
    dict(N=1, H=14, W=13, C_in=17, C_out=5, K=3, stride=2, pad=1),
    dict(N=2, H=7, W=6, C_in=4, C_out=33, K=5, stride=2, pad=2),
])
def test_fp32_infinite_operand_spares_what_no_tap_reaches(shape, plant, value):
    """A weight or gradient that is not finite reaches the results its taps reach and no other: a tap outside the image, or
    between the strides, is skipped and not multiplied by zero."""
    case = pu.make_case(233, bf16=False, relu=False, **shape)
    d = case["d"]
    r = np.random.default_rng(234)
    case["dy"] = r.standard_normal((d.N, d.C_out, d.Ho, d.Wo)).astype(np.float32)
    flat = case[plant].reshape(-1)
    flat[[0, flat.size // 3, flat.size - 1]] = value
    x, w, dy = (pu.to_dev(case[k], False) for k in ("x", "w", "dy"))
    scale, shift = pu.vec_dev(case["scale"]), pu.vec_dev(case["shift"])
    desc = B.BlockDesc(d.N, d.H, d.W, d.C_in, d.C_out, d.KH, d.KW, d.stride, d.pad, B.SOL_F32, 0)
    y, dx, dW = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w)
    ds, db = torch.empty_like(scale), torch.empty_like(scale)
    ws = torch.empty(B.sol_block_workspace_bytes(desc, B.SOL_PASS_BWD), dtype=torch.uint8, device="cuda")
    B.sol_block_fwd(desc, x, w, scale, shift, None, y, None)
    B.sol_block_bwd(desc, dy, x, w, None, dx, dW, ds, db, scale, None, None, None, None, ws)
    torch.cuda.synchronize()
    y_o = pu.orc.block_fwd(d, case["x"], case["w"], case["scale"], case["shift"])
    g = pu.orc.block_bwd(d, case["dy"], case["x"], case["w"], y_o, case["scale"])
    _same_class_and_value("y", pu.to_host(y), y_o, pu.TOL["f32"])
    _same_class_and_value("dx", pu.to_host(dx), g["dx"], pu.TOL["f32"])
    _same_class_and_value("dW", pu.to_host(dW), g["dW"], pu.TOL["f32"])
    _same_class_and_value("dshift", pu.to_host(db, None), g["dshift"], pu.TOL["f32"])


def test_fp32_tensor_with_more_tiles_than_one_dimension_of_a_launch_holds():
    """2^27 + 16 pixels of one channel: 2^23 + 1 tiles of 512 threads are more than the 2^32 - 1 threads that a dimension of a
    launch may have.  All values are small integers and the gradient is zero but for every 4096th pixel, so every result is
    exact."""
    n = (1 << 27) + 16
    desc = B.BlockDesc(1, 16, n // 16, 1, 1, 1, 1, 1, 0, B.SOL_F32, 0)
    x = (torch.arange(n, device="cuda", dtype=torch.int32) % 7).float().view(1, 16, n // 16, 1)
    one = lambda v: torch.full((1,), float(v), device="cuda")
    w, y, dx = one(3).view(1, 1, 1, 1), torch.full_like(x, -1.0), torch.full_like(x, -1.0)
    B.sol_block_fwd(desc, x, w, one(2), one(5), None, y, None)
    assert torch.equal(y, 6.0 * x + 5.0)
    dy = torch.zeros_like(x)
    dy.view(-1)[::4096] = 1.0
    dW, ds, db = torch.empty_like(w), one(-1), one(-1)
    ws = torch.empty(B.sol_block_workspace_bytes(desc, B.SOL_PASS_BWD), dtype=torch.uint8, device="cuda")
    B.sol_block_bwd(desc, dy, x, w, None, dx, dW, ds, db, one(2), None, None, None, None, ws)
    assert torch.equal(dx, 6.0 * dy)
    g = float(x.view(-1)[::4096].double().sum())
    assert (float(dW), float(ds), float(db)) == (2 * g, 3 * g, float(dy.double().sum()))


RAGGED_SHAPES = {
    "8_channels_many_taps_per_slice": dict(N=2, H=9, W=7, C_in=8, C_out=16, K=5, stride=1, pad=2),
    "56_channels_one_short_slice": dict(N=1, H=6, W=11, C_in=56, C_out=8, K=1, stride=1, pad=0, res=True),
    "72_to_104_stride_2": dict(N=1, H=13, W=11, C_in=72, C_out=104, K=3, stride=2, pad=1),
    "slices_19_and_a_fraction": dict(N=1, H=8, W=9, C_in=136, C_out=72, K=3, stride=1, pad=1),
    "strided_1x1": dict(N=2, H=9, W=11, C_in=200, C_out=24, K=1, stride=2, pad=0, relu=False),
    "rows_one_over_a_tile": dict(N=1, H=3, W=43, C_in=24, C_out=136, K=3, stride=1, pad=1),
}


@pytest.mark.parametrize("force", ["SOL_FAST_TILE=1,SOL_FAST_STAGES=2", "SOL_FAST_TILE=1,SOL_FAST_STAGES=4",
                                   "SOL_FAST_TILE=2,SOL_FAST_STAGES=2", "SOL_FAST_TILE=2,SOL_FAST_STAGES=4",
                                   "SOL_KSPLIT=1", "SOL_KSPLIT=2", "SOL_KSPLIT=3", "SOL_KSPLIT=4", "SOL_REDUCE_RIDES=1"])
@pytest.mark.parametrize("shape", list(RAGGED_SHAPES), ids=list(RAGGED_SHAPES))
def test_channels_that_are_no_multiple_of_64(shape, force, sol_env):
    """Forward, data gradient and re-packed weights (riding with the weight gradient) of channel counts that are multiples
    of 8 on every pipelined tile that serves them, and on the library's own choice."""
    SHAPES[shape] = RAGGED_SHAPES[shape]
    for setting in force.split(","):
        name, value = setting.split("=")
        sol_env(name, value)
    run_forced(shape, name, value, sol_env)


FEW_CHANNEL_SHAPES = {
    "odd_rows_and_pairs": dict(N=2, H=33, W=35, C_in=3, C_out=64, K=7, stride=2, pad=3),          # odd Ho: half a last pair
    "two_pixels_in_the_second_segment": dict(N=1, H=10, W=259, C_in=3, C_out=64, K=7, stride=2, pad=3),
    "segments_and_images_within_one_range": dict(N=33, H=37, W=261, C_in=3, C_out=64, K=7, stride=2, pad=3),
    "window_taller_than_the_image": dict(N=3, H=2, W=5, C_in=3, C_out=64, K=7, stride=2, pad=3),
    "one_row_window": dict(N=70, H=23, W=9, C_in=2, C_out=64, K=1, stride=2, pad=0),
    "even_window_1_channel": dict(N=5, H=15, W=17, C_in=1, C_out=64, K=4, stride=2, pad=1),
    "unpadded_3_rows": dict(N=7, H=31, W=31, C_in=3, C_out=64, K=3, stride=2, pad=0),
    "8x8_window_4_channels": dict(N=2, H=29, W=40, C_in=4, C_out=64, K=8, stride=2, pad=4),       # forward kernel only
}


@pytest.mark.parametrize("shape", list(FEW_CHANNEL_SHAPES), ids=list(FEW_CHANNEL_SHAPES))
def test_few_channel_row_ring(shape):
    """Forward and weight gradient of layers with up to four input channels: every way a range of output rows can begin
    and end (odd heights, several segments or images in one range, windows reaching past the image on both sides)."""
    print(f"[few channels] {shape}", flush=True)
    case = pu.make_case(221, **FEW_CHANNEL_SHAPES[shape])
    got = pu.gpu_block(case, need_dx=False, premasked=True)
    pu.check_block(case, got, need_dx=False, premasked=True)
    again = pu.gpu_block(case, need_dx=False, premasked=True)
    for key in ("y", "dW", "dscale", "dshift"):
        assert np.array_equal(got[key], again[key]), key


WIDE_WGRAD_SHAPES = {
    "one_slice": dict(N=1, H=5, W=7, C_in=64, C_out=72, K=3, stride=1, pad=1),
    "images_smaller_than_a_slice": dict(N=41, H=3, W=5, C_in=128, C_out=136, K=3, stride=1, pad=1),
    "row_advance_carries_into_the_image": dict(N=7, H=13, W=11, C_in=72, C_out=104, K=3, stride=1, pad=1),
    "stride_2_odd": dict(N=5, H=23, W=17, C_in=64, C_out=128, K=3, stride=2, pad=1),
    "strided_1x1": dict(N=9, H=15, W=19, C_in=136, C_out=200, K=1, stride=2, pad=0, relu=False),
    "taps_that_reach_no_pixel": dict(N=30, H=2, W=3, C_in=24, C_out=16, K=5, stride=1, pad=2),
    "window_at_the_edge_only": dict(N=12, H=9, W=9, C_in=8, C_out=264, K=5, stride=2, pad=0),
    "1x1": dict(N=3, H=21, W=9, C_in=256, C_out=128, K=1, stride=1, pad=0),
}


@pytest.mark.parametrize("splits", [0, 1, 3])
@pytest.mark.parametrize("shape", list(WIDE_WGRAD_SHAPES), ids=list(WIDE_WGRAD_SHAPES))
def test_eight_wave_weight_gradient(shape, splits, sol_env):
    """The eight-wave weight gradient (fewer slices than ring stages, images below a slice, carries of the walking gather,
    strides, taps without any pixel, partial tiles) with the riding re-pack, against the checker and twice the same bits."""
    sol_env("SOL_WGRAD_WIDE", 1)
    if splits:
        sol_env("SOL_WGRAD_SPLITS", splits)
    print(f"[eight-wave wgrad] {shape} splits={splits}", flush=True)
    case = pu.make_case(231, **WIDE_WGRAD_SHAPES[shape])
    got = pu.gpu_block(case, premasked=True)
    pu.check_block(case, got, premasked=True)
    again = pu.gpu_block(case, premasked=True)
    for key in ("dx", "dW", "dscale", "dshift"):
        assert np.array_equal(got[key], again[key]), key


@pytest.mark.parametrize("shape", [
    dict(N=32, H=56, W=56, C_in=64, C_out=64, K=1, stride=1, pad=0, res=True),        # one tile, four waves
    dict(N=43, H=56, W=56, C_in=8, C_out=16, K=3, stride=1, pad=1),                   # one tile, eight waves
])
def test_narrow_layer_with_more_splits_than_can_ride(shape):
    """The library's own split of one output tile and a long reduction: more than 64, so with a reduction of its own."""
    case = pu.make_case(243, **shape)
    d = case["d"]
    desc = B.BlockDesc(d.N, d.H, d.W, d.C_in, d.C_out, d.KH, d.KW, d.stride, d.pad, B.SOL_BF16, 0)
    assert B.sol_block_wgrad_partial_bytes(desc) > 64 * 4 * d.C_out * (d.KH * d.KW * d.C_in + 1)
    got = pu.gpu_block(case, premasked=True)
    pu.check_block(case, got, premasked=True)


@pytest.mark.parametrize("wide,chains", [(-1, 2), (1, 4)])
def test_weight_gradient_adds_in_several_chains(wide, chains, sol_env):
    """Error of one split of 2048 steps of 16 pixels against 64-bit sums.  A chain of n fp32 additions of random terms has a
    relative error of c * sqrt(n / 2) with c = 0.62 * 2^-24 (what one chain per output showed here, 0.4 of it the rounding of
    an addition); the bound lies between the number of chains the kernel has and half of it."""
    sol_env("SOL_WGRAD_SPLITS", 1)
    sol_env("SOL_WGRAD_WIDE", wide)
    n, hw, ci, co = 8, 64, 128, 128
    g = torch.Generator(device="cuda").manual_seed(242)
    x = torch.rand(n, hw, hw, ci, generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randn(n, hw, hw, co, generator=g, device="cuda").to(torch.bfloat16)
    W, scale = torch.zeros(co, 1, 1, ci, device="cuda").to(torch.bfloat16), torch.ones(co, device="cuda")
    d = B.BlockDesc(n, hw, hw, ci, co, 1, 1, 1, 0, B.SOL_BF16, 0)
    dW, ds, db = torch.empty(co, 1, 1, ci, device="cuda"), torch.empty(co, device="cuda"), torch.empty(co, device="cuda")
    ws = torch.empty(B.sol_block_workspace_bytes(d, B.SOL_PASS_BWD), dtype=torch.uint8, device="cuda")
    B.sol_block_bwd(d, dy, x, W, None, None, dW, ds, db, scale, None, None, None, None, ws)
    ref = dy.view(-1, co).double().t() @ x.view(-1, ci).double()
    err = float((dW.view(co, ci).double() - ref).norm() / ref.norm())
    steps = n * hw * hw / 16
    print(f"error {err:.3g}", flush=True)
    assert err <= 0.62 * 2.0 ** -24 * np.sqrt(steps / chains / 2) * 2 ** 0.25


@pytest.mark.parametrize("masked", [False, True])
def test_strided_block_adds_to_its_input_gradient_in_place(masked):
    """1x1 / stride 2 with dx as its own addend: the pixels it reaches get the sum, the others stay (or take the mask)."""
    d = B.BlockDesc(3, 13, 11, 64, 128, 1, 1, 2, 0, B.SOL_BF16, 0)
    g = torch.Generator(device="cuda").manual_seed(241)
    draw = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    W, dy, dx0 = draw(128, 1, 1, 64), draw(3, d.Ho, d.Wo, 128), draw(3, 13, 11, 64)
    x, scale, mask = draw(3, 13, 11, 64), torch.rand(128, generator=g, device="cuda"), draw(3, 13, 11, 64) if masked else None
    ws = torch.empty(B.sol_block_workspace_bytes(d, B.SOL_PASS_BWD), dtype=torch.uint8, device="cuda")
    out = []
    for in_place in (True, False):
        dx = dx0.clone() if in_place else torch.full_like(dx0, 7.0)
        B.sol_block_bwd(d, dy, x, W, None, dx, None, None, None, scale, None, dx if in_place else dx0, None, mask, ws)
        out.append(dx)
    assert torch.equal(out[0], out[1])
    if not masked:
        assert torch.equal(out[0][:, 1::2], dx0[:, 1::2]) and torch.equal(out[0][:, :, 1::2], dx0[:, :, 1::2])


@pytest.mark.parametrize("shape", [
    dict(N=4, H=16, W=44, C_in=256, C_out=1024, K=1, stride=1, pad=0, res=True),      # 704 tiles of 64 x 64: the last resident
    dict(N=4, H=16, W=45, C_in=256, C_out=1024, K=1, stride=1, pad=0, res=True),      # one column of tiles more: 128 x 64
    dict(N=1, H=32, W=40, C_in=512, C_out=2048, K=1, stride=1, pad=0, res=True),      # eight slices, 640 tiles
    dict(N=1, H=32, W=41, C_in=512, C_out=2048, K=1, stride=1, pad=0, res=True),
])
def test_pointwise_launches_around_the_resident_tile_lines(shape):
    """The library's own choice of tile on either side of the lines between small tiles resident at once and the others."""
    case = pu.make_case(251, **shape)
    got = pu.gpu_block(case, premasked=True)
    pu.check_block(case, got, premasked=True)


@pytest.mark.parametrize("how", ["plan", "environment"])
@pytest.mark.parametrize("layer", [dict(C_in=256, C_out=256, K=3, stride=1, pad=1), dict(C_in=1024, C_out=256, K=1, stride=1, pad=0),
                                   dict(C_in=72, C_out=104, K=3, stride=2, pad=1), dict(C_in=64, C_out=256, K=1, stride=1, pad=0)])
def test_image_has_the_same_bits_in_every_batch_on_request(layer, how, sol_env):
    """With a plan for the shape, or the two families of other orders switched off, the first image's forward result and data
    gradient do not depend on the batch it is in."""
    big = pu.make_case(261, N=33, H=14, W=14, res=True, **layer)
    if how == "environment":
        sol_env("SOL_HALO", -1)
        sol_env("SOL_KSPLIT", -1)
    out = {}
    try:
        for n in (1, 5, 33):
            case = dict(big, d=pu.orc.Desc(n, 14, 14, layer["C_in"], layer["C_out"], layer["K"], layer["K"], layer["stride"], layer["pad"], True),
                        **{k: big[k][:n] for k in ("x", "res", "t")})
            d = case["d"]
            desc = B.BlockDesc(d.N, d.H, d.W, d.C_in, d.C_out, d.KH, d.KW, d.stride, d.pad, B.SOL_BF16, B.SOL_RELU)
            if how == "plan":
                for which in (B.SOL_PLAN_FWD, B.SOL_PLAN_DGRAD):
                    B.sol_block_set_plan(desc, which, (1 if n == 5 else 2, 0, 0))
            # (the loss gradient depends on the batch by its 1 / numel: the stored output serves as dy instead)
            x, w, t = pu.to_dev(case["x"], True), pu.to_dev(case["w"], True), pu.to_dev(case["res"], True)
            scale, shift = pu.vec_dev(case["scale"]), pu.vec_dev(case["shift"])
            y, dx = torch.empty_like(t), torch.empty_like(x)
            ws = torch.empty(B.sol_block_workspace_bytes(desc, B.SOL_PASS_BWD), dtype=torch.uint8, device="cuda")
            B.sol_block_fwd(desc, x, w, scale, shift, t, y, None)
            B.sol_block_bwd(desc, y, x, w, y, dx, None, None, None, scale, None, None, None, None, ws)
            torch.cuda.synchronize()
            out[n] = (y[0].clone(), dx[0].clone())
    finally:
        B.sol_clear_plans()
    for n in (5, 33):
        assert torch.equal(out[n][0], out[1][0]) and torch.equal(out[n][1], out[1][1]), n
