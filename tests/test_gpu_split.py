"""The split members (wm = 1: fp32 products on the bf16 matrix pipes) against the CPU oracle: every way they find their
activations, at the sizes where it can go wrong, and operands that three bf16 numbers cannot hold."""
import numpy as np
import pytest

from oracle import conv as oc
from paper_2008_04567_amd import binding as B
from paper_2008_04567_amd import workloads as W
from tests.parity import check_layer, check_layout, to_dev, torch_dev

pytestmark = pytest.mark.gpu


def cfg(wn, bk, **kw):
    return B.make_config(64, 32 * wn, bk, 1, wn, stages=1, **kw)


# 3x3 with C % 32 == 0 and bk = 16: patches.  Pixel counts just off whole tiles, tiles over several images, one image
# row longer than a tile, padding 0 / 1 / the most that is taken, strides and dilations that still fit, one that does
# not (112 wide with dilation 2: falls back to taps), one and several chunks of channels.
PATCH = [
    W.layer("7x7_n5", 5, 64, 7, 40, 3, 1, 1, x_dist="u11", seed=1),
    W.layer("one_row", 2, 32, (1, 130), 33, 3, 1, 1, x_dist="u11", seed=2),
    W.layer("nopad", 3, 32, (9, 11), 64, 3, 1, 0, x_dist="u11", seed=3),
    W.layer("pad2", 2, 96, (6, 13), 96, 3, 1, 2, x_dist="u11", seed=4),
    W.layer("stride2", 2, 64, (17, 19), 128, 3, 2, 1, x_dist="u11", seed=5),
    W.layer("stride31", 2, 32, (20, 9), 20, 3, (3, 1), 1, x_dist="u11", seed=6),
    W.layer("dil2", 2, 32, 12, 64, 3, 1, 2, dil=2, x_dist="u11", seed=7),
    W.layer("dil31", 1, 32, (15, 10), 64, 3, 1, (3, 1), dil=(3, 1), x_dist="u11", seed=8),
    W.layer("wide", 1, 32, (5, 112), 64, 3, 1, 1, x_dist="u11", seed=9),
    # (channels padded to 16, to 32; the last chunk half empty, full)
    W.layer("c72", 2, 72, (9, 21), 100, 3, 1, 2, dil=2, x_dist="u11", seed=11),
    W.layer("c11", 3, 11, 13, 30, 3, 1, 1, x_dist="u11", seed=12),
    W.layer("c48", 2, 48, 10, 64, 3, 2, 1, x_dist="u11", seed=13),
    # (weights packed through LDS: a block per compute unit and more)
    W.layer("c200_k1100", 1, 200, 6, 1100, 3, 1, 1, x_dist="u11", seed=14),
    W.layer("too_wide", 1, 32, (7, 112), 64, 3, 1, 2, dil=2, x_dist="u11", seed=10),
]


@pytest.mark.parametrize("layer", PATCH, ids=lambda l: l["name"])
@pytest.mark.parametrize("wn", [1, 2, 4])
def test_patches(layer, wn):
    check_layer(layer, cfg(wn, 16), what=layer["name"])
    check_layout(layer, B.NHWC, cfg(wn, 16), what=layer["name"] + " nhwc")


# the other ways: 1x1 four pixels at a time (H * W % 4 == 0, stride 1), 1x1 and larger filters tap by tap, rows where padded channels
# would lengthen the reduction by more than half.
# Reductions of one step up to more than the steps in flight, odd and even.
OTHER = [
    W.layer("point_1step", 3, 32, (6, 6), 64, 1, x_dist="u11", seed=20),
    W.layer("point_11steps", 1, 352, (2, 34), 70, 1, x_dist="u11", seed=21),
    W.layer("point_odd_pixels", 5, 64, 7, 40, 1, x_dist="u11", seed=22),
    W.layer("point_stride2", 2, 96, 14, 64, 1, 2, x_dist="u11", seed=23),
    W.layer("point_pad1", 2, 32, 10, 64, 1, 1, 1, x_dist="u11", seed=24),
    W.layer("taps_5x5", 2, 32, (9, 12), 96, 5, 1, 2, x_dist="u11", seed=25),
    W.layer("taps_3x3_s2", 2, 64, (11, 14), 64, 3, 2, 1, x_dist="u11", seed=26),
    W.layer("taps_1x7", 1, 64, (8, 17), 48, (1, 7), 1, (0, 3), x_dist="u11", seed=27),
    W.layer("taps_c24_1x1", 2, 24, 9, 64, 1, x_dist="u11", seed=31),
    W.layer("taps_c43_5x5", 1, 43, (8, 15), 40, 5, 1, 2, x_dist="u11", seed=32),
    W.layer("taps_c72_wide", 1, 72, (6, 130), 40, 3, 1, 2, dil=2, x_dist="u11", seed=33),
    # (weights packed through LDS, by eight c of all taps, and of 63 and of 64 taps in place)
    W.layer("taps_5x5_k1100", 1, 96, (5, 6), 1100, 5, 1, 2, x_dist="u11", seed=37),
    W.layer("taps_9x7", 1, 64, (13, 12), 70, (9, 7), 1, (4, 3), x_dist="u11", seed=34),
    W.layer("taps_8x8", 1, 32, (12, 13), 40, 8, 1, 3, x_dist="u11", seed=35),
    W.layer("rows_16x15", 1, 5, (17, 18), 36, (16, 15), 1, (2, 3), x_dist="u11", seed=36),
    W.layer("rows_c3_7x7", 2, 3, (30, 26), 64, 7, 2, 3, x_dist="u11", seed=28),
    W.layer("rows_c20", 2, 20, (9, 10), 36, 3, 1, 1, x_dist="u11", seed=29),
    W.layer("rows_c1", 3, 1, 8, 8, 1, x_dist="u11", seed=30),
]


@pytest.mark.parametrize("layer", OTHER, ids=lambda l: l["name"])
@pytest.mark.parametrize("wn", [1, 2, 4])
def test_other_forms(layer, wn):
    check_layer(layer, cfg(wn, 32), what=layer["name"])
    for layout in (B.NHWC, B.X_NHWC, B.Y_NHWC):
        check_layout(layer, layout, cfg(wn, 32), what="%s layout %d" % (layer["name"], layout))


@pytest.mark.parametrize("kw", [dict(split_k=2), dict(split_k=3, reduce=1), dict(split_k=16), dict(persist=1),
                                dict(persist=4), dict(persist=2, reduce=1)], ids=str)
def test_schedules_and_epilogue(kw):
    """Shared tiles both ways, persistent workgroups with whole rounds and dealt-out steps, each with the fused epilogue.
    (144 and 1200 tiles of 64 x 32 on 256 compute units: less than one round, one and a remainder.)"""
    rng = np.random.default_rng(3)
    for layer in (W.layer("sched_patch", 3, 64, 28, 96, 3, 1, 1, x_dist="u11", seed=40),
                  W.layer("sched_point", 4, 96, 40, 380, 1, x_dist="u11", seed=41),
                  W.layer("sched_taps", 3, 64, 28, 96, 3, 2, 1, x_dist="u11", seed=42)):
        P, Q = B.conv_out_shape(B.make_desc(layer))
        bias = rng.uniform(-1, 1, layer["k"]).astype(np.float32)
        res = rng.uniform(-1, 1, (layer["n"], layer["k"], P, Q)).astype(np.float32)
        for wn, bk in ((1, 16), (2, 16), (4, 32)):
            c = cfg(wn, bk, **kw)
            if not B.config_legal(B.make_desc(layer), c):   # more slices than steps
                assert kw["split_k"] * bk > layer["c"] * layer["r"] * layer["s"]
                continue
            for layout in (B.NCHW, B.NHWC):
                check_layout(layer, layout, c, bias=bias, residual=res, relu=True,
                             what="%s %r layout %d" % (layer["name"], kw, layout))


# Every way of finding activations, those that pad channels with and without padding (there infinities and NaN of the next pixel or image,
# or of the last channel again, meet weights of zero): layer, layout, bk.  tests/test_split_forms.py looks up that each is what it is called.
FORMS = {
    "patch": (W.layer("f_patch", 2, 32, 9, 40, 3, 1, 1, x_dist="u11", seed=70), B.NCHW, 16),
    "patch_c27": (W.layer("f_patch27", 2, 27, 9, 40, 3, 1, 1, x_dist="u11", seed=71), B.NCHW, 16),
    "patch_quads": (W.layer("f_pquads", 2, 64, 9, 40, 3, 1, 1, x_dist="u11", seed=72), B.NHWC, 16),
    "point": (W.layer("f_point", 2, 64, 8, 40, 1, x_dist="u11", seed=73), B.NCHW, 32),
    "taps": (W.layer("f_taps", 2, 32, 9, 40, 5, 1, 2, x_dist="u11", seed=74), B.NCHW, 32),
    "quads": (W.layer("f_quads", 2, 32, 9, 40, 3, 1, 1, x_dist="u11", seed=75), B.NHWC, 32),
    "patch_quads_c27": (W.layer("f_pquads27", 2, 27, 9, 40, 3, 1, 1, x_dist="u11", seed=80), B.NHWC, 16),
    "point_c61": (W.layer("f_point61", 2, 61, 8, 40, 1, x_dist="u11", seed=81), B.NCHW, 16),       # (one wave fetches)
    "point_two_c61": (W.layer("f_point61_2", 2, 61, 8, 40, 1, x_dist="u11", seed=82), B.NCHW, 32),  # (two do)
    "taps_c27": (W.layer("f_taps27", 2, 27, 9, 40, 5, 1, 2, x_dist="u11", seed=83), B.NCHW, 32),
    "quads_c27": (W.layer("f_quads27", 2, 27, 9, 40, 5, 1, 2, x_dist="u11", seed=84), B.NHWC, 32),
    "strip": (W.layer("f_strip", 2, 3, 9, 40, 5, 2, 2, x_dist="u11", seed=85), B.NCHW, 16),
    "strip_odd_nhwc": (W.layer("f_strip_cl", 2, 3, 9, 40, 7, 1, 3, x_dist="u11", seed=86), B.NHWC, 16),
    "strip_c22": (W.layer("f_strip22", 2, 22, 9, 40, (1, 3), 1, (0, 1), x_dist="u11", seed=87), B.NCHW, 16),
    "rows": (W.layer("f_rows", 2, 5, 9, 40, 3, 1, 1, x_dist="u11", seed=76), B.NCHW, 32),
    "rows_nhwc": (W.layer("f_rows_cl", 2, 20, 9, 40, 3, 1, 1, x_dist="u11", seed=77), B.NHWC, 32),
}


def run_form(form, x, w, split_k=1):
    """The layer of a form on these operands ([N][C][H][W]); the output as [N][K][P][Q]."""
    torch, dev = torch_dev()
    layer, layout, bk = FORMS[form]
    desc = B.make_desc(layer, layout=layout)
    P, Q = B.conv_out_shape(desc)
    n, k = layer["n"], layer["k"]
    y = torch.empty((n, P, Q, k) if layout else (n, k, P, Q), device=dev)
    B.conv2d_fwd_config(desc, cfg(2, bk, split_k=split_k), to_dev(x.transpose(0, 2, 3, 1) if layout else x), to_dev(w), y)
    torch.cuda.synchronize()
    y = y.cpu().numpy()
    return y.transpose(0, 3, 1, 2) if layout else y


@pytest.mark.parametrize("c,hw,r", [(64, 14, 1), (64, 14, 3), (512, 9, 3)], ids=str)
@pytest.mark.parametrize("layout,bk", [(B.NCHW, 16), (B.NHWC, 16), (B.NCHW, 32), (B.NHWC, 32)], ids=str)
def test_error_against_64_bits(c, hw, r, layout, bk):
    """The six products and two sums leave less than fp32 multiply-adds do.  2-norm of the error over that of the result, normal
    operands, n = C R S terms: the large sum is rounded once per 16 of them, each time by 0.4 * 2^-24 (rms) of a sum that grows
    like a random walk: 0.4 * 2^-24 sqrt(n / 32) in all, and the last rounding; stated twice as large.  Leaving out one
    of the three smallest products costs 1e-6, more than is allowed at any n here."""
    layer = W.layer("precision", 2, c, hw, 64, r, 1, r // 2, seed=90)
    n = c * r * r
    rng = np.random.default_rng(17)
    x = rng.standard_normal((2, c, hw, hw)).astype(np.float32)
    w = rng.standard_normal((64, c, r, r)).astype(np.float32)
    want, _, _ = oc.conv2d(oc.shape_from_layer(layer), x, w)
    torch, dev = torch_dev()
    desc = B.make_desc(layer, layout=layout)
    xd, wd = to_dev(x.transpose(0, 2, 3, 1) if layout else x), to_dev(w)

    def error(config):
        y = torch.empty((2, hw, hw, 64) if layout else (2, 64, hw, hw), device=dev)
        B.conv2d_fwd_config(desc, config, xd, wd, y)
        torch.cuda.synchronize()
        got = y.cpu().numpy().astype(np.float64)
        return np.linalg.norm((got.transpose(0, 3, 1, 2) if layout else got) - want) / np.linalg.norm(want)

    split = error(cfg(2, bk))
    assert split <= 0.8 * 2.0 ** -24 * (1 + np.sqrt(n / 32)), split
    fp32 = error(B.make_config(64, 64, 32, 2, 2))
    assert split <= 0.75 * fp32, (split, fp32)


def scaled(a, power):
    """a * 2^power, rounded to fp32 once."""
    return np.ldexp(a.astype(np.float64), power).astype(np.float32)


# What fp32 sums are off by at most on these layers, over sum |x w|: 45 to 800 terms, each step of the sum rounded by
# 2^-24 of a partial sum that is a small part of sum |x w|; and half the smallest number.
SUM_ERROR = 1e-6


def assert_fp32_sums(got, want, d, what):
    err = np.abs(got.astype(np.float64) - want) - 2.0 ** -149
    worst = float(np.max(err / np.where(d == 0, 1.0, d)))
    assert bool(np.isfinite(got).all()) and worst <= SUM_ERROR, (what, worst)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("split_k", [1, 2])
def test_values_three_bf16_cannot_hold(form, split_k):
    """Infinities, NaN, operands of 2^111 and more and sums of 2^95 and more: what an fp32 sum gives."""
    layer = FORMS[form][0]
    rng = np.random.default_rng(9)
    x, w = W.make_inputs(layer)
    w[:, :, 0, 0] = np.where(rng.uniform(size=w.shape[:2]) < 0.5, 0.5, -2.0)   # exact in bf16: zero remainders
    sh = oc.shape_from_layer(layer)

    hot = x.copy()
    hot[0, 1, 3, 4], hot[0, 2, 5, 5], hot[1, 0, 0, 0], hot[1, -1, 7, 7] = np.inf, -np.inf, np.nan, np.inf
    # (which outputs are infinite, and of which sign, by the rules of the numbers: the oracle sums the same products)
    with np.errstate(invalid="ignore"):
        want, d, _ = oc.conv2d(sh, hot, w)
    got = run_form(form, hot, w, split_k)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    inf = np.isinf(want)
    assert inf.any() and np.array_equal(got[inf], want[inf].astype(np.float32))
    fine = np.isfinite(want)
    assert_fp32_sums(got[fine], want[fine], d[fine], form)

    # (3.4e38 rounds to infinity in bf16; the weights keep the sums finite.  Then a single large operand of either kind, and
    # ordinary operands whose sums are large.)
    one_x, one_w = x.copy(), w.copy()
    one_x[1, 2, 6, 5] = 2.0 ** 120
    one_w[7, 1, 0, 0] = -2.0 ** 120
    for xv, wv in ((np.where(x > 0.5, np.float32(3.4e38), np.float32(1e30)).astype(np.float32), w * np.float32(1e-6)),
                   (one_x, w), (x, one_w), (scaled(x, 60), scaled(w, 40)), (scaled(x, 100), scaled(w, 20))):
        want, d, _ = oc.conv2d(sh, xv, wv)
        assert_fp32_sums(run_form(form, xv, wv, split_k), want, d, form)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("powers", [(-118, 0), (-124, 40), (-126, 0), (-140, 50), (-148, 100)], ids=str)
def test_small_weights(form, powers):
    """Weights as small as fp32 has them, against ordinary and large activations, alone and in every other channel: the
    oracle's sums to fp32's precision."""
    layer = FORMS[form][0]
    x, w = W.make_inputs(layer)
    w = w / np.abs(w).max()   # the powers are those of the largest weight
    x = scaled(x, powers[1])
    small = scaled(w, powers[0])
    mixed = np.where((np.arange(layer["k"]) % 2 == 0)[:, None, None, None], small, w)
    for wv in (small, mixed):
        want, d, _ = oc.conv2d(oc.shape_from_layer(layer), x, wv)
        assert_fp32_sums(run_form(form, x, wv), want, d, (form, powers))


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("split_k", [1, 2])
@pytest.mark.parametrize("powers", [(-118, 0), (-124, 40), (-126, 0), (-140, 50), (-148, 100)], ids=str)
def test_small_activations(form, split_k, powers):
    """Activations as small as fp32 has them, against ordinary and large weights: everywhere, in one image of two, in
    single pixels and in single channels beside ordinary ones."""
    layer = FORMS[form][0]
    x, w = W.make_inputs(layer)
    x = x / np.abs(x).max()
    w = scaled(w, powers[1])
    small = scaled(x, powers[0])
    n, c, h, v = x.shape
    image = np.arange(n)[:, None, None, None] == 1
    pixel = (np.arange(h * v).reshape(h, v) // 5 % 2 == 0)[None, None]
    channel = (np.arange(c) % 2 == 0)[None, :, None, None]
    for where in (np.ones(1, bool), image, pixel, channel):
        xv = np.where(where, small, x)
        want, d, _ = oc.conv2d(oc.shape_from_layer(layer), xv, w)
        assert_fp32_sums(run_form(form, xv, w, split_k), want, d, (form, powers))


def test_weights_of_any_value_move_between_the_packed_forms():
    """The smallest numbers, the largest, infinities and NaN through the split form into the tiled one: bit for bit."""
    torch, dev = torch_dev()
    layer = W.layer("mv_any", 1, 32, 6, 48, 1, x_dist="u11", seed=63)
    desc = B.make_desc(layer)
    x = np.zeros((1, 32, 6, 6), np.float32)
    x[0, np.arange(32), np.arange(32) // 6, np.arange(32) % 6] = 1   # pixel c sees channel c alone
    rng = np.random.default_rng(4)
    w = rng.integers(0, 2 ** 32, (48, 32), dtype=np.uint32)
    w[0, :8] = (1, 0x80000001, 0x007fffff, 0x7f7fffff, 0xff7fffff, 0x77ffffff, 0x7f000000, 0x00800000)
    # infinities and NaN in filters of their own: elsewhere 0 * inf would hide its neighbours
    special = (w >> 23 & 0xff) == 0xff
    special[0] = False
    w[special] &= 0xbfffffff
    w[40], w[41], w[42] = 0x7f800000, 0xff800000, 0x7fc00000
    wd = to_dev(w.view(np.float32).reshape(48, 32, 1, 1))
    xd = to_dev(x)
    a, b = (torch.empty((1, 48, 6, 6), device=dev) for _ in range(2))
    plan = B.Plan([desc])
    plan.set_layer_config(0, cfg(2, 32))
    plan.set_weights(0, wd)
    plan.set_layer_config(0, B.make_config(64, 64, 32, 2, 2))
    plan.run_layer(0, xd, a)
    B.conv2d_fwd_config(desc, B.make_config(64, 64, 32, 2, 2), xd, wd, b)
    torch.cuda.synchronize()
    ai, bi = a.cpu().numpy(), b.cpu().numpy()
    assert np.array_equal(ai, bi, equal_nan=True)
    keep = np.arange(48) < 40
    assert np.array_equal(ai.reshape(48, 36)[keep][:, :32], w.view(np.float32)[keep])
    # and the split kernel on them
    B.conv2d_fwd_config(desc, cfg(2, 32), xd, wd, b)
    torch.cuda.synchronize()
    assert np.array_equal(b.cpu().numpy(), ai, equal_nan=True)


def test_plan_moves_its_weights_between_the_two_packed_forms():
    """A configuration of the other form set after the weights: the plan takes them from the form at hand, exactly."""
    torch, dev = torch_dev()
    for layer in (W.layer("mv_tap", 2, 64, 10, 72, 3, 1, 1, x_dist="u11", seed=60),
                  W.layer("mv_patch", 2, 24, 10, 72, 3, 1, 1, x_dist="u11", seed=62),
                  W.layer("mv_rows", 2, 20, 10, 72, 3, 1, 1, x_dist="u11", seed=61),
                  W.layer("mv_strip", 2, 3, 20, 72, 7, 2, 3, x_dist="u11", seed=64),
                  W.layer("mv_strip_c22", 2, 22, 10, 40, (1, 3), 1, (0, 1), x_dist="u11", seed=65)):
        desc = B.make_desc(layer)
        x, w = W.make_inputs(layer)
        xd, wd = to_dev(x), to_dev(w)
        shape = (layer["n"], layer["k"]) + B.conv_out_shape(desc)
        a, b = torch.empty(shape, device=dev), torch.empty(shape, device=dev)
        tiled, split, other = B.make_config(64, 64, 32, 2, 2), cfg(2, 32), cfg(2, 16)
        # (other: patches, or strips, which have an order of their own beside that of the rows)
        for first, second in ((tiled, split), (split, tiled), (tiled, other), (other, tiled), (split, other), (other, split)):
            plan = B.Plan([desc])
            plan.set_layer_config(0, first)
            plan.set_weights(0, wd)
            plan.set_layer_config(0, second)
            plan.run_layer(0, xd, a)
            B.conv2d_fwd_config(desc, second, xd, wd, b)
            torch.cuda.synchronize()
            assert torch.equal(a, b)


def test_two_threads_launch_patches_of_different_sizes():
    """Patches of more than 64 KB of LDS need a limit raised that belongs to the kernel and not to a launch: two threads on
    streams of their own, with patches of 308 and 372 positions, many launches each."""
    import threading
    torch, dev = torch_dev()
    jobs = []
    for width, seed in ((60, 80), (76, 81)):
        layer = W.layer("lds", 2, 32, (9, width), 64, 3, 1, 2, dil=2, x_dist="u11", seed=seed)
        x, w = W.make_inputs(layer)
        want, d = oc.conv2d(oc.shape_from_layer(layer), x, w)[:2]
        desc = B.make_desc(layer)
        plan = B.Plan([desc])
        plan.set_layer_config(0, cfg(2, 16))
        plan.set_weights(0, to_dev(w))
        y = torch.full(want.shape, float("nan"), device=dev)
        jobs.append((plan, to_dev(x), y, want, d, torch.cuda.Stream()))
    torch.cuda.synchronize()
    failed = []

    def work(plan, x, y, stream):
        try:
            for _ in range(300):
                plan.run_layer(0, x, y, stream)
        except Exception as e:      # pytest sees exceptions of its own thread only
            failed.append(e)

    threads = [threading.Thread(target=work, args=(p, x, y, s)) for p, x, y, _, _, s in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failed, failed
    for _, _, y, want, d, _ in jobs:
        assert_fp32_sums(y.cpu().numpy(), want, d, "threads")
