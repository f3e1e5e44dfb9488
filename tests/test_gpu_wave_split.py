"""How tiles leave the wave-split members: every wave adds up and stores a part of the tile, with the fused epilogue, over
channel counts that fill no block, pixels that fill no tile, all layouts of y, and reductions that end in the middle of
a filter tap, cut between workgroups or not.  Bar: 1e-4 * sum|x*w| against the CPU oracle, as everywhere."""
import numpy as np
import pytest

from oracle import conv as oc
from paper_2008_04567_amd import binding as B
from paper_2008_04567_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu

LAYERS = [
    # 13 x 9 pixels (117: no whole number of tiles), K = 37: no whole block and no whole quad; five taps of 96 channels to a row
    W.layer("ws_ragged", 1, 96, (13, 9), 37, (3, 5), 1, (1, 2), x_dist="u11", w_dist="u11", seed=301),
    # K = 68: whole quads, the second block of 64 has one quad; stride and dilation
    W.layer("ws_quads", 2, 32, (12, 11), 68, 3, (2, 1), 2, 2, x_dist="u11", w_dist="u11", seed=302),
    # one tap, fewer octets than eight waves in five slices have runs; K = 64 whole
    W.layer("ws_short", 3, 32, (5, 7), 64, 1, x_dist="u11", w_dist="u11", seed=303),
]


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("layer", LAYERS, ids=[l["name"] for l in LAYERS])
def test_wave_split_members_carry_tiles_out(layer, layout):
    desc = B.make_desc(layer, layout=layout)
    P, Q = B.conv_out_shape(desc)
    rng = np.random.default_rng(layer["seed"])
    bias = rng.uniform(-1, 1, layer["k"]).astype(np.float32)
    res = rng.uniform(-1, 1, (layer["n"], layer["k"], P, Q)).astype(np.float32)
    ran = 0
    for bn in (32, 64):
        for wm, wn in ((1, 1), (2, 1), (4, 1), (4, 2)):
            for split, reduce in ((1, 0), (2, 0), (5, 1), (9, 0)):
                cfg = B.make_config(32, bn, 8, wm, wn, split, 1, 0, 1 + split % 3, reduce)
                if not B.config_legal(desc, cfg):
                    continue
                print(cfg, flush=True)
                PT.check_layout(layer, layout, cfg=cfg)
                PT.check_layout(layer, layout, cfg=cfg, bias=bias, residual=res, relu=True)
                ran += 1
    assert ran >= 8


@pytest.mark.parametrize("k", [16, 37, 64])
def test_residual_that_y_takes_the_place_of(k):
    """Residuals are read ahead of the loop where four waves or more share a tile (and no slices meet): each wave reads and writes its
    own outputs.  Pixels and channels that fill no tile; 16 channels: lanes past the last pixel would be just past the tensor."""
    layer = W.layer("ws_inplace_%d" % k, 1, 64, (11, 13), k, 3, 1, 1, x_dist="u11", w_dist="u11", seed=320 + k)
    desc = B.make_desc(layer)
    P, Q = B.conv_out_shape(desc)
    x, w = W.make_inputs(layer)
    rng = np.random.default_rng(k)
    res = rng.uniform(-2, 2, (1, k, P, Q)).astype(np.float32)
    bias = rng.uniform(-1, 1, k).astype(np.float32)
    y_ref, d_ref = oc.conv2d_fused(oc.shape_from_layer(layer), x, w, bias=bias, residual=res, relu=True)
    xd, wd, bd = PT.to_dev(x), PT.to_dev(w), PT.to_dev(bias)
    ran = 0
    for bn in (32, 64):
        for wm, wn in ((1, 1), (2, 1), (4, 1), (4, 2)):
            for split in (1, 3):
                cfg = B.make_config(32, bn, 8, wm, wn, split, 1, 0, 1, 0)
                if not B.config_legal(desc, cfg):
                    continue
                print(cfg, flush=True)
                y = PT.to_dev(res)
                B.conv2d_fwd_fused(desc, xd, wd, y, bias=bd, residual=y, relu=True, cfg=cfg)
                PT.assert_close(y.cpu().numpy(), y_ref, d_ref, repr(cfg))
                ran += 1
    assert ran >= 12
