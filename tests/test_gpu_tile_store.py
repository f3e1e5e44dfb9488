"""How tiles leave the tiled and the split members: what a block adds is asked for ahead of the stores of the block before
it.  One, two, four and eight blocks per wave, every layout, each of bias, residual and rectifier alone and all together, over
channel counts that fill no block (69: no whole quad either) and pixels that fill no tile; and a residual that y takes the place of.
Bar: 1e-4 * sum|x*w| against the CPU oracle, as everywhere."""
import numpy as np
import pytest

from oracle import conv as oc
from paper_2008_04567_amd import binding as B
from paper_2008_04567_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu

# blocks of 32 x 32 per wave: 1, 2 (channels), 4, 8; split members of two and four multiplying waves
TILES = [(64, 32, 16, 2, 1), (64, 64, 8, 2, 1), (128, 64, 16, 2, 1), (256, 128, 16, 2, 2), (64, 64, 32, 1, 2), (64, 128, 16, 1, 4)]


@pytest.mark.parametrize("k", [69, 72, 128])
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
def test_tiles_leave_with_what_they_add(layout, k):
    layer = W.layer("store_k%d" % k, 2, 32, (11, 13), k, 3, 1, 1, x_dist="u11", w_dist="u11", seed=410 + k)
    desc = B.make_desc(layer, layout=layout)
    P, Q = B.conv_out_shape(desc)
    rng = np.random.default_rng(k)
    bias = rng.uniform(-1, 1, k).astype(np.float32)
    res = rng.uniform(-2, 2, (2, k, P, Q)).astype(np.float32)
    ran = 0
    for tile in TILES:
        cfg = B.make_config(*tile)
        if not B.config_legal(desc, cfg):
            continue
        print(layout, cfg, flush=True)
        for b, r, relu in ((None, None, False), (None, None, True), (bias, None, False), (None, res, False), (bias, res, True)):
            PT.check_layout(layer, layout, cfg=cfg, bias=b, residual=r, relu=relu)
        ran += 1
    assert ran >= 5


@pytest.mark.parametrize("tile", TILES)
def test_residual_that_y_takes_the_place_of(tile):
    layer = W.layer("store_inplace", 2, 32, (11, 13), 72, 1, x_dist="u11", w_dist="u11", seed=420)
    desc, cfg = B.make_desc(layer), B.make_config(*tile)
    P, Q = B.conv_out_shape(desc)
    if not B.config_legal(desc, cfg):
        pytest.skip("not a configuration of this layer")
    x, w = W.make_inputs(layer)
    res = np.random.default_rng(7).uniform(-2, 2, (2, 72, P, Q)).astype(np.float32)
    y_ref, d_ref = oc.conv2d_fused(oc.shape_from_layer(layer), x, w, residual=res, relu=True)
    y = PT.to_dev(res)
    print(cfg, flush=True)
    B.conv2d_fwd_fused(desc, PT.to_dev(x), PT.to_dev(w), y, residual=y, relu=True, cfg=cfg)
    PT.assert_close(y.cpu().numpy(), y_ref, d_ref, repr(cfg))


@pytest.mark.parametrize("tile", [(64, 32, 8, 2, 1), (64, 64, 32, 2, 2), (128, 64, 16, 2, 2), (64, 64, 32, 1, 2)])
def test_biases_of_tiles_that_follow_each_other(tile):
    """Persistent workgroups take tiles of other channels one after the other: each is stored with its own bias, which waits in LDS while
    others of the workgroup still store the tile before; also the tiles dealt out in runs."""
    layer = W.layer("store_persist", 2, 32, (61, 83), 232, 1, x_dist="u11", w_dist="u11", seed=430)
    x, w = W.make_inputs(layer)
    rng = np.random.default_rng(9)
    bias = rng.uniform(-4, 4, 232).astype(np.float32)
    y_ref, d_ref = oc.conv2d_fused(oc.shape_from_layer(layer), x, w, bias=bias)
    desc = B.make_desc(layer)
    for persist in (1, 2):
        cfg = B.make_config(*tile, persist=persist)
        assert B.config_legal(desc, cfg)
        print(cfg, flush=True)
        y = PT.run_gpu_fused(layer, x, w, bias=bias, cfg=cfg)
        PT.assert_close(y, y_ref, d_ref, repr(cfg))
