"""The split members' strips (layers of few channels) and their fetching waves against the CPU oracle, at the sizes where they
can go wrong."""
import pytest

from paper_2008_04567_amd import binding as B
from paper_2008_04567_amd import workloads as W
from tests.parity import check_layer, check_layout

pytestmark = pytest.mark.gpu


def cfg(wn, bk, **kw):
    return B.make_config(64, 32 * wn, bk, 1, wn, stages=1, **kw)


# Each number of depths (6, 10, 16, 22 octets and one less), even and odd strides (whole dwords, shifted ones), filters of two to eight
# columns and one row, rows just inside the strip's width, images of one strip and of several with a short last one, channels that
# leave waves of the last group without any, several groups.
STRIP = [
    W.layer("stem", 1, 3, 64, 64, 7, 2, 3, x_dist="u11", seed=1),
    W.layer("octets22_s8", 1, 2, (40, 37), 40, (11, 8), 1, (5, 3), x_dist="u11", seed=2),
    W.layer("octets21_odd", 2, 3, (19, 33), 70, 7, 1, 3, x_dist="u11", seed=3),
    W.layer("octets16", 1, 4, (23, 50), 33, 4, 2, 1, x_dist="u11", seed=4),
    W.layer("octets15", 2, 3, (30, 31), 130, 5, 3, 2, x_dist="u11", seed=5),
    W.layer("octets9", 3, 3, 29, 32, 3, 1, 1, x_dist="u11", seed=6),
    W.layer("octets5_s2", 1, 5, (9, 40), 64, (1, 2), (1, 2), 0, x_dist="u11", seed=7),
    W.layer("octets1_k300", 5, 1, (6, 51), 300, (1, 2), 2, 0, x_dist="u11", seed=8),
    W.layer("wide_even", 1, 3, (12, 233), 64, 7, 2, 3, x_dist="u11", seed=9),
    W.layer("wide_odd", 1, 1, (5, 231), 64, 7, 1, 3, x_dist="u11", seed=10),
    W.layer("dil_rows", 1, 3, (31, 20), 64, 5, (1, 2), (4, 2), dil=(2, 1), x_dist="u11", seed=11),
    W.layer("one_pixel", 2, 3, 7, 16, 7, x_dist="u11", seed=12),
    # (as many octets from many channels of one filter row)
    W.layer("c22_1x2", 2, 22, (9, 33), 40, (1, 2), (1, 2), 0, x_dist="u11", seed=13),
    W.layer("c22_1x3", 2, 22, (9, 33), 70, (1, 3), 1, (0, 1), x_dist="u11", seed=14),
    W.layer("c22_1x7", 1, 22, (5, 40), 64, (1, 7), 1, (0, 3), x_dist="u11", seed=15),
]


@pytest.mark.parametrize("layer", STRIP, ids=lambda l: l["name"])
def test_strips(layer):
    check_layer(layer, cfg(2, 16), what=layer["name"])
    for layout in (1, 2, 3):
        check_layout(layer, layout, cfg(2, 16), what="%s layout %d" % (layer["name"], layout))


@pytest.mark.parametrize("kw", [dict(bk=32), dict(bk=32, split_k=3), dict(bk=16, split_k=2), dict(bk=16, split_k=2, reduce=1),
                                dict(bk=16, persist=1), dict(bk=32, persist=3, reduce=1)], ids=str)
def test_row_by_row_where_strips_fit(kw):
    """Other configurations than the strips' run as asked for: slices, persistent workgroups and any number of waves, row by row."""
    for layer in (STRIP[0], STRIP[2], STRIP[-2]):
        for wn in (1, 2, 4):
            for layout in (0, 3):
                check_layout(layer, layout, cfg(wn, **kw), what="%s %r wn%d layout %d" % (layer["name"], kw, wn, layout))


# One and two fetching waves of 1x1 layers (K-steps of 16 and 32), one and two workgroups on a compute unit (the second one's
# waves change roles) and more; patches of more than 256 positions, fetched by two waves.
ROLES = [
    (W.layer("point_490", 5, 64, 56, 128, 1, x_dist="u11", seed=20), (16, 32), {}),
    (W.layer("point_300_slices", 3, 96, (20, 40), 256, 1, x_dist="u11", seed=21), (16, 32), dict(split_k=2)),
    (W.layer("point_persist2", 4, 32, 64, 128, 1, x_dist="u11", seed=22), (16, 32), dict(persist=2)),
    (W.layer("patch_400", 4, 32, 56, 128, 3, 1, 1, x_dist="u11", seed=23), (16,), {}),
    (W.layer("patch_wide", 2, 40, (12, 70), 128, 3, 1, 2, dil=2, x_dist="u11", seed=24), (16,), {}),
]


@pytest.mark.parametrize("layer,steps,more", ROLES, ids=lambda a: a["name"] if isinstance(a, dict) and "name" in a else "")
@pytest.mark.parametrize("wn", [1, 2, 4])
def test_fetching_waves(layer, steps, more, wn):
    for bk in steps:
        check_layer(layer, cfg(wn, bk, **more), what="%s wn%d bk%d" % (layer["name"], wn, bk))


# Channels that are no multiple of 32 on the forms that pad them: 1x1 four pixels and two pixels a lane, taps, channels-last quads and
# patches, with the last group one channel short, one channel long and half full; a last pixel at the very end of the tensor.
ANY = [
    W.layer("point_c31", 2, 31, (6, 10), 70, 1, x_dist="u11", seed=30),
    W.layer("point_c97", 1, 97, (4, 33), 64, 1, x_dist="u11", seed=31),
    W.layer("taps_c48_s2", 2, 48, (9, 13), 40, 1, 2, x_dist="u11", seed=32),
    W.layer("taps_c61_5x5", 1, 61, (7, 12), 64, 5, 1, 2, x_dist="u11", seed=33),
    W.layer("patch_c50", 2, 50, 9, 96, 3, 1, 1, x_dist="u11", seed=34),
    W.layer("patch_c33_s2", 1, 33, (11, 8), 64, 3, 2, 0, x_dist="u11", seed=35),
]


@pytest.mark.parametrize("layer", ANY, ids=lambda l: l["name"])
@pytest.mark.parametrize("wn", [1, 2, 4])
def test_padded_channels(layer, wn):
    for bk in (16, 32):
        for layout in range(4):
            check_layout(layer, layout, cfg(wn, bk), what="%s wn%d bk%d layout %d" % (layer["name"], wn, bk, layout))
    check_layout(layer, 1, cfg(wn, 16, split_k=2), what="%s slices" % layer["name"])
