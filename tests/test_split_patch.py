"""The patches of the split members (CPU): the bound the host allocates by, halo_positions, against every tap of every
pixel of every tile, over filters, strides, dilations, paddings and images of odd sizes."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "wpk_internal.h"
using namespace wpk;
int main()
{
    srand(7);
    long tiles = 0, refused = 0, tight = 0;
    for (int it = 0; it < 6000; ++it) {
        auto pick = [](int lo, int hi) { return lo + rand() % (hi - lo + 1); };
        wpk_conv_desc d = {pick(1, 6), 32, pick(1, 40), pick(1, 60), 64, 3, 3, pick(1, 3), pick(1, 3), pick(0, 4), pick(0, 4),
                           pick(1, 3), pick(1, 3), WPK_F32, rand() % 2 ? WPK_NHWC : WPK_NCHW};
        if (rand() % 2) d.stride_h = d.stride_w = d.dil_h = d.dil_w = d.pad_h = d.pad_w = 1;
        Problem pr;
        if (make_problem(&d, &pr) != WPK_OK) continue;
        const wpk_conv_config cfg = {64, 64, 16, 1, 2, 1, 1, 0, 1, 0};
        const int bound = halo_positions(pr, cfg);
        if (bound == 0) { ++refused; continue; }
        for (long m0 = 0; m0 < pr.M; m0 += 64, ++tiles) {
            const long m1 = m0 + 63 < pr.M ? m0 + 63 : pr.M - 1, PQ = (long)pr.P * pr.Q;
            auto at = [&](long m, int &n, int &p, int &q) { n = m / PQ; p = m % PQ / pr.Q; q = m % pr.Q; };
            int n, p, q;
            at(m0, n, p, q);
            const int j0 = patch_first(n, p, q, d.stride_h, d.stride_w, d.pad_h, d.pad_w, d.h, d.w);
            at(m1, n, p, q);
            const int j1 = patch_last(n, p, q, d.stride_h, d.stride_w, d.pad_h, d.pad_w, d.dil_h, d.dil_w, d.h, d.w);
            bool bad = j0 < 0 || j1 >= d.n * d.h * d.w || j1 - j0 + 1 > bound;
            tight += j1 - j0 + 1 == bound;
            for (long m = m0; m <= m1; ++m) {
                at(m, n, p, q);
                for (int r = 0; r < 3; ++r)
                    for (int s = 0; s < 3; ++s) {
                        const int ih = p * d.stride_h - d.pad_h + r * d.dil_h, iw = q * d.stride_w - d.pad_w + s * d.dil_w;
                        if (ih < 0 || ih >= d.h || iw < 0 || iw >= d.w) continue;
                        const int j = (n * d.h + ih) * d.w + iw;
                        bad = bad || j < j0 || j > j1;
                    }
            }
            if (bad) {
                printf("n %d h %d w %d stride %d %d pad %d %d dil %d %d tile %ld: positions %d..%d, bound %d\n", d.n, d.h, d.w,
                       d.stride_h, d.stride_w, d.pad_h, d.pad_w, d.dil_h, d.dil_w, m0 / 64, j0, j1, bound);
                return 1;
            }
        }
    }
    printf("%ld %ld %ld\n", tiles, refused, tight);
    return tiles > 10000 && refused > 100 && tight > 100 ? 0 : 2;
}
"""


# Channels of the last chunk, in layers that the split members take and whose x comes close to 2 GiB (N = 1): every channel's
# plane lies in x, also where 16 planes would not fit 32 bits.
CHANNELS = r"""
#include <stdio.h>
#include "wpk_internal.h"
using namespace wpk;
int main()
{
    const int shapes[][3] = {{11, 300000, 146}, {11, 330000, 146}, {12, 300000, 147}, {23, 150000, 150}, {45, 80000, 140},
                             {41, 90000, 142}, {200, 18000, 144}, {13, 40, 40}};
    int wide = 0, checked = 0;
    for (const auto &s : shapes) {
        wpk_conv_desc d = {1, s[0], s[1], s[2], 8, 3, 3, 1, 1, 1, 1, 1, 1, WPK_F32, WPK_NCHW};
        Problem pr;
        const wpk_conv_config cfg = {64, 32, 16, 1, 1, 1, 1, 0, 1, 0};
        if (make_problem(&d, &pr) != WPK_OK || !legal_for(pr, cfg) || halo_positions(pr, cfg) == 0) continue;
        ++checked;
        const long long plane = (long long)d.h * d.w * 4;
        for (int ch = 0; ch < reduction_of(pr, cfg).steps * 16; ++ch) {
            const long long at = patch_channel_at(ch, d.c, (int)plane);
            wide += ch * plane > 0x7fffffff;
            if (at != (ch < d.c ? ch : d.c - 1) * plane || at + plane > pr.x_elems * 4) {
                printf("c %d h %d w %d channel %d: %lld\n", d.c, d.h, d.w, ch, at);
                return 1;
            }
        }
    }
    printf("%d %d\n", checked, wide);
    return checked >= 6 && wide > 3 ? 0 : 2;
}
"""


def run_program(tmp_path, text):
    src, exe = tmp_path / "patch.cpp", tmp_path / "patch"
    src.write_text(text)
    csrc = os.path.join(ROOT, "paper_2008_04567_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", csrc, str(src),
                    os.path.join(csrc, "wpk_host.cpp"), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True)


def test_channels_of_the_last_chunk_lie_in_x(tmp_path):
    res = run_program(tmp_path, CHANNELS)
    assert res.returncode == 0, (res.returncode, res.stdout)


def test_every_tap_lies_in_the_patch_and_the_patch_within_its_bound(tmp_path):
    res = run_program(tmp_path, PROGRAM)
    assert res.returncode == 0, res.stdout
