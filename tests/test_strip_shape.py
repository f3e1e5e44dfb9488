"""Strips of the split members (CPU): what strip_shape chooses against every access of the kernel -- the columns and rows of a
pixel's octets inside the strip's LDS, every output row in one strip, the weights' rows inside the packed ones."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "wpk_internal.h"
using namespace wpk;
int main()
{
    srand(11);
    long taken = 0, refused = 0, edge = 0, units = 0;
    auto pick = [](int lo, int hi) { return lo + rand() % (hi - lo + 1); };
    for (int it = 0; it < 20000; ++it) {
        wpk_conv_desc d = {pick(1, 9), pick(1, 7), pick(1, 70), pick(1, 260), pick(1, 300), pick(1, 11), pick(1, 10), pick(1, 3), pick(1, 3),
                           pick(0, 3), pick(0, 3), pick(1, 2), rand() % 4 ? 1 : 2, WPK_F32, pick(0, 3)};
        Problem pr;
        if (make_problem(&d, &pr) != WPK_OK) continue;
        const int depths = strip_depths(pr);
        if (depths == 0) { ++refused; continue; }
        ++taken;
        const StripShape s = strip_shape(pr, 256), fewer = strip_shape(pr, 16);
        units += s.rows != fewer.rows || s.per_group != fewer.per_group;
        // a prepared layer's is the one that it was prepared with, and no launch prices another
        Problem once = pr;
        prepare_strip(&once, 16);
        if (memcmp(&once.strip, &fewer, sizeof s) || pr.strip.depths) return 3;
        const StripShape kept = strip_shape(once, 256);
        if (memcmp(&kept, &fewer, sizeof s)) return 3;
        const int in_rows = (s.rows - 1) * d.stride_h + (d.r - 1) * d.dil_h + 1, line = 3 * s.pairs * 4;
        const int per_image = (pr.P + s.rows - 1) / s.rows, groups = (d.k + 32 * s.waves_c - 1) / (32 * s.waves_c);
        bool bad = s.depths != depths || 2 * depths < d.c * d.r || d.s > 8 || s.rows < 1 || s.lds > 78 * 1024 ||
                   s.lds < d.c * in_rows * line || per_image * s.rows < pr.P || (per_image - 1) * s.rows >= pr.P ||
                   s.per_group < 1 || s.per_group > groups || split_rows(pr) != depths * 16 + pr.CRSpad ||
                   groups * 32 * s.waves_c > pr.Kpad;
        // the last byte that the octet of any pixel, filter row and channel reaches
        const int q = (pr.Q - 1) * d.stride_w, words = d.stride_w % 2 ? 5 : 4;
        bad = bad || (q >> 1) + words > s.pairs;
        const int row = (d.c - 1) * in_rows + (s.rows - 1) * d.stride_h + (d.r - 1) * d.dil_h;
        bad = bad || (row + 1) * line > s.lds;
        edge += (q >> 1) + words == s.pairs;
        // every column that a tap of the last pixel reads is one that the lanes fetch
        bad = bad || q + d.s > 2 * s.pairs;
        const wpk_conv_config c = {64, 64, 16, 1, 2, 1, 1, 0, 1, 0}, e = {64, 128, 32, 1, 4, 1, 1, 2, 1, 0};
        bad = bad || !runs_strip(pr, c) || runs_strip(pr, e) || fixup_need(pr, c, 256).bytes != 0 || reduction_of(pr, c).steps != 1 ||
              reduction_of(pr, e).steps != (pr.CRS + 31) / 32;
        if (bad) {
            printf("n %d c %d h %d w %d k %d r %d s %d stride %d %d: rows %d pairs %d lds %d\n", d.n, d.c, d.h, d.w, d.k, d.r, d.s,
                   d.stride_h, d.stride_w, s.rows, s.pairs, s.lds);
            return 1;
        }
    }
    // As many strips as a launch of 256 threads per workgroup has room for (2^32 threads), and one more: row by row.
    const wpk_conv_config one = {64, 64, 16, 1, 2, 1, 1, 0, 1, 0};
    for (const int rows : {1, 3})
        for (const int more : {0, 1, 1000000}) {
            const wpk_conv_desc d = {0xffffff / rows + more, 3, rows, 1, 1, 7, 7, 1, 1, 3, 3, 1, 1, WPK_F32, 0};
            Problem pr;
            if (make_problem(&d, &pr) != WPK_OK || !strip_depths(pr) || !legal_for(pr, one)) return 4;
            if (runs_strip(pr, one) != (more == 0)) return 5;
            wpk_conv_config c;
            default_config(pr, 256, &c);
            if (more && runs_strip(pr, c)) return 6;
            if (more) continue;
            const StripShape s = strip_shape(pr, 256);
            const int64_t groups = (int64_t)d.n * ((pr.P + s.rows - 1) / s.rows);
            if (s.rows < 1 || groups * 256 > 0xffffffffll) return 7;
        }
    printf("%ld %ld %ld %ld\n", taken, refused, edge, units);
    return taken > 2000 && refused > 2000 && edge > 10 && units > 100 ? 0 : 2;
}
"""

# One order of the reduction per layer: what fits a strip is not ordered by taps (the two overlapped at 22 channels of one filter row, which
# padding to 32 lengthens by less than half), and only what is ordered by taps is fetched four pixels at a time or in patches.
ORDERS = r"""
#include <stdio.h>
#include "wpk_internal.h"
using namespace wpk;
int main()
{
    long strips = 0, taps = 0;
    for (int c = 1; c <= 40; ++c)
        for (int r = 1; r <= 7; ++r)
            for (int s = 1; s <= 9; ++s)
                for (int v = 0; v < 16; ++v) {
                    const int stride = 1 + v % 2, pad = v / 2 % 2;
                    wpk_conv_desc d = {4, c, 20, 28, 64, r, s, stride, stride, pad, pad, 1, 1, WPK_F32, v / 4};
                    Problem pr;
                    if (make_problem(&d, &pr) != WPK_OK) continue;
                    const wpk_conv_config cfg = {64, 64, 16, 1, 2, 1, 1, 0, 1, 0};
                    const bool strip = strip_depths(pr) > 0;
                    strips += strip;
                    taps += split_taps(pr);
                    if (strip && (split_taps(pr) || split_point(pr) || halo_positions(pr, cfg) > 0)) {
                        printf("c %d, %d x %d, stride %d, layout %d: strip and taps\n", c, r, s, stride, d.layout);
                        return 1;
                    }
                }
    printf("%ld %ld\n", strips, taps);
    return strips > 3000 && taps > 3000 ? 0 : 2;
}
"""


def run_program(tmp_path, text):
    src, exe = tmp_path / "strip.cpp", tmp_path / "strip"
    src.write_text(text)
    csrc = os.path.join(ROOT, "paper_2008_04567_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I" + csrc, "-I" + os.path.join(ROOT, "include"), str(src),
                    os.path.join(csrc, "wpk_host.cpp"), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)


def test_strips_hold_what_is_read(tmp_path):
    res = run_program(tmp_path, PROGRAM)
    assert res.returncode == 0, res.stdout


def test_no_layer_has_two_orders(tmp_path):
    res = run_program(tmp_path, ORDERS)
    assert res.returncode == 0, res.stdout
