"""Where a layer without a tuned configuration goes (CPU): layers whose measured times decide between the split and the tiled
members, or between numbers of slices; and every default is a legal one."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "wpk_internal.h"
using namespace wpk;
struct Case { wpk_conv_desc d; int split, wn, slices_min, slices_max, persist; };  // (wn 0: any)
#define L(n, c, h, w, k, r, s, st, pad, dil, lay) {n, c, h, w, k, r, s, st, st, pad, pad, dil, dil, WPK_F32, lay}
// (times: tiled, split as it was by waves per SIMD alone; us)
static const Case cases[] = {
    // split members gain here
    {L(16, 64, 56, 56, 64, 3, 3, 1, 1, 1, 0), 1, 2, 1, 1, 3},
    {L(16, 128, 28, 28, 128, 3, 3, 1, 1, 1, 0), 1, 4, 1, 1, 0},
    {L(16, 256, 14, 14, 256, 3, 3, 1, 1, 1, 0), 1, 4, 2, 2, 0},
    {L(16, 64, 56, 56, 256, 1, 1, 1, 0, 1, 0), 1, 2, 1, 1, 3},
    {L(16, 256, 56, 56, 128, 1, 1, 1, 0, 1, 0), 1, 2, 1, 1, 3},
    {L(16, 128, 56, 56, 128, 3, 3, 2, 1, 1, 3), 1, 4, 1, 1, 0},
    {L(4, 72, 45, 61, 100, 3, 3, 1, 2, 2, 0), 1, 4, 1, 1, 0},
    {L(4, 576, 13, 13, 224, 3, 3, 1, 0, 1, 2), 1, 4, 2, 24, 0},        // 81 (atomics into channels-last), 22
    // small layers: start and meeting are most of it
    {L(10, 192, 23, 23, 171, 1, 1, 1, 0, 1, 0), 0, 0, 1, 1, 0},        // 8.8, 16.7
    {L(2, 43, 40, 40, 96, 3, 3, 2, 1, 1, 0), 0, 0, 1, 24, 0},          // 9.8, 12.7
    {L(3, 320, 34, 34, 24, 3, 3, 1, 0, 1, 0), 0, 0, 1, 24, 0},         // 16.3, 32.7
    // one workgroup of two waves per compute unit and a few over: slices
    {L(24, 832, 10, 10, 448, 3, 3, 1, 1, 1, 3), 1, 0, 2, 6, 0},        // 136, 183; 87 in 3 of 2 waves
    {L(47, 704, 12, 12, 137, 3, 3, 1, 1, 1, 0), 1, 0, 2, 6, 0},        // 124, 145; 78 in 3 of 2 waves
    {L(4, 96, 69, 69, 64, 5, 5, 1, 0, 1, 1), 1, 0, 2, 6, 0},           // 45, 60
    // two to two and a half tiles per compute unit, taps: one workgroup of four waves each and the rest dealt out; not where two of the
    // waves have no channels, 1x1 filters or few steps
    {L(24, 160, 56, 56, 128, 5, 5, 2, 2, 1, 0), 1, 4, 1, 1, 1},
    {L(48, 32, 56, 56, 64, 3, 3, 2, 1, 1, 0), 1, 2, 1, 1, 0},          // 20.1 by waves per SIMD, 30.7 dealt out
    {L(12, 64, 57, 57, 64, 3, 3, 1, 1, 2, 0), 1, 2, 1, 1, 0},          // 24.7, 42.7
    {L(5, 224, 101, 101, 192, 1, 1, 2, 0, 1, 0), 1, 2, 1, 1, 0},       // 16.9, 24.4
    {L(64, 32, 17, 64, 100, 3, 3, 2, 1, 1, 0), 1, 4, 1, 1, 0},         // 19.8, 22.6
    {L(31, 208, 13, 44, 96, 3, 3, 1, 1, 1, 0), 1, 1, 1, 1, 0},         // (channels of three 32-wide workgroups) 37.0, 43.5
    {L(9, 32, 31, 31, 320, 5, 5, 1, 0, 1, 0), 1, 2, 1, 1, 0},          // (128-wide tiles of 320 channels) 28.8, 34.0
    // channels-last, and patches beyond four tiles per compute unit: whole tiles where steps are few, most of a round is left over, or slices of
    // four waves are estimated to be a quarter faster
    {L(5, 160, 49, 49, 160, 1, 1, 1, 0, 1, 3), 1, 2, 1, 1, 0},         // 11.3, 15.2 dealt out
    {L(1, 256, 93, 97, 209, 5, 5, 1, 2, 1, 3), 1, 4, 5, 5, 0},
    {L(61, 37, 43, 43, 138, 3, 3, 1, 1, 1, 0), 1, 2, 1, 1, 0},         // 99.6, 117.8
    {L(9, 64, 78, 65, 96, 3, 3, 1, 1, 1, 2), 1, 4, 1, 1, 0},           // 39.2, 43.6
    {L(6, 64, 65, 73, 174, 3, 3, 1, 1, 1, 1), 1, 2, 1, 1, 2},          // (four steps)
    // strips: where little of them is padding
    {L(16, 3, 224, 224, 64, 7, 7, 2, 3, 1, 0), 1, 2, 1, 1, 0},         // 44.3, 28.4
    {L(32, 3, 112, 112, 64, 5, 5, 1, 2, 1, 3), 1, 2, 1, 1, 0},
    {L(32, 6, 112, 112, 256, 3, 3, 2, 1, 1, 0), 0, 0, 1, 1, 0},        // 46.7, 66.0
    {L(32, 3, 112, 112, 32, 4, 4, 1, 2, 1, 0), 0, 0, 1, 1, 0},         // 25.8, 29.7
    {L(32, 6, 160, 160, 96, 1, 7, 1, 0, 1, 1), 0, 0, 1, 1, 0},         // 157, 183
    // padded channels, pixel by pixel: not for 1x1 filters of few steps and many tiles
    {L(27, 44, 64, 64, 384, 1, 1, 2, 0, 1, 0), 0, 0, 1, 1, 0},         // 19.6, 28.4
    {L(33, 87, 51, 51, 512, 1, 1, 1, 0, 1, 0), 0, 0, 1, 1, 0},         // 135, 145
    {L(2, 23, 82, 82, 480, 5, 5, 1, 2, 1, 0), 0, 0, 1, 1, 0},          // 73.5, 79.4
    {L(20, 320 + 1, 45, 45, 256, 1, 1, 1, 0, 1, 0), 1, 4, 1, 1, 0},    // (eleven steps)
    {L(8, 329, 35, 35, 256, 1, 1, 1, 0, 1, 3), 1, 2, 1, 1, 2},         // (channels-last) 31.6, 23.2
    // the same up to 32 channels, with few steps, or with many waves per SIMD
    {L(43, 168, 43, 22, 32, 5, 5, 2, 0, 1, 0), 0, 0, 7, 7, 0},         // 36.8, 51.4
    {L(11, 51, 37, 11, 29, 7, 7, 1, 3, 1, 2), 1, 1, 14, 14, 0},        // (atomics into channels-last) 62.2, 22.1
    {L(3, 97, 75, 75, 32, 7, 7, 1, 3, 1, 0), 1, 1, 3, 3, 0},           // (tiles dealt out) 118, 68.4
    {L(6, 28, 79, 79, 736, 3, 1, 1, 1, 1, 2), 0, 0, 1, 1, 0},          // 68.7, 82.7
    // 1x1, up to two tiles: two fetching waves, but not for few channels, many slices or a second round
    {L(16, 512, 28, 28, 128, 1, 1, 1, 0, 1, 0), 1, 4, 1, 1, 0},        // 16.3 with one, 12.6
    {L(20, 896, 10, 10, 128, 1, 1, 1, 0, 1, 0), 1, 2, 4, 4, 0},        // 13.8, 16.6 in 8 slices
    {L(10, 992, 28, 28, 32, 1, 1, 1, 0, 1, 0), 1, 1, 5, 5, 0},         // 14.8, 16.1
    {L(12, 1344, 14, 14, 96, 1, 1, 1, 0, 1, 0), 1, 1, 5, 5, 0},        // 15.2, 16.5
    {L(7, 1440, 16, 16, 768, 1, 1, 1, 0, 1, 0), 1, 4, 1, 1, 0},        // 29.5, 33.1 in 3 slices
    // single steps: nothing to deal out
    {L(21, 32, 26, 26, 864, 1, 1, 1, 0, 1, 0), 1, 2, 1, 1, 0},         // 21.5, 45.7 dealt out, 23.3 whole
};
int main()
{
    for (const Case &t : cases) {
        Problem pr;
        wpk_conv_config c;
        if (make_problem(&t.d, &pr) != WPK_OK) return 3;
        default_config(pr, 256, &c);
        const bool split = split_member(c);
        if (split != (t.split != 0) || c.split_k < t.slices_min || c.split_k > t.slices_max ||
            (split && ((t.wn && c.wn != t.wn) || persistent_of(pr, c, 256) != t.persist))) {
            printf("n %d c %d %dx%d k %d r %d: %d x %d x %d, %d x %d, split_k %d, persist %d\n", t.d.n, t.d.c, t.d.h, t.d.w, t.d.k,
                   t.d.r, c.bm, c.bn, c.bk, c.wm, c.wn, c.split_k, c.persist);
            return 1;
        }
    }
    // Waves that fetch patches: two where that costs no workgroup, but for four workgroups of one multiplying wave (39.6 us with one, 49.5).
    static const struct { wpk_conv_desc d; int wn, producers; } fetch[] = {
        {L(7, 182, 45, 38, 160, 3, 3, 1, 1, 1, 0), 1, 1},
        {L(7, 182, 45, 38, 160, 3, 3, 1, 1, 1, 0), 4, 2},
        {L(9, 247, 11, 39, 32, 3, 3, 1, 1, 1, 1), 1, 2},     // (one workgroup per compute unit) 14.2 with two, 14.7
        {L(4, 64, 80, 80, 64, 3, 3, 1, 1, 1, 0), 1, 2},      // (three fit)
        {L(4, 64, 80, 80, 64, 3, 3, 1, 1, 1, 0), 2, 2},
        {L(16, 256, 14, 14, 256, 3, 3, 1, 1, 1, 0), 2, 1},   // (four with one, three with two)
    };
    for (const auto &t : fetch) {
        Problem pr;
        const wpk_conv_config c = {64, 32 * t.wn, 16, 1, t.wn, 1, 1, 0, 1, 0};
        if (make_problem(&t.d, &pr) != WPK_OK || halo_positions(pr, c) == 0) return 3;
        if (split_producers(pr, c, 256) != t.producers) {
            printf("c %d %dx%d, %d waves: %d fetch\n", t.d.c, t.d.h, t.d.w, t.wn, split_producers(pr, c, 256));
            return 1;
        }
    }
    // Wave-split members: how slices meet follows from what the launch has to do (us, workspace and atomics, in a pass without an
    // epilogue unless stated).
    static const struct { wpk_conv_desc d; int plain, fused; } meet[] = {  // (slices; below zero: atomics)
        {L(1, 512, 7, 7, 512, 3, 3, 1, 1, 1, 0), -8, 8},      // 9.3, 8.0; with an epilogue 9.5, 13.9
        {L(1, 256, 14, 14, 256, 3, 3, 1, 1, 1, 0), -4, 4},    // 8.2, 7.2
        {L(1, 544, 12, 12, 32, 5, 5, 1, 2, 1, 0), -24, 20},   // 9.8, 6.8
        {L(1, 416, 17, 31, 32, 3, 3, 1, 1, 1, 0), -14, 8},    // (17 tiles: with an epilogue 8.1 in 8 slices, 8.6 in 11)
        {L(1, 512, 28, 28, 128, 1, 1, 1, 0, 1, 0), 1, 1},     // 5.5; in two slices 6.2
        {L(1, 512, 7, 7, 512, 3, 3, 1, 1, 1, 2), 8, 8},       // (channels-last: 12.1 and 18 for such layers)
    };
    for (const auto &t : meet) {
        Problem pr;
        wpk_conv_config c, f;
        if (make_problem(&t.d, &pr) != WPK_OK) return 3;
        default_config(pr, 256, &c, true);
        default_config(pr, 256, &f, false);
        if (c.bm != kWaveSplitBm || f.bm != kWaveSplitBm || (c.reduce ? -c.split_k : c.split_k) != t.plain ||
            (f.reduce ? -f.split_k : f.split_k) != t.fused) {
            printf("c %d %dx%d k %d r %d layout %d: %d slices (reduce %d), fused %d (%d)\n", t.d.c, t.d.h, t.d.w, t.d.k, t.d.r,
                   t.d.layout, c.split_k, c.reduce, f.split_k, f.reduce);
            return 1;
        }
    }
    srand(5);
    long split = 0, all = 0;
    for (int it = 0; it < 60000; ++it) {
        auto pick = [](int lo, int hi) { return lo + rand() % (hi - lo + 1); };
        wpk_conv_desc d = {1 << rand() % 7, rand() % 2 ? 32 * pick(1, 32) : pick(1, 300), pick(1, 112), pick(1, 112), pick(1, 1024),
                           pick(1, 7), pick(1, 7), pick(1, 3), pick(1, 3), pick(0, 4), pick(0, 4), pick(1, 2), pick(1, 2),
                           WPK_F32, rand() % 4};
        if (rand() % 2) d.r = d.s = rand() % 2 ? 3 : 1;
        Problem pr;
        wpk_conv_config c;
        if (make_problem(&d, &pr) != WPK_OK || !pr.tiled_ok) continue;
        default_config(pr, rand() % 8 ? 256 : pick(1, 304), &c);
        ++all;
        split += split_member(c);
        if (!legal_for(pr, c)) {
            printf("n %d c %d %dx%d k %d r %d s %d: illegal default\n", d.n, d.c, d.h, d.w, d.k, d.r, d.s);
            return 2;
        }
    }
    printf("%ld of %ld\n", split, all);
    return split > 1000 && all > 20000 ? 0 : 4;
}
"""

# The configurations that same_launch puts together do make one launch: what the kernel and its grid depend on is equal, the
# one that stands for the others is legal, and the search space is so much smaller.
SAME = r"""
#include <stdio.h>
#include <stdlib.h>
#include <set>
#include "wpk_internal.h"
using namespace wpk;
int main()
{
    srand(3);
    long points = 0, launches = 0, strips = 0, rows = 0;
    for (int it = 0; it < 90; ++it) {
        auto pick = [](int lo, int hi) { return lo + rand() % (hi - lo + 1); };
        const int r = rand() % 2 ? 3 : pick(1, 5);
        wpk_conv_desc d = {pick(1, 16), it >= 60 ? pick(1, 7) : rand() % 2 ? 32 * pick(1, 20) : pick(1, 300), pick(r, 60), pick(r, 60), pick(1, 600), r, r,
                           1, 1, r / 2, r / 2, 1, 1, WPK_F32, rand() % 4};
        Problem pr;
        if (make_problem(&d, &pr) != WPK_OK || !pr.tiled_ok) continue;
        std::set<int> ids;
        const wpk_conv_config strip = {64, 64, 16, 1, 2, 1, 1, 0, 1, 0};
        const int strip_id = wpk_config_id(&strip);
        for (int id = 0;; ++id) {
            wpk_conv_config c;
            if (wpk_config_from_id(id, &c) != WPK_OK) break;
            if (!legal_for(pr, c)) continue;
            const wpk_conv_config s = same_launch(pr, c, 256), s2 = same_launch(pr, s, 256);
            if (wpk_config_id(&s) != wpk_config_id(&s2) || !legal_for(pr, s)) return 1;
            if (!split_member(c)) {
                if (wpk_config_id(&s) != id) return 2;
                continue;
            }
            ++points;
            ids.insert(wpk_config_id(&s));
            // (strips are one launch, whose workgroups follow from the layer)
            if (runs_strip(pr, c) != runs_strip(pr, s)) return 5;
            if (runs_strip(pr, c)) {
                ++strips;
                if (wpk_config_id(&s) != strip_id) return 6;
                continue;
            }
            rows += strip_depths(pr) > 0;
            const Reduction a = reduction_of(pr, c), b = reduction_of(pr, s);
            const int pa = (a.steps + c.split_k - 1) / c.split_k, pb = (b.steps + s.split_k - 1) / s.split_k;
            const FixupNeed fa = fixup_need(pr, c, 256), fb = fixup_need(pr, s, 256);
            if (s.wn != c.wn || s.bn != c.bn || halo_positions(pr, c) != halo_positions(pr, s) || a.steps != b.steps ||
                a.rows != b.rows || pa != pb || persistent_of(pr, c, 256) != persistent_of(pr, s, 256) ||
                s.xcd_remap != c.xcd_remap || fa.bytes != fb.bytes || fa.maxc != fb.maxc) {
                printf("c %d r %d: bk %d split %d persist %d reduce %d stages %d\n", d.c, r, c.bk, c.split_k, c.persist, c.reduce, c.stages);
                return 3;
            }
        }
        launches += ids.size();
    }
    printf("%ld points, %ld launches, %ld in strips, %ld row by row instead\n", points, launches, strips, rows);
    return points > 2 * launches && launches > 500 && strips > 50 && rows > 1000 ? 0 : 4;
}
"""


def run_program(tmp_path, text):
    src, exe = tmp_path / "default.cpp", tmp_path / "default"
    src.write_text(text)
    csrc = os.path.join(ROOT, "paper_2008_04567_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "include"), "-I", csrc, str(src),
                    os.path.join(csrc, "wpk_host.cpp"), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True)


def test_configurations_put_together_make_one_launch(tmp_path):
    res = run_program(tmp_path, SAME)
    assert res.returncode == 0, (res.returncode, res.stdout)


def test_defaults_follow_the_measured_times_and_are_legal(tmp_path):
    res = run_program(tmp_path, PROGRAM)
    assert res.returncode == 0, (res.returncode, res.stdout)
