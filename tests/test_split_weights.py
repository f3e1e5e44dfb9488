"""Where the split members fetch their weights (CPU): every fetch of every wave, those ahead of the end of the reduction
too, lies in the packed weights, and the weights of a depth that is multiplied are those of that depth."""
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
    srand(11);
    long fetches = 0, clamped = 0, patches = 0;
    for (int it = 0; it < 4000; ++it) {
        auto pick = [](int lo, int hi) { return lo + rand() % (hi - lo + 1); };
        const int rs[4] = {1, 3, 3, 5}, r = rs[rand() % 4];
        const int c = rand() % 2 ? 32 * pick(1, 8) : pick(1, 200);
        wpk_conv_desc d = {pick(1, 4), c, pick(r, 30), pick(r, 30), rand() % 8 ? pick(1, 400) : 2048, r, r, 1, 1,
                           r / 2, r / 2, 1, 1, WPK_F32, rand() % 2 ? WPK_NHWC : WPK_NCHW};
        Problem pr;
        if (make_problem(&d, &pr) != WPK_OK) continue;
        for (int bk = 16; bk <= 32; bk += 16) {
            const wpk_conv_config cfg = {64, 64, bk, 1, 2, 1, 1, 0, 1, 0};
            const bool patch = halo_positions(pr, cfg) > 0;
            const int NT = patch ? 9 : 2, steps = reduction_of(pr, cfg).steps;
            patches += patch;
            const uint32_t depth_bytes = pr.Kpad / 32 * 3072u;
            const uint32_t w_bytes = (uint32_t)(split_rows(pr) * pr.Kpad * kSplitWeightBytes);
            if (w_bytes % depth_bytes) return 3;
            for (int block = 0; block < pr.Kpad / 32; block += 3)
                // the walk of a wave through steps [0, steps): two depths asked for before the first, then each time
                // two ahead of the one multiplied, those of the step after from that step's first depth on
                for (long t = 0; t < (long)steps * NT + 2; ++t, ++fetches) {
                    const int step = (int)(t / NT), depth = split_depth(patch, step, (int)(t % NT));
                    const uint32_t at = split_weights_at(patch, block * 3072u, step, steps, depth_bytes) +
                                        (uint32_t)(t % NT) * split_depth(patch, 0, 1) * depth_bytes;
                    const bool used = t < (long)steps * NT;
                    if ((uint64_t)at + 3072 > w_bytes || (used && at != (uint64_t)depth * depth_bytes + block * 3072u)) {
                        printf("c %d k %d r %d bk %d depth %d: fetched at %u of %u\n", c, d.k, r, bk, depth, at, w_bytes);
                        return 1;
                    }
                    clamped += (uint64_t)depth * depth_bytes + block * 3072u != at;
                }
        }
    }
    printf("%ld %ld %ld\n", fetches, clamped, patches);
    return fetches > 100000 && clamped > 500 && patches > 100 ? 0 : 2;
}
"""


def test_every_fetch_of_weights_lies_in_the_packed_weights(tmp_path):
    src, exe = tmp_path / "weights.cpp", tmp_path / "weights"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_2008_04567_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", csrc, str(src),
                    os.path.join(csrc, "wpk_host.cpp"), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, (res.returncode, res.stdout)
