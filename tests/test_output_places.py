"""Where outputs and residuals lie (CPU): the offsets of the buffer accesses that tiles leave by.  A lane of an output gets that
output's offset; a lane past the last pixel or the last channel gets one past the tensor, aligned and not wrapped round, so that
nothing is read or written through it."""
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
    // few channels of large images too: a channel's offset past the last one exceeds 32 bits there
    struct { int N, K, PQ; } fixed[] = {{1, 16, 16}, {1, 8, 5}, {1, 16, 4200 * 4200}, {1, 1, 536870911}, {1, 24, 33}, {3, 37, 117}};
    srand(5);
    long there = 0, pixels = 0, channels = 0;
    for (int it = 0; it < 400; ++it) {
        auto pick = [](int lo, int hi) { return lo + rand() % (hi - lo + 1); };
        const int N = it < 6 ? fixed[it].N : pick(1, 5), K = it < 6 ? fixed[it].K : it % 2 ? pick(1, 8) * 8 : pick(1, 200);
        const int PQ = it < 6 ? fixed[it].PQ : pick(1, 400);
        const uint64_t bytes = (uint64_t)N * K * PQ * 4;
        if (bytes > (uint64_t)kMaxTiledBytes) return 3;
        const int M = N * PQ, first = M > 700 ? M - 700 : 0;
        for (int yl = 0; yl < 2; ++yl)
            for (int m = first; m < (M + 31) / 32 * 32; ++m)
                for (int k = 0; k < (K + 63) / 64 * 64; k += 4) {
                    const int n = m / PQ, pq = m % PQ;
                    const uint32_t ch4 = yl ? 4 : (uint32_t)PQ * 4, place = output_place(m, M, n, pq, k, K, PQ, yl != 0);
                    for (int dk = 0; dk < 64; dk += dk % 4 == 3 ? 5 : 1) {  // the channels of a lane's registers
                        // a register of a 32-channel block that has them all, or of one that does not
                        const bool whole = (k + dk) / 32 * 32 + 32 <= K;
                        const OutputAccess a = whole ? output_access<true>(place, k, dk, K, ch4)
                                                     : output_access<false>(place, k, dk, K, ch4);
                        const uint64_t at = (uint64_t)a.lane + a.uniform;
                        bool ok = true;
                        if (at != output_at(place, k, dk, K, ch4)) ok = whole && m >= M && at < (1ull << 32);
                        // (whether the uniform part counts in the range check or not)
                        if (m >= M || k + dk >= K) ok = ok && a.lane >= bytes && a.uniform < bytes;
                        if (!ok) return 4;
                        if (m < M && k + dk < K) {
                            ok = at == 4 * (yl ? (uint64_t)m * K + k + dk : ((uint64_t)n * K + k + dk) * PQ + pq);
                            ++there;
                        } else {
                            ok = at >= bytes && at + 4 <= (1ull << 32) && at % 4 == 0;
                            ++(m >= M ? pixels : channels);
                        }
                        if (!ok) {
                            printf("N %d K %d PQ %d yl %d pixel %d channel %d + %d: %llu of %llu\n", N, K, PQ, yl, m, k, dk,
                                   (unsigned long long)at, (unsigned long long)bytes);
                            return 1;
                        }
                    }
                }
    }
    printf("%ld %ld %ld\n", there, pixels, channels);
    return there > 100000 && pixels > 10000 && channels > 10000 ? 0 : 2;
}
"""


def test_lanes_of_no_output_reach_nothing(tmp_path):
    src, exe = tmp_path / "places.cpp", tmp_path / "places"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_2008_04567_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", csrc, str(src),
                    os.path.join(csrc, "wpk_host.cpp"), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, (res.returncode, res.stdout)
