"""Two-way pipelining: half of a layer's batch runs on the weights that were packed for the whole of it.  CPU: the order in which the split
members take the reduction, and the size of the packed weights, are those of the whole also where the whole is too large for padded
channels and a half by itself would not be.  GPU: such a layer."""
import os
import subprocess

import pytest

from paper_2008_04567_amd import binding as B
from tests.parity import torch_dev

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "wpk_internal.h"
using namespace wpk;
int main()
{
    srand(23);
    long checked = 0, alone = 0;
    for (int it = 0; it < 40000; ++it) {
        auto pick = [](int lo, int hi) { return lo + rand() % (hi - lo + 1); };
        const int r = 1 + 2 * pick(0, 3), c = pick(20, 130);
        wpk_conv_desc d = {pick(2, 40), c, pick(r, 3000), pick(r, 3000), pick(1, 300), r, r, 2, 2, r / 2, r / 2, 1, 1, WPK_F32, rand() % 4};
        const double bytes = 4.0 * d.n * c * d.h * d.w;
        if (bytes < 1.2e9 || bytes > 2.1e9) continue;
        Problem whole;
        if (make_problem(&d, &whole) != WPK_OK || !whole.tiled_ok) continue;
        for (const int images : {(d.n + 1) / 2, d.n / 2}) {
            Problem part, fresh;
            wpk_conv_desc p = d;
            p.n = images;
            if (make_part(whole, images, &part) != WPK_OK || make_problem(&p, &fresh) != WPK_OK) return 3;
            ++checked;
            alone += split_taps(fresh) != split_taps(whole);
            if (split_taps(part) != split_taps(whole) || split_rows(part) != split_rows(whole) || part.d.n != images ||
                part.x_elems != fresh.x_elems || part.y_elems != fresh.y_elems || part.M != fresh.M) {
                printf("n %d of %d, c %d, %d x %d, r %d, layout %d: %d, %d\n", images, d.n, c, d.h, d.w, r, d.layout, split_taps(part),
                       split_taps(whole));
                return 1;
            }
            for (int bk = 16; bk <= 32; bk += 16) {
                const wpk_conv_config cfg = {64, 64, bk, 1, 2, 1, 1, 0, 1, 0};
                if (halo_positions(part, cfg) != halo_positions(whole, cfg)) return 2;
            }
        }
    }
    printf("%ld %ld\n", checked, alone);
    return checked > 500 && alone > 100 ? 0 : 4;
}
"""


def test_halves_take_the_order_of_the_whole(tmp_path):
    src, exe = tmp_path / "half.cpp", tmp_path / "half"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_2008_04567_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", csrc, str(src),
                    os.path.join(csrc, "wpk_host.cpp"), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, (res.returncode, res.stdout)


@pytest.mark.gpu
@pytest.mark.parametrize("layout", [B.NCHW, B.NHWC])
def test_a_pipelined_plan_of_a_large_layer(layout):
    """43 channels of 2100 x 2100 pixels, two images: 64 channels of both would not fit 2 GiB, of one they do.  The pipelined plan against
    one launch of the same configuration: the same products in the same order, so the same bits."""
    torch, dev = torch_dev()
    hw, c, k = 2100, 43, 40
    desc = B.make_desc(n=2, c=c, h=hw, w=hw, k=k, r=1, s=1, stride_h=8, stride_w=8, pad_h=0, pad_w=0, dil_h=1, dil_w=1, layout=layout)
    P, Q = B.conv_out_shape(desc)
    g = torch.Generator(device=dev).manual_seed(5)
    x = torch.rand((2, hw, hw, c) if layout else (2, c, hw, hw), generator=g, device=dev) - 0.5
    w = torch.rand((k, c, 1, 1), generator=g, device=dev) - 0.5
    shape = (2, P, Q, k) if layout else (2, k, P, Q)
    plain, halves = torch.empty(shape, device=dev), torch.full(shape, float("nan"), device=dev)
    cfg = B.make_config(64, 64, 32, 1, 2, stages=1)
    plan = B.Plan([desc])
    plan.set_layer_config(0, cfg)
    plan.set_weights(0, w)
    plan.run_layer(0, x, plain)
    plan.set_pipeline(2)
    plan.set_layer_config(0, cfg)
    plan.run_layer(0, x, halves)
    torch.cuda.synchronize()
    assert torch.equal(plain, halves)
    read = (x.permute(0, 3, 1, 2) if layout else x)[:, :, ::8, ::8].reshape(2, c, P * Q).double()
    want = torch.matmul(w.double().view(k, c), read).view(2, k, P, Q)
    got = (plain.permute(0, 3, 1, 2) if layout else plain).double()
    assert ((got - want).norm() / want.norm()).item() < 5e-7
