"""The split members' forms that the tests on values name (CPU): every layer there takes the one that it is listed under."""
import os
import subprocess

from paper_2008_04567_amd import binding as B
from tests.test_gpu_split import FORMS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "wpk_internal.h"
using namespace wpk;
int main()
{
    wpk_conv_desc d;
    int bk;
    d.dtype = WPK_F32;
    while (scanf("%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d", &d.n, &d.c, &d.h, &d.w, &d.k, &d.r, &d.s, &d.stride_h, &d.stride_w, &d.pad_h,
                 &d.pad_w, &d.dil_h, &d.dil_w, &d.layout, &bk) == 15) {
        Problem pr;
        const wpk_conv_config c = {64, 64, bk, 1, 2, 1, 1, 0, 1, 0};
        if (make_problem(&d, &pr) != WPK_OK || !legal_for(pr, c)) return 1;
        const bool patch = halo_positions(pr, c) > 0, taps = split_taps(pr);
        const char *form = runs_strip(pr, c) ? "strip" : patch ? (pr.xl ? "patch_quads" : "patch") : split_point(pr) ? "point"
                           : taps ? (pr.xl ? "quads" : "taps") : "rows";
        printf("%s %d %d\n", form, taps && d.c % 32 != 0, split_producers(pr, c, 256));
    }
    return 0;
}
"""


def test_layers_take_the_forms_they_are_listed_under(tmp_path):
    src, exe = tmp_path / "forms.cpp", tmp_path / "forms"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_2008_04567_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I" + csrc, "-I" + os.path.join(ROOT, "include"), str(src),
                    os.path.join(csrc, "wpk_host.cpp"), "-o", str(exe)], check=True)
    lines = []
    for layer, layout, bk in FORMS.values():
        d = B.make_desc(layer, layout=layout)
        lines.append(" ".join(str(getattr(d, f)) for f in ("n", "c", "h", "w", "k", "r", "s", "stride_h", "stride_w", "pad_h", "pad_w",
                                                           "dil_h", "dil_w", "layout")) + " %d" % bk)
    res = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True)
    assert res.returncode == 0
    took = [line.split() for line in res.stdout.splitlines()]
    assert len(took) == len(FORMS)
    for name, (form, padded, producers) in zip(FORMS, took):
        parts = name.split("_")
        wanted = "_".join(p for p in parts if p in ("patch", "point", "quads", "rows", "strip", "taps"))
        assert form == wanted, (name, form)
        odd = parts[-1].startswith("c") and wanted not in ("rows", "strip")
        assert int(padded) == odd, (name, padded)
        if wanted == "point":
            assert int(producers) == (1 if FORMS[name][2] == 16 else 2), name
    # (with and without padding, each that pads)
    assert {f for f, p, _ in took if p == "1"} == {"patch", "patch_quads", "point", "quads", "taps"} == {f for f, p, _ in took if p == "0"} - {"rows", "strip"}
