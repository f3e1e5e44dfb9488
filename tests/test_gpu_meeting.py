"""A plan's layers run with one configuration without an epilogue and with another with one, where slices of a small layer's
reduction meet by other means: one plan run plainly, with a residual, with bias and rectifier, and plainly again, layer by
layer and as a pass, over y of any content, eagerly and captured.  Bar: 1e-4 * sum|x*w| against the CPU oracle, as everywhere."""
import numpy as np
import pytest

from oracle import conv as oc
from paper_2008_04567_amd import binding as B
from paper_2008_04567_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu

LAYERS = [W.layer("meet_512", 1, 512, (7, 7), 512, 3, 1, 1, x_dist="u11", w_dist="u11", seed=501),
          W.layer("meet_37", 1, 256, (9, 5), 37, 3, 1, 1, x_dist="u11", w_dist="u11", seed=502)]


def _reference(layer, bias=None, res=None, relu=False):
    x, w = W.make_inputs(layer)
    return oc.conv2d_fused(oc.shape_from_layer(layer), x, w, bias=bias, residual=res, relu=relu)


def test_one_plan_with_and_without_an_epilogue():
    import torch
    plan = B.Plan([B.make_desc(l) for l in LAYERS])
    st = torch.cuda.current_stream()
    xs, ys, res, bias = [], [], [], []
    for i, l in enumerate(LAYERS):
        assert plan.layer_config(i).reduce == 1 and plan.layer_config(i).split_k >= 4
        x, w = W.make_inputs(l)
        xs.append(PT.to_dev(x))
        plan.set_weights(i, PT.to_dev(w), st)
        torch.cuda.synchronize()
        shape = (l["n"], l["k"]) + B.conv_out_shape(B.make_desc(l))
        ys.append(torch.full(shape, float("nan"), device="cuda"))
        rng = np.random.default_rng(i)
        res.append(rng.uniform(-2, 2, shape).astype(np.float32))
        bias.append(rng.uniform(-1, 1, l["k"]).astype(np.float32))
    rd = [PT.to_dev(r) for r in res]
    bd = [PT.to_dev(b) for b in bias]
    xa, ya = plan.pointer_arrays(xs, ys)
    ra = plan.residual_array(rd)

    def check(what, **kw):
        torch.cuda.synchronize()
        for i, l in enumerate(LAYERS):
            y_ref, d_ref = _reference(l, **{k: v[i] if isinstance(v, list) else v for k, v in kw.items()})
            PT.assert_close(ys[i].cpu().numpy(), y_ref, d_ref, "%s, layer %d" % (what, i))
            ys[i].fill_(float("nan"))

    def by_layer(residuals):
        for i in range(len(LAYERS)):
            plan.run_layer_fused(i, xs[i], residuals[i], ys[i], st)

    none = plan.residual_array([None] * len(LAYERS))
    for turn in range(2):
        plan.run(xa, ya, st)
        check("plain pass")
        by_layer([None, None])
        check("plain layers")
        plan.run_fused(xa, ra, ya, st)
        check("pass with residuals", res=res)
        by_layer(rd)
        check("layers with residuals", res=res)
        for i in range(len(LAYERS)):
            plan.set_epilogue(i, bias=bd[i], relu=True, stream=st)
            assert plan.layer_config(i).reduce == 0
        plan.run_fused(xa, none, ya, st)
        check("pass with bias and rectifier", bias=bias, relu=True)
        plan.run_fused(xa, ra, ya, st)
        check("pass with everything", bias=bias, res=res, relu=True)
        for i in range(len(LAYERS)):
            plan.set_epilogue(i, bias=None, relu=False, stream=st)

    # captured: both ways in one graph, replayed between eager passes
    s = torch.cuda.Stream()
    s.wait_stream(st)
    plain = [torch.empty_like(y) for y in ys]
    xb, yb = plan.pointer_arrays(xs, plain)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        cs = torch.cuda.current_stream()
        plan.run(xb, yb, cs)
        plan.run_fused(xa, ra, ya, cs)
    for turn in range(3):
        for y in plain:
            y.fill_(float("nan"))
        g.replay()
        check("replay %d with residuals" % turn, res=res)
        for i, l in enumerate(LAYERS):
            y_ref, d_ref = _reference(l)
            PT.assert_close(plain[i].cpu().numpy(), y_ref, d_ref, "replay %d, layer %d" % (turn, i))
        plan.run(xa, ya, st)
        check("pass between replays")
    plan.destroy()
