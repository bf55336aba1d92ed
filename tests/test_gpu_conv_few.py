"""Few-pixel conv kernel (conv_few) on the GPU: every tile at the edges of its
range - one pixel, pixels and channels that do not fill a tile, reductions shorter
and longer than what the waves hold in flight, padding, strides, each epilogue -
within one bf16 ulp of the oracle, all tiles bit for bit alike, and the layers the
planner gives it."""

import pytest
import torch

import oracle
from paper_2105_03215_amd import capi, runtime
from paper_2105_03215_amd.workloads import GraphBuilder
from parity_util import announce, term_scale_graph, within_one_ulp
from test_gpu_conv_pipe import CASES as PIPE_CASES, _conv, _run

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TILES = ["f16x16", "f16x32", "f32x16", "f32x32"]
CASES = dict(PIPE_CASES)
CASES["one_pixel"] = lambda g: _conv(g, (1, 128, 1, 1), 20, 1, pad=0, act="relu")
CASES["long_reduction"] = lambda g: _conv(g, (1, 512, 3, 5), 40, 3, act=None)


@pytest.mark.parametrize("case", sorted(CASES))
def test_tiles_at_their_edges(case, monkeypatch):
    monkeypatch.setenv("BYOC_DENSE_ROWS", "0")
    g = GraphBuilder("few_" + case, 6000 + sorted(CASES).index(case))
    g.output(CASES[case](g))
    wl = g.finish()
    ref = oracle.run_graph(wl.graph, wl.consts, wl.inputs, mode="bf16io")[0]
    scale = term_scale_graph(wl.graph, wl.consts, wl.inputs)[0]
    first = None
    for tile in TILES:
        announce("conv_few %s %s" % (case, tile))
        out, names = _run(wl, tile, monkeypatch)
        assert len(names) == 1 and names[0].startswith("conv_few_" + tile[1:]), (tile, names)
        if first is None:
            ok = within_one_ulp(runtime.to_host_f64(out), ref, scale)
            assert ok.all(), "%d elements beyond one ulp" % int((~ok).sum())
            first = out
        assert torch.equal(out.view(torch.int16), first.view(torch.int16)), tile


@pytest.mark.parametrize("n,c,hw,k,r", [(1, 256, 14, 256, 3), (1, 1024, 14, 256, 1), (1, 64, 56, 64, 3), (3, 128, 9, 96, 1)])
def test_built_in_choice(n, c, hw, k, r):
    """Layers of few pixels: planned on conv_few, the same bits after tuning."""
    g = GraphBuilder("few_rule", 6100 + n + c)
    g.output(_conv(g, (n, c, hw, hw), k, r, act="relu"))
    wl = g.finish()
    announce("conv_few built-in %s" % ((n, c, hw, k, r),))
    ref = oracle.run_graph(wl.graph, wl.consts, wl.inputs, mode="bf16io")[0]
    outs = {}
    with capi.Subgraph(wl.graph, wl.consts, device=0) as sg:
        ins = runtime.inputs_for(sg, wl.inputs, DEV)
        for tuned in (False, True):
            sg.set_options(autotune=tuned)
            names = [l["name"] for l in sg.launches() if l["kind"] == "conv_mfma"]
            assert len(names) == 1 and names[0].startswith("conv_few"), names
            outs[tuned] = runtime.outputs_for(sg, DEV)[0]
            sg.run(ins, [outs[tuned]])
            torch.cuda.synchronize()
    assert torch.equal(outs[False].view(torch.int16), outs[True].view(torch.int16))
    assert within_one_ulp(runtime.to_host_f64(outs[False]), ref, term_scale_graph(wl.graph, wl.consts, wl.inputs)[0]).all()


@pytest.mark.parametrize("n,c,hw,k,r,segs,plan", [
    (1, 256, 14, 256, 3, 8, {"BYOC_CONV_SPLIT": "8"}),         # a split per wave, the last of one step
    (1, 512, 7, 512, 3, 15, {"BYOC_CONV_SPLIT": "16"}),        # two per wave, one left over
    (1, 1024, 5, 40, 1, 4, {"BYOC_CONV_SPLIT": "4"}),
    (3, 1024, 3, 256, 3, 16, {"BYOC_CONV_SPLIT": "16"}),       # more steps of a wave than it holds in flight
    (1, 64, 56, 64, 3, 4, {"BYOC_CONV_TILE": "d64x64s2t1024k4"}),  # four interleaved groups, shares of 3, 2, 2, 2 steps
    (8, 512, 8, 512, 1, 2, {"BYOC_CONV_TILE": "d64x64s3t512k2"}),  # two interleaved groups
    (1, 256, 56, 64, 1, 1, {"BYOC_CONV_SPLIT": "1"}),          # one accumulator
])
def test_sums_of_the_plan_it_replaces(n, c, hw, k, r, segs, plan, monkeypatch):
    """Bit for bit the split-K, reduction-group or plain plan that the layer would
    have, on every tile, with residual and bias."""
    g = GraphBuilder("few_plan", 6200 + c + k)
    x = g.input("x", [n, c, hw, hw])
    res = g.input("res", [n, k, hw, hw])
    g.output(g.conv(x, k, r, act="relu", residual=res, name="y"))
    wl = g.finish()

    def run(env):
        announce("conv_few against %s: %s" % (plan, env))
        with monkeypatch.context() as mp:
            for key, v in env.items():
                mp.setenv(key, v)
            with capi.Subgraph(wl.graph, wl.consts, device=0) as sg:
                out = runtime.outputs_for(sg, DEV)[0].fill_(float("nan"))
                sg.run(runtime.inputs_for(sg, wl.inputs, DEV), [out])
                torch.cuda.synchronize()
                return out.view(torch.int16), [l["name"] for l in sg.launches() if l["kind"] == "conv_mfma"][0]

    ref, name = run(plan)
    assert not name.startswith("conv_few"), name
    for tile in TILES:
        out, name = run({"BYOC_CONV_TILE": tile})
        assert name.startswith("conv_few") and "_k%d_" % segs in name, name
        assert torch.equal(out, ref), name
