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
