"""Large-tile conv kernel (conv_pipe) on the GPU: every tile at the edges of
its range - rows and channels that do not fill a tile, one reduction stage
(fewer than the ring holds), strides, padding on every side, rectangular
kernels, each epilogue - against the oracle (within one bf16 ulp) and bit for bit
against the pipelined kernel's 64x64 tile, which sums in the same order."""

import pytest
import torch

import oracle
from paper_2105_03215_amd import capi, runtime
from paper_2105_03215_amd.workloads import GraphBuilder
from parity_util import announce, term_scale_graph, within_one_ulp

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TILES = ["p256x256s2t512", "p256x128s3t512", "p128x256s3t512", "p128x192s3t512", "p128x128s2t512", "p128x64s3t256",
         "p64x128s3t256", "p64x64s3t256"]


def _conv(g, shape, k, r, **kw):
    return g.conv(g.input("x", list(shape)), k, r, name="y", **kw)


def _dense(g, m, k, n, act):
    return g.dense(g.input("x", [m, k], "normal"), n, act=act, w_std=0.05, name="y")


CASES = {
    "one_stage_one_pixel_tile": lambda g: _conv(g, (1, 64, 5, 3), 8, 1, pad=0, act=None),
    "ragged_3x3": lambda g: _conv(g, (3, 64, 11, 9), 72, 3, act="relu"),
    "stride2": lambda g: _conv(g, (2, 128, 15, 14), 264, 3, stride=2, act="relu6"),
    "rect_leaky": lambda g: _conv(g, (2, 64, 7, 13), 200, (1, 7), act="leaky"),
    "dense_gelu": lambda g: _dense(g, 300, 192, 328, "gelu"),
    "dense_257_rows": lambda g: _dense(g, 257, 320, 256, None),
}


def _residual(g):
    x = g.input("x", [2, 64, 13, 12])
    return g.conv(x, 64, 3, act="relu", residual=x, name="y")


def _post_add(g):  # the add after the activation is folded into the conv
    x = g.input("x", [2, 64, 12, 13])
    return g.add(x, g.conv(x, 64, 3, act="leaky", name="c"), name="y")


CASES["residual"] = _residual
CASES["post_add"] = _post_add


def _run(wl, tile, monkeypatch):
    monkeypatch.setenv("BYOC_CONV_TILE", tile)
    monkeypatch.setenv("BYOC_CONV_SPLIT", "1")  # (the 64x64 tile without split-K)
    with capi.Subgraph(wl.graph, wl.consts, device=0) as sg:
        ins = runtime.inputs_for(sg, wl.inputs, DEV)
        outs = runtime.outputs_for(sg, DEV)
        outs[0].fill_(float("nan"))
        sg.run(ins, outs)
        torch.cuda.synchronize()
        return outs[0], [l["name"] for l in sg.launches() if l["kind"] == "conv_mfma"]


@pytest.mark.parametrize("case", sorted(CASES))
def test_tiles_at_their_edges(case, monkeypatch):
    monkeypatch.setenv("BYOC_DENSE_ROWS", "0")
    g = GraphBuilder("pipe_" + case, 4000 + sorted(CASES).index(case))
    g.output(CASES[case](g))
    wl = g.finish()
    ref = oracle.run_graph(wl.graph, wl.consts, wl.inputs, mode="bf16io")[0]
    scale = term_scale_graph(wl.graph, wl.consts, wl.inputs)[0]
    first, _ = _run(wl, "d64x64s2t256k1", monkeypatch)
    ok = within_one_ulp(runtime.to_host_f64(first), ref, scale)
    assert ok.all(), "%d elements beyond one ulp" % int((~ok).sum())
    for tile in TILES:
        announce("conv_pipe %s %s" % (case, tile))
        out, names = _run(wl, tile, monkeypatch)
        assert len(names) == 1 and names[0].startswith("conv_pipe_" + tile[1:].split("s")[0]), (tile, names)
        assert torch.equal(out.view(torch.int16), first.view(torch.int16)), tile


def test_other_convs_keep_their_kernel(monkeypatch):
    """A conv whose channels are not whole 64-channel slices is not conv_pipe's."""
    g = GraphBuilder("pipe_unaligned", 4100)
    g.output(_conv(g, (2, 40, 10, 11), 48, 3, act="relu"))
    wl = g.finish()
    out, names = _run(wl, "p128x128s2t512", monkeypatch)
    assert not any(n.startswith("conv_pipe") for n in names), names
    ref = oracle.run_graph(wl.graph, wl.consts, wl.inputs, mode="bf16io")[0]
    assert within_one_ulp(runtime.to_host_f64(out), ref, term_scale_graph(wl.graph, wl.consts, wl.inputs)[0]).all()


@pytest.mark.parametrize("n,c,hw,k,r", [(20, 256, 28, 256, 3), (9, 64, 56, 256, 1), (8, 128, 32, 256, 3)])
def test_built_in_choice_over_many_tiles(n, c, hw, k, r, monkeypatch):
    """Layers with more 64x64 tiles than CUs: the modelled choice against the 64x64 tile."""
    g = GraphBuilder("pipe_rule", 4200 + n)
    g.output(_conv(g, (n, c, hw, hw), k, r, act="relu"))
    wl = g.finish()
    first, _ = _run(wl, "d64x64s2t256k1", monkeypatch)
    monkeypatch.delenv("BYOC_CONV_TILE")
    monkeypatch.delenv("BYOC_CONV_SPLIT")
    announce("built-in choice %s" % ((n, c, hw, k, r),))
    with capi.Subgraph(wl.graph, wl.consts, device=0) as sg:
        outs = runtime.outputs_for(sg, DEV)
        outs[0].fill_(float("nan"))
        sg.run(runtime.inputs_for(sg, wl.inputs, DEV), outs)
        torch.cuda.synchronize()
        names = [l["name"] for l in sg.launches() if l["kind"] == "conv_mfma"]
    assert names[0].startswith(("conv_pipe", "conv_halo")), names
    a, b = runtime.to_host_f64(outs[0]), runtime.to_host_f64(first)
    if names[0].startswith("conv_pipe") and (r == 1 or c < 256):
        assert (a == b).all()
    else:  # another summation order: one bf16 ulp, and the fp32 rounding of sums of O(1) terms
        assert (abs(a - b) <= 2.0 ** -7 * abs(b) + 1e-4).all()


@pytest.mark.parametrize("n,c,hw,k", [(8, 128, 32, 256), (16, 192, 14, 512), (10, 64, 32, 256)])
def test_sums_tap_by_tap_under_256_channels(n, c, hw, k, monkeypatch):
    """3x3 layers of fewer channels than the windowed kernel's rule asks for keep the
    64x64 tile's bits, whatever kernel has the least modelled time."""
    g = GraphBuilder("pipe_tap_order", 4400 + c)
    g.output(_conv(g, (n, c, hw, hw), k, 3, act="leaky"))
    wl = g.finish()
    first, _ = _run(wl, "d64x64s2t256k1", monkeypatch)
    monkeypatch.delenv("BYOC_CONV_TILE")
    monkeypatch.delenv("BYOC_CONV_SPLIT")
    with capi.Subgraph(wl.graph, wl.consts, device=0) as sg:
        ins = runtime.inputs_for(sg, wl.inputs, DEV)
        for tuned in (False, True):
            announce("tap order %s tuned %s" % ((n, c, hw, k), tuned))
            sg.set_options(autotune=tuned)
            out = runtime.outputs_for(sg, DEV)[0].fill_(float("nan"))
            sg.run(ins, [out])
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), first.view(torch.int16)), [l["name"] for l in sg.launches()]


def test_windowed_kernels_order_is_shared():
    """A 3x3 layer of the windowed kernel's class that conv_pipe takes over
    keeps the windowed kernel's bits, before and after tuning."""
    g = GraphBuilder("pipe_slice_major", 4300)
    g.output(_conv(g, (24, 256, 28, 28), 320, 3, act="relu"))
    wl = g.finish()
    outs = {}
    for name, env in (("built-in", {}), ("windowed", {"BYOC_CONV_HALO": "1"})):
        with pytest.MonkeyPatch.context() as mp:
            for k, v in env.items():
                mp.setenv(k, v)
            announce("summation order " + name)
            with capi.Subgraph(wl.graph, wl.consts, device=0) as sg:
                names = [l["name"] for l in sg.launches() if l["kind"] == "conv_mfma"]
                assert names[0].startswith("conv_halo" if env else "conv_pipe"), names
                ins = runtime.inputs_for(sg, wl.inputs, DEV)
                for tuned in (False, True):
                    sg.set_options(autotune=tuned)
                    outs[name, tuned] = runtime.outputs_for(sg, DEV)[0]
                    sg.run(ins, [outs[name, tuned]])
                    torch.cuda.synchronize()
    first = outs["built-in", False].view(torch.int16)
    for key, o in outs.items():
        assert torch.equal(o.view(torch.int16), first), key


I8_CASES = [
    # n, c, h, w, k, r, stride, pad, zx, act, residual, output scale
    (2, 128, 5, 7, 24, 1, 1, 0, 3, None, False, 0.023),
    (2, 128, 14, 13, 200, 3, 1, 1, 37, "relu", True, 0.023),     # border correction, residual
    (3, 256, 11, 9, 136, 3, 2, 1, -100, "relu6", False, 0.023),
    (1, 128, 13, 12, 264, 3, 1, 1, -40, "leaky", True, 0.023),
    (2, 128, 9, 9, 72, 1, 1, 0, 9, None, True, 1e-6),            # rescaled terms saturate at +-2^20
    (2, 128, 9, 9, 72, 1, 1, 0, 9, "relu", False, 1e-6),
]


@pytest.mark.parametrize("case", I8_CASES, ids=[str(i) for i in range(len(I8_CASES))])
def test_int8_tiles_exact(case, monkeypatch):
    """int8 codes: every conv_pipe tile, the implicit-GEMM kernel and the built-in
    choice give the oracle's codes."""
    import numpy as np
    from oracle import quant as oq
    from test_gpu_quant import _conv_graph, _run as run_i8
    g, consts, inputs = _conv_graph(*case[:11], seed=70 + I8_CASES.index(case))
    g["nodes"][0]["quant"]["scale"] = case[11]
    ref = oq.run_quantized_graph(g, consts, inputs)[0].astype(np.float64)
    for tile in [None, "64x64s3w4"] + ["p" + t[1:].replace("t256", "w4").replace("t512", "w8") for t in TILES[1:]]:
        announce("int8 conv_pipe %s %s" % (case, tile))
        if tile:
            monkeypatch.setenv("BYOC_I8_TILE", tile)
        got, launches = run_i8(g, consts, inputs)
        name = [l["name"] for l in launches if l["kind"] == "conv_i8"][0]
        assert not (tile and tile[0] == "p") or name.startswith("conv_i8_pipe_" + tile[1:].split("s")[0]), name
        assert np.array_equal(got[0], ref), (tile, name)
