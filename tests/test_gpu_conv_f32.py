"""fp32 convs and dense layers on the matrix cores: each tile of the launch rule
at sizes that do not fill it - pixels, channels and reductions around the
tile edges, strides, padding, buffers aligned to one element - against the exact
oracle.  Bound per element: (terms + 3) rounding errors of 2^-24, each at most the
summed magnitudes of the terms."""

import numpy as np
import pytest
import torch

import oracle
from paper_2105_03215_amd import capi, runtime
from paper_2105_03215_amd.workloads import GraphBuilder
from parity_util import announce, term_scale_graph

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# n, c, h, w, k, (r, s), stride, pad, act, residual
CONVS = [(1, 1, 3, 3, 1, (1, 1), 1, 0, None, False), (1, 16, 7, 9, 17, (3, 3), 1, 1, "relu", False),
         (2, 27, 13, 11, 33, (5, 5), 2, 2, "relu6", False), (1, 64, 28, 28, 64, (3, 3), 1, 1, "relu", True),
         (4, 37, 30, 31, 70, (3, 3), 1, 1, "leaky", False), (6, 20, 56, 55, 40, (3, 3), 1, 1, "relu", False),
         (3, 5, 40, 41, 130, (1, 7), 1, 3, "gelu", False), (5, 129, 33, 17, 66, (1, 1), 2, 0, None, False),
         (2, 6, 20, 20, 24, (4, 8), 1, 2, None, False), (1, 3, 24, 24, 16, (7, 7), 2, 3, "relu", False)]
# rows, in, out, act, residual
DENSE = [(1, 30, 7, None, False), (3, 768, 300, "gelu", False), (30, 257, 64, "relu", True), (257, 64, 514, None, False),
         (700, 100, 600, "relu6", True), (2500, 36, 1000, "leaky", False)]


def _check(wl, terms, what):
    announce("fp32 " + what)
    ref = oracle.run_graph(wl.graph, wl.consts, wl.inputs, mode="exact")[0]
    scale = term_scale_graph(wl.graph, wl.consts, wl.inputs)[0]
    with capi.Subgraph(wl.graph, wl.consts, device=0) as sg:
        for offset in (0, 1):  # elements past an allocation's alignment
            bufs = []
            for a in wl.inputs + [np.full(ref.shape, np.nan, dtype=np.float32)]:
                t = torch.empty(a.size + offset, dtype=torch.float32, device=DEV)[offset:].view(a.shape)
                bufs.append(t.copy_(torch.from_numpy(np.ascontiguousarray(a))))
            sg.run(bufs[:-1], bufs[-1:])
            torch.cuda.synchronize()
            err = np.abs(runtime.to_host_f64(bufs[-1]) - ref)
            assert (err <= (terms + 3) * 2.0 ** -24 * np.abs(scale) + 1e-30).all(), (what, offset, float(err.max()))
        return [l["name"] for l in sg.launches()]


@pytest.mark.parametrize("case", CONVS, ids=["x".join(map(str, c[:5])) for c in CONVS])
def test_conv(case):
    n, c, h, w, k, r, stride, pad, act, res = case
    g = GraphBuilder("f32_mfma", 5000 + CONVS.index(case), dtype="f32")
    x = g.input("x", [n, c, h, w], "normal")
    g.output(g.conv(x, k, r, stride=stride, pad=pad, act=act, residual=x if res else None, name="y"))
    names = _check(g.finish(), c * r[0] * r[1], "conv %s" % (case,))
    assert names == ["conv_f32_mfma" if r[0] * r[1] <= 32 else "conv_f32_direct"], names


# many pixels and few channels: the register-blocked kernel (3x3 and 1x1) and the
# direct one (other sizes), channels that do not fill a block of four, strides, residual
FEW_CHANNELS = [(4, 3, 80, 81, 5, (3, 3), 1, 1, "relu", False), (2, 1, 301, 170, 1, (3, 3), 1, 1, None, False),
                (7, 8, 121, 119, 8, (3, 3), 2, 1, "leaky", False), (1, 5, 190, 181, 5, (1, 1), 1, 0, "relu6", True),
                (30, 4, 30, 31, 3, (1, 1), 1, 0, None, False), (3, 1, 160, 121, 3, (5, 5), 1, 2, "gelu", False),
                (4, 3, 160, 121, 2, (1, 7), 1, [0, 3, 0, 3], "relu", False)]


@pytest.mark.parametrize("case", FEW_CHANNELS, ids=["x".join(map(str, c[:5])) for c in FEW_CHANNELS])
def test_few_channels_of_many_pixels(case):
    n, c, h, w, k, r, stride, pad, act, res = case
    g = GraphBuilder("f32_few_channels", 5050 + FEW_CHANNELS.index(case), dtype="f32")
    x = g.input("x", [n, c, h, w], "normal")
    g.output(g.conv(x, k, r, stride=stride, pad=pad, act=act, residual=x if res else None, name="y"))
    assert _check(g.finish(), c * r[0] * r[1], "conv %s" % (case,)) == ["conv_f32_direct"]


@pytest.mark.parametrize("case", DENSE, ids=["x".join(map(str, c[:3])) for c in DENSE])
def test_dense(case):
    m, kin, n, act, res = case
    g = GraphBuilder("f32_mfma_dense", 5100 + DENSE.index(case), dtype="f32")
    x = g.input("x", [m, kin], "normal")
    r = g.input("r", [m, n], "normal") if res else None
    g.output(g.dense(x, n, act=act, residual=r, w_std=0.05, name="y"))
    _check(g.finish(), kin, "dense %s" % (case,))


@pytest.mark.parametrize("pad,stride", [(1, 1), (1, 2), (1, 3), ([1, 0, 0, 0], 2), ([0, 1, 0, 0], 2), ([0, 0, 1, 1], 2),
                                        ([0, 0, 1, 0], 1)], ids=str)
def test_1x1_conv_of_padded_1x1_map(pad, stride):
    """A 1x1 map with padding is no plain matrix product: outputs beside the pixel are the bias."""
    g = GraphBuilder("f32_padded_pixel", 5200, dtype="f32")
    g.output(g.conv(g.input("x", [3, 37, 1, 1], "normal"), 21, 1, stride=stride, pad=pad, act=None, name="y"))
    _check(g.finish(), 37, "padded 1x1 map %s %s" % (pad, stride))


def test_infinities_and_denormals():
    """Infinities reach the outputs that read them and no others; denormal products count."""
    g = GraphBuilder("f32_special", 5300, dtype="f32")
    x = g.input("x", [2, 40, 9, 8], "normal")
    g.output(g.conv(x, 20, 3, bn=False, act=None, name="y"))
    wl = g.finish()
    w = next(i for i, c in enumerate(wl.graph["constants"]) if len(c["shape"]) == 4)
    xs, ws = wl.inputs[0].copy(), [np.array(c) for c in wl.consts]
    xs[0, 3, 4, 4], xs[0, 7, 0, 0], xs[1, 39, 8, 7] = np.inf, -np.inf, -np.inf
    ws[w][np.abs(ws[w]) < 1e-3] = 1e-3  # (no zero times infinity)
    announce("fp32 infinities")
    ref = oracle.run_graph(wl.graph, ws, [xs], mode="exact")[0]
    with capi.Subgraph(wl.graph, ws, device=0) as sg:
        out = runtime.outputs_for(sg, DEV)
        sg.run([torch.from_numpy(xs).to(DEV)], out)
        got = runtime.to_host_f64(out[0])
        special = ~np.isfinite(ref)
        assert special.any() and not special.all()
        assert np.array_equal(got[special], ref[special])
        assert np.allclose(got[~special], ref[~special], rtol=1e-4, atol=1e-4)
        # products around 2^-136, sums of 360 of them below the normal range
        tiny = np.full_like(xs, 2.0 ** -126)
        sg2 = capi.Subgraph(wl.graph, [np.full_like(c, 2.0 ** -10) if c.ndim == 4 else np.zeros_like(c) for c in ws], device=0)
        sg2.run([torch.from_numpy(tiny).to(DEV)], out)
        torch.cuda.synchronize()
        mid = out[0].double().cpu().numpy()[:, :, 1:-1, 1:-1]
        sg2.close()
        assert (mid == 360 * 2.0 ** -136).all(), mid.flat[0] / 2.0 ** -136


def test_weights_are_not_padded_by_rows():
    """A layer of one output holds about its weights (columns are padded to 256)."""
    g = GraphBuilder("f32_one_output", 5400, dtype="f32")
    g.output(g.dense(g.input("x", [3, 5000], "normal"), 1, name="y"))
    wl = g.finish()
    with capi.Subgraph(wl.graph, wl.consts, device=0) as sg:
        assert [l["name"] for l in sg.launches()] == ["conv_f32_mfma"]
        assert sg.stats()["weight_bytes"] <= 4 * 5120 + 1024
