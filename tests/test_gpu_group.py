"""Independent convs in one launch (engine.cpp, group_launches) on the GPU: the
branches of a block - 1x1, 3x3, 1x7 and 7x1 convs of different sizes, reductions of
whole and of ragged stages, slices of a concatenation, a residual and two outputs -
give the bits of the separate launches, eagerly, replayed as a graph and with the
intermediates in the static scratch."""

import pytest
import torch

from paper_2105_03215_amd import capi, profiling, runtime
from paper_2105_03215_amd.workloads import GraphBuilder
from parity_util import announce

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _branches(g, n, c, hw, widths):
    """One conv per width, kernel sizes in turn; 2nd and 3rd continue by another conv."""
    x = g.input("x", [n, c, hw, hw])
    kernels = [(1, 0), (3, 1), (1, 0), (5, 2), (1, 0), (3, 1)]
    ends = []
    for i, k in enumerate(widths):
        r, pad = kernels[i % len(kernels)]
        y = g.conv(x, k, r, pad=pad, act="relu" if i % 2 else None)
        if i in (1, 2):
            y = g.conv(y, 32 + 8 * i, 3, pad=1, act="relu")
        ends.append(y)
    return ends


CASES = {
    # (batch, channels, map, branch widths): few-pixel tiles, one and several images
    "one_image": (1, 64, 7, [64, 40, 64, 8]),
    "unequal": (1, 256, 9, [256, 8, 16]),
    "six_branches": (2, 64, 6, [32, 32, 32, 32, 32, 32]),
    # 64x64 tiles: whole stages, ragged stages, a mix of the two
    "tiles64": (8, 512, 17, [192, 160, 128, 64]),
    "ragged": (8, 520, 17, [160, 128, 192, 160]),
    "most_tiles": (24, 128, 17, [128, 128, 64]),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_same_bits_as_apart(case, monkeypatch):
    n, c, hw, widths = CASES[case]
    g = GraphBuilder("group_" + case, 7000 + sorted(CASES).index(case))
    ends = _branches(g, n, c, hw, widths)
    g.output(g.concat(ends[:-1]) if len(ends) > 2 else ends[0])
    g.output(ends[-1])
    wl = g.finish()
    outs, order = {}, {}
    for group in ("0", "1"):
        monkeypatch.setenv("BYOC_GROUP", group)
        with capi.Subgraph(wl.graph, wl.consts, device=0) as sg:
            ins = runtime.inputs_for(sg, wl.inputs, DEV)
            for mode in ("eager", "replay", "static", "profiled", "tuned"):
                announce("group %s %s %s" % (case, group, mode))
                out = runtime.outputs_for(sg, DEV)
                if mode == "tuned":
                    sg.set_options(autotune=True)
                else:
                    sg.set_options(graph_replay=mode == "replay")
                if mode == "profiled":
                    sg.profile_begin(2)
                for _ in range(3):
                    for o in out:
                        o.fill_(float("nan"))
                    (sg.run_static if mode == "static" else sg.run)(ins, out)
                    torch.cuda.synchronize()
                if mode == "profiled":
                    ms, runs = sg.profile_end()
                    launches = sg.launches()
                    assert runs == 2 and len(ms) == len(launches) and min(ms) > 0
                    # a group's time is divided by FLOPs: equal rates tell its members
                    rates = [l["flops"] / t for l, t in zip(launches, ms)]
                    if group == "1":
                        assert any(a > 0 and abs(a - b) < 1e-5 * a for a, b in zip(rates, rates[1:])), rates
                outs[group, mode] = [o.view(torch.int16).cpu() for o in out]
            order[group] = [l["node"] for l in sg.launches()]
    assert sorted(order["0"]) == sorted(order["1"])
    for key, got in outs.items():
        for a, b in zip(got, outs["0", "eager"]):
            assert torch.equal(a, b), key


def test_members_name_their_group():
    """Entries of one device launch say so, and count once."""
    g = GraphBuilder("group_names", 7100)
    for e in _branches(g, 1, 256, 9, [256, 128, 64]):
        g.output(e)
    wl = g.finish()
    announce("group names")
    with capi.Subgraph(wl.graph, wl.consts, device=0) as sg:
        names = [l["name"] for l in sg.launches()]
    heads = [i for i, n in enumerate(names) if "_g1/" in n]
    assert heads, names
    for i in heads:
        size = int(names[i].rsplit("/", 1)[1])
        assert size > 1 and [n.rsplit("_g", 1)[1] for n in names[i:i + size]] == ["%d/%d" % (k + 1, size) for k in range(size)]
    members = sum(int(names[i].rsplit("/", 1)[1]) for i in heads)
    assert sum("_g" in n for n in names) == members
    assert profiling.dispatches([{"name": n} for n in names]) == len(names) - members + len(heads)


@pytest.mark.parametrize("branches", [3, 12])
def test_order_that_fits_the_static_scratch_stays(branches):
    """Branches of an 8 MiB map each: side by side, twelve of them need more than the
    static scratch, one after the other they do not, so their order stays and run_static works."""
    g = GraphBuilder("group_scratch", 7200)
    x = g.input("x", [1, 64, 256, 256])
    for _ in range(branches):
        g.output(g.conv(g.conv(x, 64, 1, act="relu"), 64, 1, stride=8, pad=0, act=None))
    wl = g.finish()
    announce("group order and the static scratch, %d branches" % branches)
    with capi.Subgraph(wl.graph, wl.consts, device=0) as sg:
        assert sg.stats()["arena_bytes"] <= 64 << 20
        assert any("_g1/" in l["name"] for l in sg.launches()) == (branches == 3), [l["name"] for l in sg.launches()]
        ins = runtime.inputs_for(sg, wl.inputs, DEV)
        outs = [runtime.outputs_for(sg, DEV) for _ in range(2)]
        sg.run(ins, outs[0])
        sg.run_static(ins, outs[1])
        torch.cuda.synchronize()
    for a, b in zip(*outs):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
