"""The work a program has this library do, as measurable cases.

A case is one offloaded function (a serialized subgraph) on one engine:
``prepare`` makes the function's weights and inputs from a seed, builds the
engine and allocates the output buffers, as a program does once; ``run`` is
one invocation, ``Subgraph.run`` on torch's current stream.

The listed cases stand for the library's three compute types (f32, bf16,
int8), its operator families (conv, dense, depthwise, pooling, residual and
post-activation adds, concatenation) and its range of sizes, from one small
composite to the batch-32 classifier; ``draw`` takes further sizes of the same
kinds.
"""

import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2105_03215_amd import capi, quantize, workloads

DEVICE = "cuda:0"

_STAGES = [(64, 64, 1, 56), (256, 128, 2, 56), (512, 256, 2, 28), (1024, 512, 2, 14)]  # ResNet-50: in, mid, stride, hw


def listed():
    return [
        # the smallest call: one fp32 conv + bias + ReLU composite; latency and
        # host work only
        {"name": "conv_f32_single", "kind": "conv_f32", "n": 1, "c": 16, "h": 32, "w": 32, "k": 32, "r": 3, "stride": 1},
        # a float32 function of ordinary size: a basic residual block at batch 8
        {"name": "block_f32_b8", "kind": "basic_block", "dtype": "f32", "n": 8, "c": 128, "h": 28, "w": 28},
        # one bf16 residual block for one image (latency)
        {"name": "basic_block_b1", "kind": "basic_block", "dtype": "bf16", "n": 1, "c": 64, "h": 56, "w": 56},
        # the classifier serving one float32 image, replayed as a HIP graph
        {"name": "resnet50_b1", "kind": "resnet50", "n": 1, "hw": 224, "variant": "v1", "input": "f32", "autotune": True,
         "graph_replay": True},
        # the throughput benchmark: the classifier at batch 32, tuned once
        {"name": "resnet50_b32", "kind": "resnet50", "n": 32, "hw": 224, "variant": "v1", "input": "bf16",
         "autotune": True, "graph_replay": False},
        # a partially quantized region: the 14x14 stage of the classifier, batch 32
        {"name": "int8_stage3_b32", "kind": "int8_stage", "stage": 3, "n": 32, "blocks": 3},
        # mobile network region: two inverted residual blocks (stride 2, then a residual one), batch 16
        {"name": "inverted_b16", "kind": "inverted", "n": 16, "hw": 28, "cin": 32, "c": 64, "t": 6, "stride": 2, "blocks": 2},
        # transformer feed-forward layer, 8 x 128 tokens
        {"name": "ffn_1024", "kind": "ffn", "dtype": "bf16", "rows": 1024, "hidden": 768, "ffn": 3072},
        # the same layer on a long batch, 16 x 512 tokens
        {"name": "ffn_8192", "kind": "ffn", "dtype": "bf16", "rows": 8192, "hidden": 768, "ffn": 3072},
        # the large-GEMM convolutions: third stage of a VGG network with its pool, batch 16
        {"name": "vgg_stage_b16", "kind": "vgg_stage", "n": 16, "cin": 128, "c": 256, "h": 56, "w": 56, "convs": 4},
        # odd maps, 1x7 / 7x1 kernels, average pool and concatenation, batch 8
        {"name": "inception_b8", "kind": "inception", "n": 8, "h": 17, "w": 17, "cin": 768, "c7": 160},
        # leaky ReLU and adds after the activation: a stride-2 stage of a DarkNet network, batch 8
        {"name": "darknet_stage_b8", "kind": "darknet", "n": 8, "cin": 128, "hw": 64, "blocks": 3},
    ]


# a drawn case does no more work than these (the largest listed one, and the
# largest listed one of the float32 graphs)
_MOST_FLOPS = 2.4e11
_MOST_FLOPS_F32 = 3.6e9


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_one(rng):
    kind = rng.choice(["conv_f32", "basic_block", "basic_block", "resnet50", "int8_stage", "int8_stage", "inverted",
                       "inverted", "ffn", "ffn", "ffn", "vgg_stage", "vgg_stage", "inception", "darknet"])
    if kind == "conv_f32":
        h = _log_int(rng, 8, 64)
        return {"kind": kind, "n": _log_int(rng, 1, 16), "c": _log_int(rng, 3, 160), "h": h,
                "w": max(8, h + rng.randint(-3, 3)), "k": _log_int(rng, 8, 200), "r": rng.choice([1, 3, 3, 5]),
                "stride": rng.choice([1, 1, 2])}
    if kind == "basic_block":
        h = _log_int(rng, 7, 64)
        return {"kind": kind, "dtype": rng.choice(["f32", "bf16"]), "n": _log_int(rng, 1, 32),
                "c": rng.choice([24, 40, 64, 96, 128, 200, 256]), "h": h, "w": max(7, h + rng.randint(-3, 3))}
    if kind == "resnet50":
        return {"kind": kind, "n": _log_int(rng, 1, 24), "hw": rng.choice([160, 192, 224]),
                "variant": rng.choice(["v1", "v1b"]), "input": rng.choice(["bf16", "f32"]), "autotune": True,
                "graph_replay": rng.choice([False, True])}
    if kind == "int8_stage":
        return {"kind": kind, "stage": rng.randint(1, 4), "n": _log_int(rng, 1, 40), "blocks": rng.randint(1, 4)}
    if kind == "inverted":
        cin, c, hw = rng.choice([(16, 24, 112), (24, 32, 56), (32, 64, 28), (64, 96, 14), (96, 160, 14)])
        return {"kind": kind, "n": _log_int(rng, 1, 32), "hw": hw + rng.randint(-3, 3), "cin": cin, "c": c, "t": 6,
                "stride": rng.choice([1, 2]), "blocks": rng.randint(1, 3)}
    if kind == "ffn":
        return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "bf16", "f32"]), "rows": _log_int(rng, 1, 10000),
                "hidden": rng.choice([192, 256, 384, 512, 768, 1000, 1024]),
                "ffn": rng.choice([768, 1024, 1500, 2048, 3072, 4096])}
    if kind == "vgg_stage":
        h = _log_int(rng, 14, 112)
        return {"kind": kind, "n": _log_int(rng, 1, 24), "cin": rng.choice([64, 128, 256, 512]),
                "c": rng.choice([64, 128, 256, 320, 512]), "h": h, "w": h + rng.randint(-3, 3),
                "convs": rng.randint(1, 4)}
    if kind == "inception":
        h = rng.randint(8, 20)
        return {"kind": kind, "n": _log_int(rng, 1, 24), "h": h, "w": h + rng.randint(-1, 1), "cin": 768,
                "c7": rng.choice([128, 160, 192])}
    return {"kind": kind, "n": _log_int(rng, 1, 16), "cin": rng.choice([64, 128, 256, 512]),
            "hw": rng.choice([14, 16, 26, 32, 52, 64]), "blocks": rng.randint(1, 4)}


def draw(rng):
    while True:
        case = _draw_one(rng)
        if work(case)["flops"] <= (_MOST_FLOPS_F32 if _is_f32(case) else _MOST_FLOPS):
            return case


def _is_f32(case):
    return case["kind"] == "conv_f32" or case.get("dtype") == "f32"


# ---- the functions -----------------------------------------------------------

def _bottleneck(g, x, mid, out, stride, project, stride_on, name):
    s1, s3 = (stride, 1) if stride_on == "1x1" else (1, stride)
    sc = g.conv(x, out, 1, stride=stride, pad=0, act=None, name=name + ".down") if project else x
    a = g.conv(x, mid, 1, stride=s1, pad=0, act="relu", name=name + ".a")
    b = g.conv(a, mid, 3, stride=s3, pad=1, act="relu", name=name + ".b")
    return g.conv(b, out, 1, pad=0, act="relu", residual=sc, name=name + ".c")


def _build(case, seed):
    """The case's function: a workloads.GraphBuilder with its graph, constants and inputs, all drawn from the seed."""
    kind = case["kind"]
    dtype = "f32" if _is_f32(case) else "bf16"
    g = workloads.GraphBuilder(kind, 1000 + int(seed), dtype=dtype)
    if kind == "conv_f32":
        x = g.input("x", [case["n"], case["c"], case["h"], case["w"]])
        y = g.conv(x, case["k"], case["r"], stride=case["stride"], act="relu", bn=False, w_std=0.1, b_std=0.01)
    elif kind == "basic_block":
        x = g.input("x", [case["n"], case["c"], case["h"], case["w"]])
        y = g.conv(g.conv(x, case["c"], 3), case["c"], 3, residual=x)
    elif kind == "resnet50":
        x = g.input("x", [case["n"], 3, case["hw"], case["hw"]], dtype=case["input"])
        y = g.max_pool(g.conv(x, 64, 7, stride=2, pad=3, name="stem"), 3, 2, 1, name="pool")
        for si, (mid, blocks, stride) in enumerate([(64, 3, 1), (128, 4, 2), (256, 6, 2), (512, 3, 2)]):
            for bi in range(blocks):
                y = _bottleneck(g, y, mid, 4 * mid, stride if bi == 0 else 1, bi == 0,
                                "1x1" if case["variant"] == "v1" else "3x3", "s%d.b%d" % (si + 1, bi))
        y = g.dense(g.global_avg_pool(y, name="gap"), 1000, name="fc")
    elif kind == "int8_stage":
        cin, mid, stride, hw = _STAGES[case["stage"] - 1]
        y = g.input("x", [case["n"], cin, hw, hw])
        for bi in range(case["blocks"]):
            y = _bottleneck(g, y, mid, 4 * mid, stride if bi == 0 else 1, bi == 0, "1x1", "b%d" % bi)
    elif kind == "inverted":
        y = g.input("x", [case["n"], case["cin"], case["hw"], case["hw"]])
        cin = case["cin"]
        for bi in range(case["blocks"]):
            stride = case["stride"] if bi == 0 else 1
            h = g.conv(y, cin * case["t"], 1, pad=0, act="relu6", name="b%d.expand" % bi)
            h = g.conv(h, cin * case["t"], 3, stride=stride, pad=1, groups=cin * case["t"], act="relu6",
                       name="b%d.dw" % bi)
            y = g.conv(h, case["c"], 1, pad=0, act=None, residual=y if stride == 1 and cin == case["c"] else None,
                       name="b%d.project" % bi)
            cin = case["c"]
    elif kind == "ffn":
        x = g.input("x", [case["rows"], case["hidden"]], "normal")
        h = g.dense(x, case["ffn"], act="gelu", w_std=0.02, b_std=0.02, name="ffn1")
        y = g.dense(h, case["hidden"], residual=x, w_std=0.02, b_std=0.02, name="ffn2")
    elif kind == "vgg_stage":
        y = g.input("x", [case["n"], case["cin"], case["h"], case["w"]])
        for i in range(case["convs"]):
            y = g.conv(y, case["c"], 3, name="conv%d" % i)
        y = g.max_pool(y, 2, 2, 0, name="pool")
    elif kind == "inception":
        c7 = case["c7"]
        x = g.input("x", [case["n"], case["cin"], case["h"], case["w"]])
        b1 = g.conv(x, 192, 1, name="b1")
        b7 = g.conv(g.conv(g.conv(x, c7, 1, name="b7a"), c7, (1, 7), name="b7b"), 192, (7, 1), name="b7c")
        bd = g.conv(x, c7, 1, name="bda")
        for i, (ks, k) in enumerate([((7, 1), c7), ((1, 7), c7), ((7, 1), c7), ((1, 7), 192)]):
            bd = g.conv(bd, k, ks, name="bd%d" % i)
        bp = g.conv(g.avg_pool(x, 3, 1, 1, name="avg"), 192, 1, name="bp")
        y = g.concat([b1, b7, bd, bp], name="cat")
    elif kind == "darknet":
        c = 2 * case["cin"]
        x = g.input("x", [case["n"], case["cin"], case["hw"], case["hw"]])
        y = g.conv(x, c, 3, stride=2, act="leaky", name="down")
        for b in range(case["blocks"]):
            h = g.conv(y, c // 2, 1, act="leaky", name="b%d.a" % b)
            h = g.conv(h, c, 3, act="leaky", gamma=0.3, name="b%d.b" % b)
            y = g.add(y, h, name="b%d.add" % b)
    else:
        raise ValueError("unknown kind %r" % kind)
    if kind == "int8_stage":
        g.output(y, dtype="f32")
    else:
        g.output(y)
    return g


def _function(case, seed):
    g = _build(case, seed)
    wl = g.finish()
    graph = wl.graph
    if case["kind"] == "int8_stage":
        # ranges as a calibration would find them for these normalized layers
        ranges = {"x": (0.0, 1.0)}
        for node in graph["nodes"]:
            hi = 5.0 * math.sqrt(g.m2[node["name"]])
            ranges[node["name"]] = (0.0 if node["composite"].endswith("relu") else -hi, hi)
        graph = quantize.quantize_graph(graph, ranges)
    return graph, wl.consts, wl.inputs


def prepare(case, seed):
    graph, consts, arrays = _function(case, seed)
    sg = capi.Subgraph(graph, consts, device=0)
    if case.get("autotune"):
        sg.set_options(autotune=True)
    if case.get("graph_replay"):
        sg.set_options(graph_replay=True)
    kinds = {"bf16": torch.bfloat16, "f32": torch.float32}
    ins = [torch.from_numpy(np.ascontiguousarray(a)).to(DEVICE).to(kinds[d["dtype"]])
           for a, d in zip(arrays, graph["inputs"])]
    outs = [torch.empty(d["shape"], dtype=kinds[d["dtype"]], device=DEVICE)
            for d in (sg.io_desc(1, j) for j in range(sg.n_out))]
    # a graph replay needs a stream of its own (the null stream is never captured)
    stream = torch.cuda.Stream(DEVICE) if case.get("graph_replay") else None
    return {"engine": sg, "inputs": ins, "outputs": outs, "stream": stream}


def run(state):
    sg, stream = state["engine"], state["stream"]
    if stream is None:
        sg.run(state["inputs"], state["outputs"])
        return state["outputs"]
    # ordered with the program's own stream on both sides
    stream.wait_stream(torch.cuda.current_stream(DEVICE))
    sg.run(state["inputs"], state["outputs"], stream)
    torch.cuda.current_stream(DEVICE).wait_stream(stream)
    return state["outputs"]


def work(case):
    """Multiply-accumulates of the convs and dense layers; inputs and weights read once, outputs written once."""
    g = _build(case, 0)
    esize = 4 if _is_f32(case) else 1 if case["kind"] == "int8_stage" else 2
    size = {"f32": 4, "bf16": 2}
    nbytes = sum(int(np.prod(i["shape"])) * size[i["dtype"]] for i in g.inputs)
    nbytes += sum(int(np.prod(c["shape"])) * (esize if len(c["shape"]) > 1 else 4) for c in g.constants)
    nbytes += sum(int(np.prod(g.shapes[o["name"]])) * size[o["dtype"]] for o in g.outputs)
    return {"bytes": nbytes, "flops": 2 * g.macs}


def tolerance(case):
    # about four times the largest distance from the 64-bit values seen over
    # the listed and some drawn cases (bf16: 4e-3 and 4e-2, one to eight layers
    # as well as the 50-layer network; float32: 6e-7 and 6e-6, more for longer
    # sums); int8 graphs are integers up to the final scale
    if case["kind"] == "int8_stage":
        return "exact"
    if _is_f32(case):
        return {"rel": 4e-6, "max": 4e-5}
    return {"rel": 1.2e-2, "max": 0.15}


# ---- the same functions in 64 bits, in plain torch ----------------------------

def _conv64(x, w, strides, pads, groups):
    pt, pl, pb, pr = pads
    xp = F.pad(x, (pl, pr, pt, pb))
    n, c, h, wd = xp.shape
    k, cg, r, s = w.shape
    p, q = (h - r) // strides[0] + 1, (wd - s) // strides[1] + 1
    y = torch.zeros((n, k, p, q), dtype=torch.float64, device=x.device)
    for i in range(r):
        for j in range(s):
            win = xp[:, :, i:i + strides[0] * (p - 1) + 1:strides[0], j:j + strides[1] * (q - 1) + 1:strides[1]]
            if groups == 1:
                rows = win.permute(0, 2, 3, 1).reshape(-1, c)
                y += (rows @ w[:, :, i, j].t().contiguous()).reshape(n, p, q, k).permute(0, 3, 1, 2)
            else:  # depthwise
                y += win * w[:, 0, i, j].view(1, -1, 1, 1)
    return y


def _act64(y, act, alpha):
    if act == "relu":
        return y.clamp(min=0.0)
    if act == "relu6":
        return y.clamp(0.0, 6.0)
    if act == "leaky":
        return torch.where(y < 0, y * alpha, y)
    if act == "gelu":
        return 0.5 * y * torch.special.erfc(-y / math.sqrt(2.0))
    return y


def _parts(composite):
    base, tail = next((b, composite[len(b):]) for b in ("conv2d", "dense", "max_pool2d", "avg_pool2d",
                                                        "global_avg_pool2d", "concatenate", "add")
                      if composite.startswith(b))
    parts = [t for t in tail.split("_") if t]
    act = next((a for a in parts if a in ("relu", "relu6", "gelu", "leaky")), None)
    return base, "bias" in parts, "add" in parts, act


def _node64(node, vals, consts):
    op, bias, add, act = _parts(node["composite"])
    a, ins = node.get("attrs", {}), list(node["inputs"])
    x = vals[ins[0]]
    if op in ("conv2d", "dense"):
        w = consts[ins[1]]
        y = _conv64(x, w, a["strides"], a["padding"], a["groups"]) if op == "conv2d" else x @ w.t().contiguous()
        if bias:
            b = consts[ins[2]]
            y = y + (b.view(1, -1, 1, 1) if op == "conv2d" else b)
        if add:
            y = y + vals[ins[-1]]
        return _act64(y, act, a.get("alpha", 0.1))
    if op == "max_pool2d":
        pt, pl, pb, pr = a["padding"]
        xp = F.pad(x, (pl, pr, pt, pb), value=-math.inf)
        return xp.unfold(2, a["pool_size"][0], a["strides"][0]).unfold(3, a["pool_size"][1], a["strides"][1]).amax((4, 5))
    if op == "avg_pool2d":
        pt, pl, pb, pr = a["padding"]
        def windows(t):
            return F.pad(t, (pl, pr, pt, pb)).unfold(2, a["pool_size"][0], a["strides"][0]) \
                .unfold(3, a["pool_size"][1], a["strides"][1]).sum((4, 5))
        return windows(x) / windows(torch.ones_like(x[:1, :1]))
    if op == "global_avg_pool2d":
        return x.mean((2, 3))
    if op == "concatenate":
        return torch.cat([vals[i] for i in ins], 1)
    return _act64(x + vals[ins[1]], act, a.get("alpha", 0.1))


def _rescale(a, m):
    m32 = m.to(torch.float32) if isinstance(m, torch.Tensor) else torch.tensor(m, dtype=torch.float32, device=a.device)
    return (a.to(torch.float32) * m32).round().clamp(-2.0 ** 20, 2.0 ** 20).to(torch.float64)


def _node_int8(node, codes, quant, consts):
    """A quantized conv composite: integer codes in, integer codes out."""
    op, bias, add, act = _parts(node["composite"])
    a, ins = node["attrs"], node["inputs"]
    (sx, zx), (sy, zy) = quant[ins[0]], quant[node["name"]]
    w = consts[ins[1]]
    sw = w.abs().amax((1, 2, 3)) / 127.0
    wq = (w / sw.view(-1, 1, 1, 1)).round().clamp(-127, 127)
    acc = _conv64(codes[ins[0]] - zx, wq, a["strides"], a["padding"], a["groups"])
    if bias:
        acc = acc + (consts[ins[2]] / (sx * sw)).round().view(1, -1, 1, 1)
    v = zy + _rescale(acc, (sx * sw / sy).view(1, -1, 1, 1))
    if add:
        sr, zr = quant[ins[-1]]
        v = v + _rescale(codes[ins[-1]] - zr, sr / sy)
    return v.clamp(zy if act == "relu" else -128, 127)


def exact(case, seed):
    graph, consts, arrays = _function(case, seed)
    dev = DEVICE if torch.cuda.is_available() else "cpu"
    int8, f32 = case["kind"] == "int8_stage", _is_f32(case)

    def bf16(t):  # bf16 graphs round float32 weights and inputs once
        return t if int8 or f32 else t.to(torch.bfloat16).to(torch.float64)

    cvals = {}
    for c in graph["constants"]:
        t = torch.from_numpy(np.asarray(consts[c["index"]])).to(dev)
        cvals[c["name"]] = bf16(t).to(torch.float64) if len(c["shape"]) > 1 else t.to(torch.float64)
    vals, quant = {}, {}
    for d, arr in zip(graph["inputs"], arrays):
        t = torch.from_numpy(np.asarray(arr)).to(dev)
        if int8:
            s, z = quant[d["name"]] = (d["quant"]["scale"], d["quant"]["zero_point"])
            t = ((t * torch.tensor(1.0 / s, dtype=torch.float32, device=dev)).round() + z).clamp(-128, 127)
            vals[d["name"]] = t.to(torch.float64)
        else:
            vals[d["name"]] = bf16(t).to(torch.float64)
    for node in graph["nodes"]:
        if int8:
            quant[node["name"]] = (node["quant"]["scale"], node["quant"]["zero_point"])
            vals[node["name"]] = _node_int8(node, vals, quant, cvals)
        else:
            vals[node["name"]] = _node64(node, vals, cvals)
    outs = []
    for o in graph["outputs"]:
        v = vals[o["name"]]
        if int8:
            s, z = quant[o["name"]]
            v = torch.tensor(s, dtype=torch.float32, device=dev) * (v - z).to(torch.float32)
        outs.append(v.to(torch.float64))
    return outs
