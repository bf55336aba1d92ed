"""Boundary layout transforms on the GPU.  A 1x1 max pool is the identity, so a
graph of one returns what the transforms around it make of the input: the
input rounded to bf16 (or quantized and dequantized), bit for bit.  Shapes at the
edges of the tiled kernels: planes that do not fill a run of pixels or a
vector, channels that do not fill a group or a tile, one image and many, and
buffers that are aligned to one element only."""

import numpy as np
import pytest
import torch

from oracle import quant as oq
from paper_2105_03215_amd import capi
from parity_util import announce

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
DT = {"bf16": torch.bfloat16, "f32": torch.float32}
SHAPES = [(1, 9, 4, 4), (2, 24, 5, 7), (3, 64, 16, 16), (1, 72, 15, 17), (5, 130, 1, 19), (70, 16, 12, 11),
          (600, 40, 6, 6), (9, 256, 28, 28), (33, 100, 17, 17), (2, 33, 3, 5), (4, 8, 20, 20)]


def _graph(shape, src, dst, quant):
    n, c, h, w = shape
    g = {"format": "byoc-subgraph", "version": 1,
         "inputs": [{"name": "x", "shape": list(shape), "dtype": src, "layout": "NCHW"}], "constants": [],
         "nodes": [{"name": "y", "composite": "max_pool2d", "inputs": ["x"],
                    "attrs": {"pool_size": [1, 1], "strides": [1, 1], "padding": [0] * 4},
                    "out_dtype": "int8" if quant else "bf16"}],
         "outputs": [{"name": "y", "dtype": dst, "layout": "NCHW"}]}
    if quant:
        for d in (g["inputs"][0], g["nodes"][0]):
            d["quant"] = {"scale": quant[0], "zero_point": quant[1]}
    return g


def _buffer(shape, dtype, offset):
    n = int(np.prod(shape))
    return torch.zeros(n + 8, dtype=dtype, device=DEV)[offset:offset + n].view(shape)


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
@pytest.mark.parametrize("quant", [None, (0.031, -7)], ids=["bf16", "int8"])
def test_round_trip(shape, quant):
    rng = np.random.default_rng(list(shape))
    a = rng.standard_normal(shape).astype(np.float32) * 2.0
    a.reshape(-1)[:3] = [np.inf, -np.inf, -0.0]
    for src, dst, offset in (("bf16", "bf16", 0), ("f32", "f32", 0), ("bf16", "f32", 1), ("f32", "bf16", 3)):
        announce("layout %s %s->%s offset %d %s" % (shape, src, dst, offset, quant))
        x = _buffer(shape, DT[src], offset)
        x.copy_(torch.from_numpy(a))
        y = _buffer(shape, DT[dst], offset)
        y.fill_(float("nan"))
        with capi.Subgraph(_graph(shape, src, dst, quant), [], device=0) as sg:
            sg.run([x], [y])
            torch.cuda.synchronize()
        if quant:
            codes = oq.quantize(x.float().cpu().numpy(), *quant)
            want = torch.from_numpy(oq.dequantize(codes, *quant)).to(DT[dst])
        else:
            want = x.cpu().to(torch.bfloat16).to(DT[dst])
        assert torch.equal(y.cpu(), want)
