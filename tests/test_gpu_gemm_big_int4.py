"""GPU parity of the large tiles on an INT4 base against the fp64 oracle.

Plain projections of the caller's activations above 384 tokens (one and a half
row tiles) take them, when the call holds at least 16 k-steps of a 256 x 256
tile per compute unit; both lines, ragged rows, columns in one half of a
tile only, inputs of one, two, five and eleven scale groups (one or two groups
per k-range are the k-loop's shortest runs), split and unsplit tiles, and
ranks from 0 to 64 are covered.  The error rule is that of the other parity
tests."""
import numpy as np
import pytest

import workloads as wl
from workloads.gpu import DeviceLayer, device_to_float, load_adapters, make_pool
from oracle import bdlora, quant

pytestmark = pytest.mark.gpu
TOL = 1e-2
RANKS = [0, 16, 64, 5, 24, 33]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    import paper_2510_23346_amd as bd
    bd.lib()
    return torch


SMALL = [
    wl.ProjSpec("qkv", "column", 256, (128, 64, 64)),
    wl.ProjSpec("o", "row", 128, (192,)),
    wl.ProjSpec("up", "column", 640, (320,)),
    wl.ProjSpec("down", "row", 1408, (448,)),
]
PROJS = {
    "small": SMALL,
    # split tiles (176 k-steps and 44) beside unsplit ones of 4, 8 and 20
    "deep": SMALL + [wl.ProjSpec("gate", "column", 5632, (2112,))],
    # no tile is split
    "wide": [wl.ProjSpec("up", "column", 1408, (16000,))],
}


@pytest.mark.parametrize("name,T,path", [("wide", 384, "tile64"), ("wide", 385, "large"), ("wide", 512, "large"),
                                         ("small", 1025, "tile64"), ("deep", 769, "large"), ("deep", 1025, "large")])
def test_int4_large_tiles(torch_cuda, name, T, path):
    torch = torch_cuda
    projs = PROJS[name]
    ids = np.random.default_rng(T).integers(-1, len(RANKS), size=T)
    spec = wl.custom_workload(f"int4-big-{T}", projs, T, RANKS, scales=[0.5 + 0.25 * i for i in range(len(RANKS))],
                              ids=ids, seed=T, weight_format="int4_g128")
    layer = wl.draw_layer(spec, slots=range(len(RANKS)))
    pool = make_pool(spec, max_tokens=T)
    load_adapters(pool, spec, range(len(RANKS)), cache=layer.adapters)
    dl = DeviceLayer(layer)
    idx = list(range(len(projs)))
    base = [torch.empty_like(o) for o in dl.out]
    for outs, i in ((dl.out, dl.ids), (base, torch.full_like(dl.ids, -1))):
        for o in outs:
            o.fill_(float("nan"))
        pool.forward_layer(idx, dl.X, dl.W, outs, i)
        torch.cuda.synchronize()
        assert pool.last_path() == path
    refs = quant.layer_forward_w4(layer)
    for p, pi in enumerate(layer.projs):
        y, yb = device_to_float(dl.out[p]), device_to_float(base[p])
        rb = pi.X.astype(np.float64) @ quant.dequantize(pi.Wq, pi.Ws_bits, pi.spec.d_in)
        assert bdlora.rel_errors(y, refs[p])["pointwise"] <= TOL, f"T={T} {pi.spec.name}"
        assert bdlora.rel_errors(yb, rb)["pointwise"] <= TOL, f"T={T} {pi.spec.name} base"
        assert bdlora.delta_errors(y, yb, refs[p], rb) <= TOL, f"T={T} {pi.spec.name} LoRA term"
    assert pool.device_error() == 0
    pool.close()
