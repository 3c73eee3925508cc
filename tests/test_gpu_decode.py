"""The one-launch decode path at the edges of its tiles, against the oracle.

Token counts around the 16-row blocks; inputs of one k-step, an odd number of
them and more than the waves' shares; output widths that end inside a
workgroup's columns; slices that end inside a pair of 16-column blocks (their
columns read different rank slices of one wave); one adapter holding several
16-token items, many adapters, ranks from 0 to 128 in one pool, bf16 and INT4
bases, gate and up of different weight formats.

Tolerance: the sums are fp32 and the output is rounded once to bf16, half a
unit in the last place, 2^-9 of the value; 2^-8 of max(value, rms) leaves the
same again for the fp32 sums and the exact split of Z.
"""
import numpy as np
import pytest

import workloads as wl
from oracle import bdlora, quant
from workloads.gpu import DeviceLayer, bits_to_device, device_to_float, load_adapters, make_pool

pytestmark = pytest.mark.gpu
TOL = 2.0 ** -8


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    import paper_2510_23346_amd as bd
    bd.lib()
    return torch


PROJS = [
    wl.ProjSpec("qkv", "column", 32, (16, 48, 16, 32)),        # one k-step, slices of odd block counts
    wl.ProjSpec("o", "row", 544, (144,)),                      # 17 k-steps
    wl.ProjSpec("up", "column", 2080, (1040,)),                # 65 k-steps, 65 column blocks
]


@pytest.mark.parametrize("T,ids_kind", [(1, "one"), (15, "many"), (16, "one"), (17, "many"), (32, "none"), (33, "one"),
                                        (48, "many"), (49, "many"), (63, "one"), (64, "many")])
def test_decode_tile_edges(torch_cuda, T, ids_kind):
    torch = torch_cuda
    ranks = [8, 128, 1, 0, 24, 64, 16, 5, 40, 8, 16, 7]
    rng = np.random.default_rng(T)
    ids = {"one": np.full(T, 1), "none": np.full(T, -1), "many": rng.integers(-1, len(ranks), size=T)}[ids_kind]
    spec = wl.custom_workload(f"dec-{T}-{ids_kind}", PROJS, T, ranks, ids=ids, seed=60 + T)
    layer = wl.draw_layer(spec, slots=range(len(ranks)))
    pool = make_pool(spec)
    load_adapters(pool, spec, range(len(ranks)), cache=layer.adapters)
    dl = DeviceLayer(layer)
    refs = bdlora.layer_forward(layer)
    for rep in range(3):                     # (the later calls find the first one's Z and flags)
        for o in dl.out:
            o.fill_(float("nan"))
        pool.forward_layer([0, 1, 2], dl.X, dl.W, dl.out, dl.ids)
        torch.cuda.synchronize()
        for p, y in enumerate(dl.outputs()):
            e = bdlora.rel_errors(y, refs[p])
            assert e["pointwise"] <= TOL, f"T={T} {ids_kind} call {rep} {spec.projs[p].name}: {e}"
    assert pool.last_path() == "decode" and pool.device_error() == 0
    pool.close()


@pytest.mark.parametrize("T", [5, 30, 64])
def test_decode_int4_and_bf16_projections_in_one_call(torch_cuda, T):
    # one launch over an INT4 and a bf16 projection, and the gated MLP with
    # gate and up on different bases (either way round)
    torch = torch_cuda
    import paper_2510_23346_amd as bd
    projs = [wl.ProjSpec("gate", "column", 640, (384,)), wl.ProjSpec("up", "column", 640, (384,)),
             wl.ProjSpec("down", "row", 384, (192,))]
    ranks = [8, 32, 16]
    ids = np.random.default_rng(T).integers(-1, 3, size=T)
    spec = wl.custom_workload(f"dec-mix-{T}", projs, T, ranks, ids=ids, seed=80 + T, weight_format="int4_g128")
    layer = wl.draw_layer(spec, slots=range(3))
    q_layer = layer.projs
    X = [bits_to_device(p.X_bits) for p in q_layer]
    for fmts in ((bd.WEIGHT_INT4_G128, bd.WEIGHT_BF16, bd.WEIGHT_BF16),
                 (bd.WEIGHT_BF16, bd.WEIGHT_INT4_G128, bd.WEIGHT_INT4_G128)):
        pool = bd.Pool(projs, 3, 32, T, weight_formats=list(fmts))
        load_adapters(pool, spec, range(3), cache=layer.adapters)
        W, Wf = [], []
        for p, f in zip(q_layer, fmts):
            if f == bd.WEIGHT_BF16:
                W.append(bd.pack_weight(bits_to_device(np.ascontiguousarray(p.W_bits.T))))
                Wf.append(p.W.astype(np.float64))
            else:
                W.append(bd.pack_weight_int4(torch.from_numpy(p.Wq).cuda(), bits_to_device(p.Ws_bits)))
                Wf.append(quant.dequantize(p.Wq, p.Ws_bits, p.spec.d_in))
        out = [torch.full((T, p.d_out), float("nan"), dtype=torch.bfloat16, device="cuda") for p in projs]
        idd = torch.from_numpy(ids.astype(np.int32)).cuda()
        pool.forward_layer([0, 1, 2], X, W, out, idd)
        torch.cuda.synchronize()

        def ref(i, x):
            y = x @ Wf[i]
            for t, a in enumerate(ids):
                if a >= 0:
                    ad = layer.adapters[int(a)]
                    y[t] += ad.scale * (x[t] @ ad.A[i][0].astype(np.float64)) @ ad.B[i][0].astype(np.float64)
            return y
        for i in range(3):
            e = bdlora.rel_errors(device_to_float(out[i]), ref(i, q_layer[i].X.astype(np.float64)))
            assert e["pointwise"] <= TOL, f"{fmts} {projs[i].name}: {e}"
        pool.forward_mlp(bd.ACT_SILU_MUL, [0, 1], 2, X[0], W[:2], W[2], out[2], idd)
        torch.cuda.synchronize()
        x0 = q_layer[0].X.astype(np.float64)
        g, u = ref(0, x0), ref(1, x0)
        h = wl.bf16_round((g / (1.0 + np.exp(-g)) * u).astype(np.float32))[1].astype(np.float64)
        e = bdlora.rel_errors(device_to_float(out[2]), ref(2, h))
        # (H is rounded to bf16 on both sides; where the fp32 sums move it over
        # a rounding boundary the down product sees a full unit, 2^-8)
        assert e["pointwise"] <= 2 * TOL, f"{fmts} mlp: {e}"
        assert pool.device_error() == 0
        pool.close()
