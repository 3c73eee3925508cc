"""The one-launch decode path at the edges of its tiles, against the oracle,
also over the row groups of batches above the decode size; the shrink of
larger batches on activations beyond 32-bit offsets.

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
import ctypes

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
    # the same tokens in another order: the later calls find another call's Z and flags
    for rep, order in enumerate((np.arange(T), rng.permutation(T), np.arange(T)[::-1].copy())):
        at = torch.from_numpy(order).cuda()
        for o in dl.out:
            o.fill_(float("nan"))
        pool.forward_layer([0, 1, 2], [x[at].contiguous() for x in dl.X], dl.W, dl.out, dl.ids[at].contiguous())
        torch.cuda.synchronize()
        for p, y in enumerate(dl.outputs()):
            e = bdlora.rel_errors(y, refs[p][order])
            assert e["pointwise"] <= TOL, f"T={T} {ids_kind} call {rep} {spec.projs[p].name}: {e}"
    assert pool.last_path() == "decode" and pool.device_error() == 0
    pool.close()


def _launches(bd, pool):
    """The pool's launch counts and flags."""
    f = bd.lib().bdlora_internal_launches
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64, ctypes.POINTER(ctypes.c_int64), ctypes.c_void_p,
                  ctypes.c_int64, ctypes.POINTER(ctypes.c_int64)]
    nc, nf = ctypes.c_int64(), ctypes.c_int64()
    assert f(pool.handle, None, 0, ctypes.byref(nc), None, 0, ctypes.byref(nf)) == 0
    count, flags = np.zeros(nc.value, np.uint32), np.zeros(nf.value, np.uint64)
    assert f(pool.handle, count.ctypes.data, nc.value, ctypes.byref(nc), flags.ctypes.data, nf.value, ctypes.byref(nf)) == 0
    return count, flags


def test_every_launch_has_a_number_of_its_own(torch_cuda):
    # eager calls of several sizes, row groups, the MLP and replays of a graph,
    # on streams made and destroyed in between: after each launch all
    # workgroups' counts agree, one higher than before, also those that the
    # launch has no workgroup for; and the flags that it raised carry its
    # number, so that none of an earlier launch can be taken for one of its own
    torch = torch_cuda
    import paper_2510_23346_amd as bd
    projs = [wl.ProjSpec("gate", "column", 640, (384,)), wl.ProjSpec("up", "column", 640, (384,)),
             wl.ProjSpec("down", "row", 384, (192,))]
    T, ranks = 200, [8, 32, 16]
    ids = np.random.default_rng(1).integers(0, 3, size=T)
    spec = wl.custom_workload("launch-no", projs, T, ranks, ids=ids, seed=5)
    layer = wl.draw_layer(spec, slots=range(3))
    pool = make_pool(spec)
    load_adapters(pool, spec, range(3), cache=layer.adapters)
    dl = DeviceLayer(layer)
    hip = bd.lib()                           # (the HIP runtime that the library uses)

    def layer_call(t, s=None):
        pool.forward_layer([0, 1, 2], [x[:t] for x in dl.X], dl.W, [o[:t] for o in dl.out], dl.ids[:t], stream=s)

    def mlp_call(t, s=None):
        pool.forward_mlp(bd.ACT_SILU_MUL, [0, 1], 2, dl.X[0][:t], dl.W[:2], dl.W[2], dl.out[2][:t], dl.ids[:t], stream=s)
    layer_call(1)
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            layer_call(64)
    calls = [(1, lambda s: layer_call(1, s)), (1, lambda s: layer_call(16, s)), (2, lambda s: mlp_call(33, s)),
             (1, lambda s: layer_call(200, s)), (1, lambda s: layer_call(5, s)), (2, lambda s: mlp_call(130, s))]
    n, seen = 1, set()
    for rep in range(3):
        for k, call in calls + [(1, None)]:
            if call is None:
                g.replay()
            else:
                s = ctypes.c_void_p()
                assert hip.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0
                call(s.value)
                assert hip.hipStreamSynchronize(s) == 0 and hip.hipStreamDestroy(s) == 0
            torch.cuda.synchronize()
            n += k
            count, flags = _launches(bd, pool)
            assert count.min() == count.max() == n
            mine = set(flags[(flags >> np.uint64(32)) == n].tolist())
            assert len(mine) == 1 and not mine & seen, f"flags of launch {n}"
            seen |= mine
    assert pool.device_error() == 0
    pool.close()


@pytest.mark.parametrize("fmt", ["bf16", "int4_g128"])
@pytest.mark.parametrize("T", [1, 17, 33, 64, 150])
def test_a_wait_that_gives_up(torch_cuda, T, fmt):
    # with no time to wait, every main workgroup computes what its shrink
    # workgroups do (and writes it beside them): the same bits.  A layer of
    # projections with one and several slices, the gated MLP, the static
    # scratch, row groups.
    torch = torch_cuda
    import paper_2510_23346_amd as bd
    projs = [wl.ProjSpec("gate", "column", 640, (384,)), wl.ProjSpec("up", "column", 640, (384,)),
             wl.ProjSpec("down", "row", 384, (192,)), wl.ProjSpec("qkv", "column", 256, (16, 48, 16, 48))]
    ranks = [8, 128, 0, 24, 16, 5]
    ids = np.random.default_rng(T).integers(-1, len(ranks), size=T)
    spec = wl.custom_workload(f"gives-up-{T}", projs, T, ranks, ids=ids, seed=90 + T, weight_format=fmt)
    layer = wl.draw_layer(spec, slots=range(len(ranks)))
    pool = make_pool(spec)
    load_adapters(pool, spec, range(len(ranks)), cache=layer.adapters)
    dl = DeviceLayer(layer)
    set_wait = bd.lib().bdlora_internal_set_wait
    set_wait.argtypes = [ctypes.c_void_p, ctypes.c_uint32]

    def results(at):
        X, i = [x[at].contiguous() for x in dl.X], dl.ids[at].contiguous()
        got = []
        for call in (pool.forward_layer, pool.forward_layer_static) if T <= bd.DECODE_MAX_T else (pool.forward_layer,):
            for o in dl.out:
                o.fill_(float("nan"))
            call([0, 1, 2, 3], X, dl.W, dl.out, i)
            torch.cuda.synchronize()
            got += [y.view(np.uint32).copy() for y in dl.outputs()]
        dl.out[2].fill_(float("nan"))
        pool.forward_mlp(bd.ACT_SILU_MUL, [0, 1], 2, X[0], dl.W[:2], dl.W[2], dl.out[2], i)
        torch.cuda.synchronize()
        return got + [dl.outputs()[2].view(np.uint32).copy()]
    rng = np.random.default_rng(2)
    for rep in range(3):
        at = torch.from_numpy(rng.permutation(T)).cuda()
        want = results(at)
        other = results(torch.flip(at, [0]))               # another call's Z and flags in between
        assert set_wait(pool.handle, 0) == 0
        got = results(at)
        assert set_wait(pool.handle, 20000) == 0
        assert len(got) == len(want) == len(other)
        for k, (a, b) in enumerate(zip(got, want)):
            assert np.array_equal(a, b), f"T={T} {fmt} call {rep} output {k}"
    refs = (quant.layer_forward_w4 if fmt != "bf16" else bdlora.layer_forward)(layer)
    for p in range(4):
        e = bdlora.rel_errors(got[p].view(np.float32), refs[p][at.cpu().numpy()])
        assert e["pointwise"] <= TOL, f"T={T} {fmt} {projs[p].name}: {e}"
    assert pool.device_error() == 0
    pool.close()


@pytest.mark.parametrize("T", [5, 30, 64, 130])
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


@pytest.mark.parametrize("T,ids_kind", [(65, "many"), (127, "one"), (128, "many"), (129, "many"), (193, "none"),
                                        (256, "many")])
def test_row_groups(torch_cuda, T, ids_kind):
    # batches of 65 to 256 tokens run the decode launch in groups of nearly
    # equal size, the last one shorter; ids and segments give the same bits
    torch = torch_cuda
    import paper_2510_23346_amd as bd
    ranks = [8, 64, 3, 0, 24, 16]
    rng = np.random.default_rng(T)
    ids = {"one": np.full(T, 1), "none": np.full(T, -1), "many": rng.integers(-1, len(ranks), size=T)}[ids_kind]
    spec = wl.custom_workload(f"rows-{T}-{ids_kind}", PROJS, T, ranks, ids=ids, seed=160 + T)
    layer = wl.draw_layer(spec, slots=range(len(ranks)))
    pool = make_pool(spec)
    load_adapters(pool, spec, range(len(ranks)), cache=layer.adapters)
    dl = DeviceLayer(layer)
    refs = bdlora.layer_forward(layer)
    pool.forward_layer([0, 1, 2], dl.X, dl.W, dl.out, dl.ids)
    torch.cuda.synchronize()
    assert pool.last_path() == "tile64"
    first = dl.outputs()
    for p, y in enumerate(first):
        e = bdlora.rel_errors(y, refs[p])
        assert e["pointwise"] <= TOL, f"T={T} {ids_kind} {spec.projs[p].name}: {e}"
    for o in dl.out:
        o.fill_(float("nan"))
    pool.forward_layer([0, 1, 2], dl.X, dl.W, dl.out, None, segs=bd.Segments.from_ids(ids))
    torch.cuda.synchronize()
    for p, y in enumerate(dl.outputs()):
        assert np.array_equal(y.view(np.uint32), first[p].view(np.uint32)), f"segments, {spec.projs[p].name}"
    assert pool.device_error() == 0
    pool.close()


def test_row_groups_captured_before_an_adapter_was_loaded(torch_cuda):
    # above the decode size a captured forward holds for adapters loaded later
    torch = torch_cuda
    T, ranks = 100, [8, 16, 24]
    ids = np.random.default_rng(5).integers(0, 3, size=T)
    spec = wl.custom_workload("rows-capture", PROJS, T, ranks, ids=ids, seed=9)
    layer = wl.draw_layer(spec, slots=range(3))
    pool = make_pool(spec)
    load_adapters(pool, spec, [0], cache=layer.adapters)
    dl = DeviceLayer(layer)
    with torch.cuda.stream(torch.cuda.Stream()):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            pool.forward_layer([0, 1, 2], dl.X, dl.W, dl.out, dl.ids)
    load_adapters(pool, spec, [1, 2], cache=layer.adapters)
    refs = bdlora.layer_forward(layer)
    for rep in range(3):
        for o in dl.out:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for p, y in enumerate(dl.outputs()):
            e = bdlora.rel_errors(y, refs[p])
            assert e["pointwise"] <= TOL, f"replay {rep} {spec.projs[p].name}: {e}"
    assert pool.device_error() == 0
    pool.close()


@pytest.mark.parametrize("T,K", [(4100, 262144), (32768, 32800)])
def test_shrink_of_activations_beyond_two_gigabytes(torch_cuda, T, K):
    # X of 4100 x 262144 bf16 (2.15 GB), and one of an odd number of k-steps
    # that ends where its memory does (2050 MiB): the prefill launches address
    # it with 64-bit offsets; a few rows (the last ones past 2 GB) against float64
    torch = torch_cuda
    import paper_2510_23346_amd as bd
    N, ranks = 64, [8, 5]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)

    def normal(*shape, std=1.0):
        return (torch.randn(*shape, generator=gen, device="cuda") * std).to(torch.bfloat16)
    pool = bd.Pool([("row", K, (N,))], 2, 8, T)
    A = [normal(K, r, std=K ** -0.5) for r in ranks]
    B = [normal(r, N, std=r ** -0.5) for r in ranks]
    bits = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)  # noqa: E731
    for s in range(2):
        pool.load_adapter(s, ranks[s], 2.0, [[bits(A[s])]], [[bits(B[s])]])
    X = torch.empty(T, K, dtype=torch.bfloat16, device="cuda")
    for t in range(0, T, 410):
        X[t:t + 410] = normal(min(410, T - t), K)
    W = normal(N, K, std=K ** -0.5)
    out = torch.full((T, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    ids = (torch.arange(T, device="cuda") % 3 - 1).to(torch.int32)
    pool.forward_shard(0, X, bd.pack_weight(W), ids, out)
    torch.cuda.synchronize()
    for t in (0, 1, 2, 2047, 4095, T - 5, T - 4, T - 3, T - 2, T - 1):
        x, a = X[t].double(), int(ids[t])
        y = x @ W.double().t()
        if a >= 0:
            y += 2.0 * (x @ A[a].double()) @ B[a].double()
        err = (out[t].double() - y).abs() / torch.maximum(y.abs(), y.square().mean().sqrt())
        assert float(err.max()) <= 1e-2, f"row {t}: {float(err.max())}"
    assert pool.device_error() == 0
    pool.close()


def test_mlp_intermediate_beyond_two_gigabytes(torch_cuda):
    # the same for an intermediate of 32768 x 32800, which down's shrink reads
    # in its packed form (an odd number of k-steps, no row of padding)
    torch = torch_cuda
    import paper_2510_23346_amd as bd
    T, K, H, N = 32768, 64, 32800, 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)

    def normal(*shape, std=1.0):
        return (torch.randn(*shape, generator=gen, device="cuda") * std).to(torch.bfloat16)
    pool = bd.Pool([("column", K, (H,)), ("row", H, (N,))], 1, 8, T)
    A, B = [normal(K, 8, std=K ** -0.5), normal(H, 8, std=H ** -0.5)], [normal(8, H, std=8 ** -0.5), normal(8, N, std=8 ** -0.5)]
    bits = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)  # noqa: E731
    pool.load_adapter(0, 8, 2.0, [[bits(a)] for a in A], [[bits(b)] for b in B])
    X, W0, W1 = normal(T, K), normal(H, K, std=K ** -0.5), normal(N, H, std=H ** -0.5)
    out = torch.full((T, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    ids = (torch.arange(T, device="cuda") % 2 - 1).to(torch.int32)
    pool.forward_mlp(bd.ACT_NONE, [0], 1, X, [bd.pack_weight(W0)], bd.pack_weight(W1), out, ids)
    torch.cuda.synchronize()
    for t in (0, 1, 15, 16, 4095, T - 17, T - 16, T - 2, T - 1):
        y, a = X[t].double(), int(ids[t])
        for i, w in enumerate((W0, W1)):
            z = y @ w.double().t()
            if a >= 0:
                z = z + 2.0 * (y @ A[i].double()) @ B[i].double()
            y = z.bfloat16().double() if i == 0 else z
        err = (out[t].double() - y).abs() / torch.maximum(y.abs(), y.square().mean().sqrt())
        assert float(err.max()) <= 1e-2, f"row {t}: {float(err.max())}"
    assert pool.device_error() == 0
    pool.close()


@pytest.mark.parametrize("T,fmt,entry,path", [
    (1, "bf16", "layer", "decode"), (16, "bf16", "static", "decode"), (64, "bf16", "layer", "decode"),
    (64, "int4", "static", "decode"), (100, "bf16", "layer", "medium"), (100, "int4", "layer", "tile64"),
    (200, "bf16", "layer", "tile64"), (300, "bf16", "layer", "large"), (300, "int4", "layer", "tile64"),
    (400, "int4", "wide", "tile64")])
def test_out_may_share_memory_with_x(torch_cuda, T, fmt, entry, path):
    # an out on top of its own X and of the X that another projection shares,
    # another one beginning inside an X: every X is read as it was before the
    # call.  (Each launch sequence; "wide" would take the INT4 large tiles.)
    # Against the same call with memory of its own, to the tolerance above
    # (twice: both sides round): the large tiles add k-steps in another order.
    torch = torch_cuda
    import paper_2510_23346_amd as bd
    projs = [("column", 1408, (16000,))] if entry == "wide" else [
        ("column", 256, (256,)), ("column", 256, (192,)), ("row", 128, (320,))]
    f = bd.WEIGHT_INT4_G128 if fmt == "int4" else bd.WEIGHT_BF16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T)

    def normal(*shape, std=1.0):
        return (torch.randn(*shape, generator=gen, device="cuda") * std).to(torch.bfloat16)
    pool = bd.Pool(projs, 16, 24, T, weight_formats=f)
    bits = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)  # noqa: E731
    for s in range(16):
        r = (8, 24, 16)[s % 3]
        pool.load_adapter(s, r, 2.0, [[bits(normal(k, r, std=k ** -0.5))] for _, k, _ in projs],
                          [[bits(normal(r, n[0], std=r ** -0.5))] for _, _, n in projs])
    W = []
    for _, k, (n,) in projs:
        if fmt == "bf16":
            W.append(bd.pack_weight(normal(n, k, std=k ** -0.5)))
        else:
            q = torch.randint(0, 256, (n, k // 2), generator=gen, device="cuda", dtype=torch.uint8)
            W.append(bd.pack_weight_int4(q, (torch.rand(n, k // 128, generator=gen, device="cuda") * 0.01).bfloat16()))
    x0 = [normal(T, k) for _, k, _ in projs]
    if entry != "wide":
        x0[1] = x0[0]
    ids = torch.randint(-1, 16, (T,), generator=gen, device="cuda", dtype=torch.int32)
    call = pool.forward_layer_static if entry == "static" else pool.forward_layer
    idx = list(range(len(projs)))
    want = [torch.empty(T, n, dtype=torch.bfloat16, device="cuda") for _, _, (n,) in projs]
    call(idx, x0, W, want, ids)
    torch.cuda.synchronize()
    for rep in range(3):
        if entry == "wide":
            mem = [normal(T * 16000)]
            X, out = [mem[0][:T * 1408].view(T, 1408)], [mem[0].view(T, 16000)]
        else:
            mem = [normal(T * 256), normal(T * 192), normal(T * (128 + 320))]
            X = [mem[0].view(T, 256), mem[0].view(T, 256), mem[2][:T * 128].view(T, 128)]
            at = T * 64                                       # half way into the third X
            out = [mem[0].view(T, 256), mem[1].view(T, 192), mem[2][at:at + T * 320].view(T, 320)]
        if rep == 2:                                          # the last one as a replay
            with torch.cuda.stream(torch.cuda.Stream()):
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph):
                    call(idx, X, W, out, ids)
        for x, v in zip(X, x0):
            x.copy_(v)
        torch.cuda.synchronize()
        if rep == 2:
            graph.replay()
        else:
            call(idx, X, W, out, ids)
        torch.cuda.synchronize()
        assert pool.last_path() == path
        for i in idx:
            y, r = out[i].double(), want[i].double()
            err = float(((y - r).abs() / torch.maximum(r.abs(), r.square().mean().sqrt())).max())
            assert err <= (0.0 if path != "large" and entry != "wide" else 2 * TOL), f"call {rep} projection {i}: {err}"
    assert pool.device_error() == 0
    pool.close()


@pytest.mark.parametrize("mean", [0.0, 1.0])
@pytest.mark.parametrize("T,N,path", [(5, 256, "decode"), (32, 256, "decode"), (48, 256, "decode"), (64, 256, "decode"),
                                      (200, 256, "tile64"), (800, 2688, "large")])
def test_int4_sums_are_as_exact_as_the_64_row_kernel(torch_cuda, T, N, path, mean):
    # The fp32 sums of an INT4 base, seen through outputs that are exactly zero:
    # the second half of the inputs repeats the first, permuted inside each
    # scale group, with the opposite weights.  What comes out is the sums'
    # rounding.  The 64-row kernel (above 256 tokens) takes the offset of the
    # stored nibbles out of every single k-step; the rounding of the decode
    # launch and of the large tiles, over the same rows, is no larger.
    torch = torch_cuda
    import paper_2510_23346_amd as bd
    K, G, TB = 4096, 16, 300
    R = max(T, TB)
    rng = np.random.default_rng(17)
    q = rng.integers(-7, 8, size=(N, G, 128))
    s = np.tile(rng.uniform(0.005, 0.02, size=(N, G)).astype(np.float32), 2)
    x = torch.from_numpy(rng.standard_normal((R, G, 128)).astype(np.float32) + np.float32(mean)).bfloat16()
    perm = np.stack([rng.permutation(128) for _ in range(G)])
    take = torch.from_numpy(perm)[None].expand(R, G, 128)
    X = torch.cat([x, torch.gather(x, 2, take)], dim=1).reshape(R, K).cuda()
    qq = np.concatenate([q, -np.take_along_axis(q, np.broadcast_to(perm, q.shape), axis=2)], axis=1).reshape(N, K) + 8
    nib = torch.from_numpy((qq[:, 0::2] | (qq[:, 1::2] << 4)).astype(np.uint8)).cuda()
    W = bd.pack_weight_int4(nib, torch.from_numpy(s).bfloat16().cuda())
    pool = bd.Pool([("row", K, (N,))], 1, 8, R, weight_formats=bd.WEIGHT_INT4_G128)
    rms = {}
    for t, want in ((T, path), (TB, "tile64")):
        out = torch.full((t, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        pool.forward_shard(0, X[:t], W, torch.full((t,), -1, dtype=torch.int32, device="cuda"), out)
        torch.cuda.synchronize()
        rms[t] = float(out[:min(T, TB)].double().square().mean().sqrt())
        assert pool.last_path() == want
    assert rms[TB] > 0
    assert rms[T] <= rms[TB], f"rounding {rms[T]:.3e}, 64-row kernel {rms[TB]:.3e}"
    pool.close()


@pytest.mark.parametrize("T", [60, 100, 250])
def test_replay_with_more_to_shrink_than_at_capture(torch_cuda, T):
    # the launch counts its shrink workgroups by the adapters loaded when it is
    # captured: adapters of rank 128 in every slot afterwards make several
    # times as many units, which they take in turns
    torch = torch_cuda
    n, few = 48, 60 if T <= 64 else 1
    n = max(n, few)
    ranks = [128 if s else 120 for s in range(n)]
    projs = [wl.ProjSpec("qkv", "column", 160, (32, 32, 32, 32)), wl.ProjSpec("o", "row", 96, (144,)),
             wl.ProjSpec("up", "column", 160, (64,))]
    ids = np.random.default_rng(T).integers(-1, n, size=T)
    spec = wl.custom_workload(f"more-{T}", projs, T, ranks, ids=ids, seed=T)
    layer = wl.draw_layer(spec, slots=range(n))
    pool = make_pool(spec)
    zero = lambda r: ([[np.zeros((p.d_in, r), np.uint16) for _ in p.slices] for p in projs],  # noqa: E731
                      [[np.zeros((r, o), np.uint16) for o in p.slices] for p in projs])
    for s in range(few):
        pool.load_adapter(s, 8, 1.0, *zero(8))
    dl = DeviceLayer(layer)
    with torch.cuda.stream(torch.cuda.Stream()):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            pool.forward_layer([0, 1, 2], dl.X, dl.W, dl.out, dl.ids)
    load_adapters(pool, spec, range(n), cache=layer.adapters)
    refs = bdlora.layer_forward(layer)
    for rep in range(3):
        for o in dl.out:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for p, y in enumerate(dl.outputs()):
            e = bdlora.rel_errors(y, refs[p])
            assert e["pointwise"] <= TOL, f"T={T} replay {rep} {projs[p].name}: {e}"
    assert pool.device_error() == 0
    pool.close()


@pytest.mark.parametrize("ranks,order", [("16", "blocks"), ("16", "spread"), ("mixed", "blocks"), ("mixed", "spread")])
@pytest.mark.parametrize("T", [16, 17, 32, 33, 48, 64, 150])
def test_many_adapters(torch_cuda, T, ranks, order):
    # forty adapters (eighteen in row groups): the expand row block by row block (each adapter's tokens
    # in few of them) or for all row blocks at once (spread over them); of rank
    # 16, and of ranks up to 128, whose shrink workgroups take four blocks of
    # A^T; a layer of projections with one and several slices, inputs of one
    # and of an odd number of k-steps, and the gated MLP
    torch = torch_cuda
    import paper_2510_23346_amd as bd
    n, few = (40, 12) if T <= 64 else (18, 6)              # (more, and 150 tokens take the medium-batch launches)
    projs = [wl.ProjSpec("gate", "column", 96, (160,)), wl.ProjSpec("up", "column", 96, (160,)),
             wl.ProjSpec("down", "row", 160, (80,)), wl.ProjSpec("qkv", "column", 96, (16, 48, 32, 32)),
             wl.ProjSpec("o", "row", 32, (1040,))]
    some = (128, 64, 8, 120, 0, 33) if T <= 64 else (128, 120, 64)
    rank = [16] * n if ranks == "16" else [some[i % len(some)] for i in range(n)]
    rng = np.random.default_rng(T)
    ids = rng.integers(-1, n, size=T)
    ids = np.sort(ids) if order == "blocks" else np.where(ids < 0, -1, np.arange(T) % few + few * (np.arange(T) // 64))
    spec = wl.custom_workload(f"many-{T}-{ranks}-{order}", projs, T, rank, ids=ids, seed=40 + T)
    layer = wl.draw_layer(spec, slots=range(n))
    pool = make_pool(spec)
    load_adapters(pool, spec, range(n), cache=layer.adapters)
    dl = DeviceLayer(layer)
    set_wait = bd.lib().bdlora_internal_set_wait
    set_wait.argtypes = [ctypes.c_void_p, ctypes.c_uint32]
    seen = []
    for ticks in (20000, 20000, 0):                     # (0: the main workgroups compute Z themselves)
        assert set_wait(pool.handle, ticks) == 0
        for o in dl.out:
            o.fill_(float("nan"))
        pool.forward_layer([0, 1, 2, 3, 4], dl.X, dl.W, dl.out, dl.ids)
        torch.cuda.synchronize()
        got = [y.copy() for y in dl.outputs()]
        pool.forward_mlp(bd.ACT_SILU_MUL, [0, 1], 2, dl.X[0], dl.W[:2], dl.W[2], dl.out[2], dl.ids)
        torch.cuda.synchronize()
        seen.append(got + [dl.outputs()[2].copy()])
    for other in seen[1:]:
        assert all(np.array_equal(a.view(np.uint32), b.view(np.uint32)) for a, b in zip(seen[0], other))
    refs = bdlora.layer_forward(layer)
    for p in range(len(projs)):
        e = bdlora.rel_errors(seen[0][p], refs[p])
        assert e["pointwise"] <= TOL, f"{projs[p].name}: {e}"

    def ref(i, x):
        y = x @ layer.projs[i].W.astype(np.float64)
        for t, a in enumerate(ids):
            if a >= 0 and rank[a]:
                ad = layer.adapters[int(a)]
                y[t] += ad.scale * (x[t] @ ad.A[i][0].astype(np.float64)) @ ad.B[i][0].astype(np.float64)
        return y
    x0 = layer.projs[0].X.astype(np.float64)
    g, u = ref(0, x0), ref(1, x0)
    h = wl.bf16_round((g / (1.0 + np.exp(-g)) * u).astype(np.float32))[1].astype(np.float64)
    e = bdlora.rel_errors(seen[0][5], ref(2, h))
    assert e["pointwise"] <= 2 * TOL, f"mlp: {e}"          # (H may round the other way, as above)
    assert pool.last_path() == ("decode" if T <= 64 else "tile64") and pool.device_error() == 0
    pool.close()
