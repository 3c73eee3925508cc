"""The work that users of this library have it do, as measurable cases.

A case is one call pattern of the BD-LoRA shard forward (a single projection,
a decoder-layer shard or an MLP shard of a Llama model at tensor-parallel
degree ``tp``) over one batch of tokens that name their own adapters.  The
shapes are those of the benchmark workloads in ``workloads/``; batch sizes run
from one decode token to a prefill of several thousand.

Decode batches up to 256 tokens are captured once into a HIP graph over
``layers`` consecutive layers, each with its own weights and adapter pool, and
a pass replays it, as a serving engine replays its decode step for each new
token (several layers, so that the weights come from HBM and not from the
256 MB Infinity Cache).  The other cases call the library eagerly.

Inputs are random with the value distributions of ``workloads/``: activations
N(0, 1), weights and A factors N(0, 1 / d_in), B factors N(0, 1 / rank), all
rounded to bfloat16; an INT4 base is the bf16 weight rounded to nearest in
groups of 128 inputs.
"""
import math

import numpy as np
import torch

import paper_2510_23346_amd as bd
from workloads import finite_zipf_probs, model_projs

SCALE = 2.0
MODELS = {"1b": "llama-3.2-1b", "8b": "llama-3.1-8b", "70b": "llama-3.1-70b"}


def _case(name, model, part, T, slots, ranks, ids, *, tp=8, layers=1, graph=False, fmt="bf16", requests=0,
          active=0, base_share=0.0, segments=False):
    """part: "up" (one projection), "layer" (qkv, o, gate, up, down) or "mlp"
    (gate, up, H, down).  ranks: the adapters' ranks, "/"-separated, dealt to
    the slots in turn ("mixed": drawn from 8, 16, 32, 64).  ids: "uniform" or
    "zipf" over the slots per token, "requests" (prefill: `requests` runs of
    tokens, one adapter each) or "mixed" (`requests` runs of 1024 tokens, then
    decode tokens).  active: adapters the batch may use (0: all slots).
    base_share: share of decode tokens without an adapter.  segments: the
    batch goes in as host segments instead of device ids."""
    return {"name": name, "model": model, "part": part, "T": T, "slots": slots, "ranks": ranks, "ids": ids, "tp": tp,
            "layers": layers, "graph": graph, "fmt": fmt, "requests": requests, "active": active,
            "base_share": base_share, "segments": segments}


def listed():
    return [
        # one projection of a small decode batch, called eagerly: launch and
        # call latency count as much as the 15 MB of weight
        _case("8b-up-T16", "8b", "up", 16, 4, "8", "uniform"),
        # a single user's decode: one token, one adapter, weight streaming only
        _case("8b-layer-T1", "8b", "layer", 1, 1, "16", "uniform", layers=4, graph=True),
        # an odd decode batch over adapters of ranks 8 and 64, some tokens
        # served by the base model alone
        _case("8b-layer-T37-mixed", "8b", "layer", 37, 16, "8/64", "zipf", layers=4, graph=True, base_share=0.2),
        # the usual multi-adapter decode batch: 32 resident adapters, Zipf ids
        _case("8b-layer-T64", "8b", "layer", 64, 32, "16", "zipf", layers=4, graph=True),
        # the same on a weight-only INT4 base
        _case("8b-layer-T64-int4", "8b", "layer", 64, 32, "16", "zipf", layers=4, graph=True, fmt="int4"),
        # the MLP shard alone (gate, up, silu(gate) * up, down), decode
        _case("8b-mlp-T64", "8b", "mlp", 64, 32, "16", "zipf", layers=4, graph=True),
        # a decode batch between the small-batch and the large-batch launches,
        # few adapters
        _case("8b-layer-T150", "8b", "layer", 150, 8, "16", "uniform", layers=4, graph=True),
        # a large decode batch of a large model: 128 resident adapters
        _case("70b-layer-T256", "70b", "layer", 256, 128, "16", "zipf", layers=1, graph=True),
        # prefill of one short prompt of odd length
        _case("8b-prefill-333", "8b", "layer", 333, 8, "32", "requests", requests=1, segments=True),
        # prefill of eight prompts of 512 tokens, eight adapters
        _case("8b-prefill-8x512", "8b", "layer", 4096, 8, "32", "requests", requests=8, segments=True),
        # prefill on a weight-only INT4 base, two prompts, odd length
        _case("8b-prefill-int4-1001", "8b", "layer", 1001, 8, "32", "requests", fmt="int4", requests=2, segments=True),
        # continuous batching of a large model: four prompts of 1024 tokens
        # prefill beside 192 decode tokens, 512-slot pool, 64 adapters active
        _case("70b-mixed-4288", "70b", "layer", 4288, 512, "mixed", "mixed", requests=4, active=64),
    ]


def draw(rng):
    """One more case of the same ranges."""
    part = rng.choice(["up", "layer", "layer", "layer", "mlp"])
    model = rng.choice(["1b", "8b", "8b", "70b"])
    fmt = "int4" if model != "70b" and rng.random() < 0.25 else "bf16"
    tp = 8 if model == "70b" else rng.choice([4, 8, 8])
    prefill = rng.random() < 0.45
    top = 1024 if fmt == "int4" else 4096
    T = int(math.exp(rng.uniform(math.log(65), math.log(top)))) if prefill else int(
        math.exp(rng.uniform(0, math.log(256.99))))
    slots = int(math.exp(rng.uniform(0, math.log(128.99))))
    ranks = rng.choice(["8", "16", "32", "64", "8/64", "4/16", "12/32"])
    if prefill:
        requests = rng.randint(1, max(1, min(16, T // 32)))
        c = _case("", model, part, T, slots, ranks, "requests", tp=tp, fmt=fmt, requests=requests,
                  segments=rng.random() < 0.5)
    else:
        layers = 1 if model == "70b" else rng.choice([2, 4])
        c = _case("", model, part, T, slots, ranks, rng.choice(["uniform", "zipf"]), tp=tp, fmt=fmt, layers=layers,
                  graph=rng.random() < 0.8, base_share=rng.choice([0.0, 0.0, 0.25]))
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs

def _projs(case):
    ps = model_projs(MODELS[case["model"]], case["tp"])
    pick = {"up": ["up"], "layer": ["qkv", "o", "gate", "up", "down"], "mlp": ["gate", "up", "down"]}[case["part"]]
    return [p for p in ps if p.name in pick]


def _ranks(case, seed):
    if case["ranks"] == "mixed":
        return [int(r) for r in np.random.default_rng([seed, 1]).choice([8, 16, 32, 64], size=case["slots"])]
    r = [int(x) for x in case["ranks"].split("/")]
    return [r[i % len(r)] for i in range(case["slots"])]


def _ids(case, seed):
    """Per-token adapter ids (numpy int32), -1 for none."""
    rng = np.random.default_rng([seed, 0])
    T, n = case["T"], case["slots"]
    act = np.sort(rng.choice(n, size=case["active"], replace=False)) if case["active"] else np.arange(n)
    if case["ids"] == "uniform":
        ids = rng.choice(act, size=T)
    elif case["ids"] == "zipf":
        ids = act[rng.choice(act.size, size=T, p=finite_zipf_probs(act.size))]
    elif case["ids"] == "requests":
        q = case["requests"]
        each = np.full(q, T // q)
        each[:T % q] += 1
        who = act[rng.permutation(act.size)[:q]] if q <= act.size else rng.choice(act, size=q)
        ids = np.repeat(who, each)
    else:                                    # mixed: prompts, then decode tokens
        who = rng.choice(act, size=case["requests"])
        ids = np.concatenate([np.repeat(who, 1024), rng.choice(act, size=T - 1024 * case["requests"])])
    if case["base_share"]:
        ids = np.where(rng.random(T) < case["base_share"], -1, ids)
    return np.ascontiguousarray(ids.astype(np.int32))


def _gen(seed, layer, what, k=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(((int(seed) * 64 + layer) * 8 + what) * 1024 + k)
    return g


def _normal(shape, std, g):
    return (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)


def _x(case, seed, layer, p):
    """Activations of projection p; gate and up of a layer share theirs."""
    name = p.name if p.name != "up" or case["part"] == "up" else "gate"
    return _normal((case["T"], p.d_in), 1.0, _gen(seed, layer, 0, "qkv o gate up down".split().index(name)))


def _w(case, seed, layer, i, p):
    """Base weight [d_out, d_in]: bf16, or (q, scales) with q in 0..15 (value
    + 8) and one bf16 scale per group of 128 inputs."""
    w = _normal((p.d_out, p.d_in), p.d_in ** -0.5, _gen(seed, layer, 1, i))
    if case["fmt"] == "bf16":
        return w
    g = w.float().view(p.d_out, p.d_in // 128, 128)
    s = (g.abs().amax(2) / 7).to(torch.bfloat16)
    q = (torch.round(g / s.float()[..., None]).clamp(-8, 7) + 8).to(torch.uint8).view(p.d_out, p.d_in)
    return q, s


def _adapter(projs, rank, seed, layer, slot):
    """One adapter's factors as one flat bf16 tensor on the GPU (see _split)."""
    z = torch.randn(sum(rank * (p.d_in + o) for p in projs for o in p.slices),
                    generator=_gen(seed, layer, 2, slot), device="cuda")
    for f, k in zip(*_split(z, projs, rank)):
        for a, b in zip(f, k):
            a *= a.shape[0] ** -0.5
            b *= rank ** -0.5
    return z.to(torch.bfloat16)


def _split(z, projs, rank):
    """[proj][slice] views A [d_in, rank] and B [rank, out] of a flat adapter."""
    A, B, at = [], [], 0
    for p in projs:
        A.append([])
        B.append([])
        for o in p.slices:
            A[-1].append(z[at:at + p.d_in * rank].reshape(p.d_in, rank))
            at += p.d_in * rank
            B[-1].append(z[at:at + rank * o].reshape(rank, o))
            at += rank * o
    return A, B


def _used(case, seed):
    """Slots that hold an adapter: all, or (pools larger than the working
    set) those that the batch may use."""
    if not case["active"]:
        return list(range(case["slots"]))
    rng = np.random.default_rng([seed, 0])
    return [int(s) for s in np.sort(rng.choice(case["slots"], size=case["active"], replace=False))]


def prepare(case, seed):
    projs, ranks, ids = _projs(case), _ranks(case, seed), _ids(case, seed)
    fmt = bd.WEIGHT_INT4_G128 if case["fmt"] == "int4" else bd.WEIGHT_BF16
    s = {"part": case["part"], "T": case["T"], "layers": [], "graph": None, "ids": None, "segs": None}
    if case["segments"]:
        s["segs"] = bd.Segments.from_ids(ids)
    else:
        s["ids"] = torch.from_numpy(ids).cuda()
    for layer in range(case["layers"]):
        pool = bd.Pool(projs, case["slots"], max(ranks), case["T"], weight_formats=fmt)
        for slot in _used(case, seed):
            z = _adapter(projs, ranks[slot], seed, layer, slot).view(torch.int16).cpu().numpy().view(np.uint16)
            pool.load_adapter(slot, ranks[slot], SCALE, *_split(z, projs, ranks[slot]))
        X, W, out = [], [], []
        for i, p in enumerate(projs):
            if case["part"] == "mlp" and p.name == "down":
                X.append(None)               # down reads H, which stays in the library
            elif p.name == "up" and case["part"] != "up":
                X.append(X[-1])              # gate's
            else:
                X.append(_x(case, seed, layer, p))
            w = _w(case, seed, layer, i, p)
            if case["fmt"] == "bf16":
                W.append(bd.pack_weight(w))
            else:
                W.append(bd.pack_weight_int4((w[0][:, 0::2] | (w[0][:, 1::2] << 4)).contiguous(), w[1].contiguous()))
            out.append(torch.empty(case["T"], p.d_out, dtype=torch.bfloat16, device="cuda"))
        s["layers"].append((pool, X, W, out))
    if case["graph"]:
        _calls(s)                            # warm up, then capture the step
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            _calls(s)
        s["graph"] = g
    return s


def _calls(s):
    for pool, X, W, out in s["layers"]:
        if s["part"] == "up":
            pool.forward_shard(0, X[0], W[0], s["ids"], out[0], segs=s["segs"])
        elif s["part"] == "layer":
            pool.forward_layer(range(len(X)), X, W, out, s["ids"], segs=s["segs"])
        else:
            pool.forward_mlp(bd.ACT_SILU_MUL, [0, 1], 2, X[0], W[:2], W[2], out[2], s["ids"], segs=s["segs"])


def run(s):
    if s["graph"] is not None:
        s["graph"].replay()
    else:
        _calls(s)
    return [out[2:] if s["part"] == "mlp" else out for _, _, _, out in s["layers"]]


# ---------------------------------------------------------------- what a pass needs

def work(case):
    """Every base weight, activation, used adapter factor and output once;
    the base products and the used adapters' shrink and expand."""
    projs, ranks, ids = _projs(case), _ranks(case, 0), _ids(case, 0)
    T, used = case["T"], np.unique(ids[ids >= 0])
    nbytes, flops, xs = 4 * T, 0, set()
    for p in projs:
        n = p.d_out
        nbytes += 2 * p.d_in * n if case["fmt"] == "bf16" else p.d_in * n // 2 + n * p.d_in // 64
        key = "gate" if p.name == "up" else p.name
        if key not in xs and not (case["part"] == "mlp" and p.name == "down"):
            nbytes += 2 * T * p.d_in
        xs.add(key)
        if case["part"] != "mlp" or p.name == "down":
            nbytes += 2 * T * n
        flops += 2 * T * p.d_in * n
        per_rank = len(p.slices) * p.d_in + n
        nbytes += 2 * per_rank * sum(ranks[a] for a in used)
        flops += 2 * per_rank * sum(ranks[a] for a in ids if a >= 0)
    return {"bytes": float(nbytes * case["layers"]), "flops": float(flops * case["layers"])}


def tolerance(case):
    # bf16 outputs of fp32 sums: two correct implementations differ by a
    # rounding of the last bit of some outputs (of H too in the MLP)
    return {"rel": 6e-3, "max": 0.03} if case["part"] == "mlp" else {"rel": 4e-3, "max": 0.02}


def _project(x, w, A, B, ids, projs, i):
    y = x @ w.t()
    for a in A:
        rows = torch.from_numpy(np.flatnonzero(ids == a)).cuda()
        at = 0
        for j, o in enumerate(projs[i].slices):
            y[rows, at:at + o] += SCALE * (x[rows] @ A[a][i][j].double()) @ B[a][i][j].double()
            at += o
    return y


def exact(case, seed):
    projs, ranks, ids = _projs(case), _ranks(case, seed), _ids(case, seed)
    outs = []
    for layer in range(case["layers"]):
        A, B = {}, {}
        for a in np.unique(ids[ids >= 0]):
            A[a], B[a] = _split(_adapter(projs, ranks[a], seed, layer, int(a)), projs, ranks[a])
        ys = []
        for i, p in enumerate(projs):
            w = _w(case, seed, layer, i, p)
            if case["fmt"] == "int4":
                w = (w[0].double() - 8) * w[1].double().repeat_interleave(128, dim=1)
            if case["part"] == "mlp" and p.name == "down":
                x = torch.nn.functional.silu(ys[0]) * ys[1]
            else:
                x = _x(case, seed, layer, p).double()
            ys.append(_project(x, w.double(), A, B, ids, projs, i))
        outs.append(ys[2:] if case["part"] == "mlp" else ys)
    return outs
