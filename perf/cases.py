"""The layer calls whose speed this repository is measured by.

A program that uses this library holds the weights of one Mixture-of-Experts
layer, a workspace and output buffers, and calls the layer once per decode step
or prefill batch.  Each case is one such call: its shape, storage type, batch,
pruning rule and expert popularity.  ``prepare`` makes what the program holds,
``run`` is the call, ``exact`` the same results in float64 plain torch.
"""
from __future__ import annotations

import math

import torch

from paper_2606_29982_amd import caee

DEV = torch.device("cuda:0")

# The DeepSeek-R1-shaped layer of this repository's benchmark and tests.
R1 = dict(d=7168, f=2048, E=256, n_group=8, topk_group=4, k=8, n_shared=1, scaling=2.5, bias=True)
# A generic fine-grained layer: fewer, smaller experts, an odd multiple of 128
# as the expert width, no groups, two shared experts.
FINE = dict(d=2048, f=1408, E=64, n_group=1, topk_group=1, k=6, n_shared=2, scaling=1.0, bias=False)
# The small float32 layer of the parity tests.
TINY = dict(d=256, f=128, E=16, n_group=4, topk_group=2, k=4, n_shared=1, scaling=1.0, bias=False)


def _case(shape, **kw):
    c = dict(entry="layer", dtype="bf16", layout="tiled", rule="max", tau=0.0, n_bins=1, skew=0.0)
    c.update(shape)
    c.update(kw)
    return c


def listed():
    return [
        # The smallest call: launches, routing latency and the host path.
        _case(TINY, name="f32-small-16", dtype="f32", layout="rowmajor", T=16, tau=0.1, n_bins=4),
        # One user's decode step with the bf16 layer: nine experts stream.
        _case(R1, name="bf16-decode-1", T=1, n_bins=8, skew=1.1),
        # A few users, experts pruned by the on-device rule (summed importance).
        _case(R1, name="bf16-decode-8-sum", T=8, n_bins=8, skew=1.1, rule="sum", tau=0.6),
        # The benchmark's headline: 32 users, evenly used experts, no pruning.
        _case(R1, name="bf16-decode-32", T=32),
        # A full decode batch with popular experts, pruned by the offloading rule.
        _case(R1, name="bf16-decode-128-cir", T=128, n_bins=8, skew=1.1, rule="cir", tau=0.8),
        # A prompt of 2048 tokens through the bf16 layer.
        _case(R1, name="bf16-prefill-2048", T=2048),
        # One user's decode step with 8-bit weights, what a W8 deployment runs.
        _case(R1, name="fp8-decode-1", dtype="fp8", T=1, n_bins=8, skew=1.1, tau=0.05),
        # The on-device deployment at 128 requests: 8-bit, SUM rule, popular experts.
        _case(R1, name="fp8-decode-128-sum", dtype="fp8", T=128, n_bins=16, skew=1.1, rule="sum", tau=0.8),
        # The benchmark's 8-bit prefill.
        _case(R1, name="fp8-prefill-4096", dtype="fp8", T=4096, n_bins=8, tau=0.05),
        # The expert FFN alone, under a program's own router: an odd batch, a
        # width that is no multiple of 256, several shared experts.
        _case(FINE, name="bf16-ffn-509", entry="ffn", T=509, skew=1.1),
        # Routing and pruning alone, as an expert-parallel dispatcher calls it.
        _case(R1, name="route-4096-sum", entry="route", T=4096, n_bins=16, skew=1.1, rule="sum", tau=4.0),
        # An offloaded layer whose experts have all been fetched: the steady
        # state of a decode loop, with the call's one host synchronisation.
        _case(FINE, name="bf16-offload-16", entry="offload", T=16, skew=1.2),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def draw(rng):
    """One more case of the listed ranges: decode to prefill batches (odd ones
    mostly), the R1 layer or smaller ones, every storage type, rule and entry."""
    entry = rng.choice(["layer"] * 6 + ["noalloc", "ffn", "route", "offload"])
    dtype = rng.choice(["bf16", "bf16", "fp8", "fp8", "f32"])
    if entry == "offload":
        dtype = rng.choice(["bf16", "f32"])
    if dtype != "f32" and entry != "offload" and rng.random() < 0.45:
        shape = dict(R1)
    else:
        E, n_group = rng.choice([(16, 4), (32, 1), (48, 3), (64, 1), (64, 8), (96, 3), (128, 4), (128, 1)])
        topk_group = rng.randint(max(1, n_group // 2), n_group)
        small = dtype == "f32" or entry == "offload"
        d = 128 * _log_int(rng, 2, 8 if small else 32)
        f = 128 * _log_int(rng, 1, 8 if small else 16)
        k = min(rng.choice([2, 4, 6, 8]), topk_group * (E // n_group))
        shape = dict(d=d, f=f, E=E, n_group=n_group, topk_group=topk_group, k=k, n_shared=rng.randint(0, 2),
                     scaling=rng.choice([1.0, 2.5]), bias=rng.random() < 0.5)
    hi = {"bf16": 2048, "fp8": 4096, "f32": 256}[dtype]
    if entry == "noalloc":
        hi = 96 if shape["d"] > 2048 else 32
    elif entry == "offload":
        hi = 64
    T = _log_int(rng, 1, hi)
    rule = rng.choice(["max", "max", "sum", "cir"])
    tau = {"max": rng.choice([0.0, 0.05, 0.1]), "cir": rng.choice([0.7, 0.8, 0.9]),
           "sum": rng.choice([0.6, 0.8, 1.2])}[rule]
    n_bins = rng.choice([1, 4, 8])
    if n_bins > 1 and shape["E"] % n_bins:
        n_bins = 1
    if entry in ("ffn", "offload"):
        # the FFN prunes nothing; an offloaded call's pruning depends on what
        # the calls before it left in the cache
        rule, tau, n_bins = "max", 0.0, 1
    layout = "rowmajor" if shape["d"] < 4096 and rng.random() < 0.2 else "tiled"
    return _case(shape, entry=entry, dtype=dtype, T=T, rule=rule, tau=tau, n_bins=n_bins, layout=layout,
                 skew=rng.choice([0.0, 1.1]))


# ---------------------------------------------------------------------------
# Inputs, from the seed alone.
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}


def _x_dtype(case):
    return "f32" if case["dtype"] == "f32" else "bf16"


def _gen(seed, stream, device):
    g = torch.Generator(device=device)
    g.manual_seed((int(seed) * 1000003 + stream) & 0x7FFFFFFFFFFFFFFF)
    return g


def _zipf(E, s):
    p = torch.arange(1, E + 1, dtype=torch.float64) ** -s
    return p / p.sum()


def _router_inputs(case, seed):
    """Logits N(0,1) plus a Zipf popularity offset over a random expert order, a
    small selection bias, and a cost table (bytes of an expert times a skewed
    factor of mean one), made on the host and small."""
    T, E = case["T"], case["E"]
    g = _gen(seed, 1, "cpu")
    logits = torch.randn((T, E), generator=g)
    if case["skew"]:
        p = _zipf(E, case["skew"])[torch.randperm(E, generator=g)]
        logits = logits + torch.log(E * p).to(torch.float32)
    bias = torch.randn(E, generator=g) * 0.01 if case["bias"] else None
    q = _zipf(E, 1.1)[torch.randperm(E, generator=g)]
    size = 3 * case["d"] * case["f"] * {"f32": 4, "bf16": 2, "fp8": 1}[case["dtype"]]
    cost = ((0.5 + 0.5 * E * q) * size).to(torch.float32)
    nb = case["n_bins"]
    bins = (torch.arange(E, dtype=torch.int32) // (E // nb)).to(torch.int32) if nb > 1 else None
    return logits.contiguous(), bias, cost, bins


def _hidden(case, seed):
    return torch.randn((case["T"], case["d"]), generator=_gen(seed, 2, DEV), device=DEV).to(_TORCH[_x_dtype(case)])


def _own_topk(case, logits):
    """A program's own router: the k best sigmoid scores, normalised."""
    s = torch.sigmoid(logits)
    w, ids = torch.topk(s, case["k"], dim=1)
    return ids.to(torch.int32).contiguous(), (case["scaling"] * w / w.sum(1, keepdim=True)).contiguous()


def _blocks_e4m3(w):
    """E4M3 codes and fp32 scales per 128x128 block of float32 [n][R][C]."""
    n, R, C = w.shape
    b = w.view(n, R // 128, 128, C // 128, 128)
    amax = b.abs().amax(dim=(2, 4))
    scale = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
    codes = (b / scale[:, :, None, :, None]).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn)
    return codes.view(torch.uint8).view(n, R, C), scale.contiguous()


def _weights(case, seed):
    """Row-major expert weights N(0, 0.02), drawn on the GPU 16 experts at a time."""
    d, f, E, S = case["d"], case["f"], case["E"], case["n_shared"]
    dt = torch.uint8 if case["dtype"] == "fp8" else _TORCH[case["dtype"]]
    g = _gen(seed, 3, DEV)
    W = {}
    for prefix, n in (("", E), ("sh_", S)):
        for name, R, C in (("w13", 2 * f, d), ("w2", d, f)):
            out = torch.empty((n, R, C), dtype=dt, device=DEV)
            if case["dtype"] == "fp8":
                W[prefix + name + "_scale"] = torch.empty((n, R // 128, C // 128), device=DEV)
            for i in range(0, n, 16):
                m = min(16, n - i)
                if case["dtype"] == "fp8":
                    w = torch.empty((m, R, C), dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g)
                    codes, sc = _blocks_e4m3(w.float())
                    out[i:i + m].copy_(codes)
                    W[prefix + name + "_scale"][i:i + m].copy_(sc)
                else:
                    out[i:i + m].normal_(0.0, 0.02, generator=g)
            W[prefix + name] = out
    if S == 0:
        W = {key: v for key, v in W.items() if not key.startswith("sh_")}
    return W


def _layer(case, **kw):
    return caee.Layer(T=case["T"], d=case["d"], f=case["f"], E=case["E"], n_group=case["n_group"],
                      topk_group=case["topk_group"], k=case["k"], n_shared=case["n_shared"],
                      routed_scaling=case["scaling"], tau=case["tau"], n_bins=case["n_bins"],
                      w_dtype=case["dtype"], x_dtype=_x_dtype(case), y_dtype=_x_dtype(case),
                      importance=case["rule"], **kw)


def prepare(case, seed):
    s = {"case": case, "layer": _layer(case)}
    logits, bias, cost, bins = (None if t is None else t.to(DEV) for t in _router_inputs(case, seed))
    s.update(logits=logits, bias=bias, cost=cost, bins=bins)
    s["out"] = caee.alloc_route_out(s["layer"], DEV)
    if case["entry"] != "noalloc":
        s["ws"] = caee.alloc_workspace(s["layer"], DEV)
    if case["entry"] == "route":
        return s
    s["x"] = _hidden(case, seed)
    s["y"] = torch.empty((case["T"], case["d"]), dtype=_TORCH[_x_dtype(case)], device=DEV)
    W = _weights(case, seed)
    if case["layout"] == "tiled":
        W = caee.pack_weights(W, case["dtype"])
    if case["entry"] == "ffn":
        s["ids"], s["w"] = _own_topk(case, logits)
    if case["entry"] == "offload":
        # every expert in page-locked host memory, as many cache slots as experts
        E = case["E"]
        host = caee.pin_host_weights(W)
        s13, s2 = caee.alloc_slots(s["layer"], E + 4, DEV)
        size = W["w13"][0].nbytes + W["w2"][0].nbytes
        s["offload"] = caee.Offload(s["layer"], host["w13"], host["w2"], s13, s2, W.get("sh_w13"), W.get("sh_w2"),
                                    E, 4, size / 56e9 * 1e6, 4, host["layout"])
        torch.cuda.synchronize()
    else:
        s["W"] = W
    return s


def run(s):
    e = s["case"]["entry"]
    if e == "layer":
        caee.moe_layer(s["layer"], s["x"], s["logits"], s["bias"], s["cost"], s["bins"], s["W"], s["y"], s["ws"],
                       s["out"])
    elif e == "noalloc":
        caee.moe_layer_noalloc(s["layer"], s["x"], s["logits"], s["bias"], s["cost"], s["bins"], s["W"], s["y"],
                               s["out"])
    elif e == "ffn":
        caee.expert_ffn(s["layer"], s["x"], s["ids"], s["w"], s["W"], s["y"], s["ws"])
        return {"y": s["y"]}
    elif e == "route":
        caee.route_prune(s["layer"], s["logits"], s["bias"], s["cost"], s["bins"], s["out"], s["ws"])
        return dict(s["out"])
    else:
        s["offload"](s["layer"], s["x"], s["logits"], s["bias"], s["y"], s["ws"], s["out"])
        # the cost table is the residency, so the loads change from the first
        # call to the next: they are not part of the answer
        return {"y": s["y"], "topk_ids": s["out"]["topk_ids"], "topk_w": s["out"]["topk_w"]}
    return {"y": s["y"], **s["out"]}


# ---------------------------------------------------------------------------
# The same in float64.
def _route64(case, logits, bias, cost, bins):
    """Routing, pruning and compensation, host tensors in and out: K_final
    (-1 in empty slots), its weights, the executed experts, the bin loads."""
    T, E, k, nb = case["T"], case["E"], case["k"], case["n_bins"]
    tau = float(torch.tensor(case["tau"], dtype=torch.float32))
    s = torch.sigmoid(logits.double())
    key = s + (0.0 if bias is None else bias.double())
    gs = key.view(T, case["n_group"], -1)
    gscore = torch.topk(gs, min(2, gs.shape[2]), dim=2).values.sum(2)
    gsel = torch.zeros_like(gscore, dtype=torch.bool).scatter_(1, torch.topk(gscore, case["topk_group"], 1).indices, True)
    masked = torch.where(gsel.repeat_interleave(E // case["n_group"], 1), key, -math.inf)
    ids = torch.topk(masked, k, 1).indices
    sk = s.gather(1, ids)
    G = sk / sk.sum(1, keepdim=True)
    act = torch.zeros(E, dtype=torch.bool)
    act[ids.flatten()] = True
    imp = torch.zeros(E, dtype=torch.float64).scatter_reduce_(0, ids.flatten(), G.flatten(), "amax")
    must = torch.zeros(E, dtype=torch.bool)
    if case["rule"] == "sum":
        imp = torch.zeros(E, dtype=torch.float64).index_add_(0, ids.flatten(), G.flatten())
        must = act & (imp >= tau)
    elif case["rule"] == "max":
        must[ids[G >= tau]] = True
    else:
        order = torch.sort(sk, dim=1, descending=True, stable=True).indices
        ss = sk.gather(1, order)
        cum = ss.cumsum(1) / ss.sum(1, keepdim=True)
        before = torch.cat([torch.zeros(T, 1, dtype=torch.float64), cum[:, :-1]], 1)
        must[ids.gather(1, order)[before < tau]] = True
        must[ids.gather(1, order)[:, 0]] = True
    b = torch.zeros(E, dtype=torch.long) if bins is None else bins.long()
    c = cost.double()

    def expand(must):
        load = torch.zeros(nb, dtype=torch.float64).index_add_(0, b[must], c[must])
        base, trans, final = float(load.max()), must.clone(), load.clone()
        for e in sorted(torch.nonzero(act & ~must).flatten().tolist(), key=lambda e: (-float(imp[e]), e)):
            if float(final[b[e]]) + float(c[e]) <= base:
                trans[e] = True
                final[b[e]] += c[e]
        return load, trans, final

    load, trans, final = expand(must)
    if not bool(trans.any()):
        top = torch.max(G, 1).values
        must[torch.where(G == top[:, None], ids, E).min(1).values] = True
        load, trans, final = expand(must)
    loads = torch.stack([torch.zeros(nb, dtype=torch.float64).index_add_(0, b[act], c[act]), load, final])
    # compensation: kept experts first, freed slots from the rest of A_trans by key
    in_k = torch.zeros((T, E), dtype=torch.bool).scatter_(1, ids, True)
    keep = in_k & trans
    score = torch.where(keep, key + 1e3, torch.where(trans, key, -math.inf))
    fin = torch.topk(score, k, 1)
    sel = torch.where(torch.isfinite(fin.values), fin.indices, -1)
    rank = torch.where(sel >= 0, key.gather(1, sel.clamp(min=0)), -math.inf)
    sel = sel.gather(1, torch.sort(rank, dim=1, descending=True, stable=True).indices)
    sw = torch.where(sel >= 0, s.gather(1, sel.clamp(min=0)), 0.0)
    rs = float(torch.tensor(case["scaling"], dtype=torch.float32))
    return sel, rs * sw / sw.sum(1, keepdim=True), trans, loads


def _quant64(v):
    """Values after the 8-bit path's activation quantiser (per row and 128
    columns, in fp32), as float64."""
    b = v.float().view(v.shape[0], -1, 128)
    amax = b.abs().amax(2, keepdim=True)
    sc = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
    q = (b / sc).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return (q.double() * sc.double()).view(v.shape)


def _ffn64(case, x, ids, w, W):
    fp8 = case["dtype"] == "fp8"
    f = case["f"]
    xd = _quant64(x) if fp8 else x.double()
    ids, w = ids.to(DEV), w.double().to(DEV)

    def matrix(name, i):
        m = W[name][i]
        if not fp8:
            return m.double()
        sc = W[name + "_scale"][i].double().repeat_interleave(128, 0).repeat_interleave(128, 1)
        return m.view(torch.float8_e4m3fn).double() * sc

    def expert(prefix, i, rows):
        gu = rows @ matrix(prefix + "w13", i).T
        h = torch.nn.functional.silu(gu[:, :f]) * gu[:, f:]
        return (_quant64(h) if fp8 else h) @ matrix(prefix + "w2", i).T

    y = torch.zeros((case["T"], case["d"]), dtype=torch.float64, device=DEV)
    for e in torch.unique(ids[ids >= 0]).tolist():
        t, j = torch.nonzero(ids == e, as_tuple=True)
        y.index_add_(0, t, expert("", e, xd[t]) * w[t, j][:, None])
    for i in range(case["n_shared"]):
        y += expert("sh_", i, xd)
    return y


def exact(case, seed):
    r = _router_inputs(case, seed)
    e = case["entry"]
    if e == "ffn":
        ids, w = _own_topk(case, r[0].to(DEV))
        return {"y": _ffn64(case, _hidden(case, seed), ids, w, _weights(case, seed))}
    if e == "offload":
        r = (r[0], r[1], torch.zeros_like(r[2]), None)
    ids, w, _, loads = _route64(case, *r)
    if e == "route":
        return {"topk_w": w, "bin_loads": loads}
    y = _ffn64(case, _hidden(case, seed), ids, w, _weights(case, seed))
    return {"y": y, "topk_w": w} if e == "offload" else {"y": y, "topk_w": w, "bin_loads": loads}


# ---------------------------------------------------------------------------
def work(case):
    """The weights of the executed experts once (the experts that one batch of
    these inputs executes), the hidden states, logits and tables read, the
    outputs written; the products of every (token, expert) row."""
    T, d, f, k, S = (case[n] for n in ("T", "d", "f", "k", "n_shared"))
    e = case["entry"]
    router = T * case["E"] * 4 + 12 * case["E"]
    result = T * k * 12
    if e == "route":
        return {"bytes": router + result, "flops": 0}
    r = _router_inputs(case, 0)
    if e == "ffn":
        ids = _own_topk(case, r[0])[0]
        experts, rows, router, result = int(torch.unique(ids).numel()), T * k, T * k * 8, 0
    else:
        ids, _, trans, _ = _route64(case, *(r if e != "offload" else (r[0], r[1], torch.zeros_like(r[2]), None)))
        experts, rows = int(torch.unique(ids[ids >= 0]).numel()), int((ids >= 0).sum())
    wb = 3 * d * f * {"f32": 4, "bf16": 2, "fp8": 1}[case["dtype"]]
    if case["dtype"] == "fp8":
        wb += 4 * 3 * (f // 128) * (d // 128)
    xb = 4 if case["dtype"] == "f32" else 2
    return {"bytes": (experts + S) * wb + 2 * T * d * xb + router + result, "flops": (rows + T * S) * 6 * d * f}


def tolerance(case):
    """About four times the distance to ``exact``: 3e-8 for the fp32 routing
    weights, 3e-7 to 5e-7 for float32 layers, 0.0023 for bf16 (SwiGLU rows and
    outputs rounded to 8 significant bits), 0.015 for the 8-bit path (a sum that
    differs moves SwiGLU values across a step of their 3-bit codes)."""
    if case["entry"] == "route":
        return {"rel": 1e-6, "max": 1e-5}
    return {"f32": {"rel": 5e-6, "max": 1e-3}, "bf16": {"rel": 1e-2, "max": 0.1},
            "fp8": {"rel": 0.03, "max": 0.3}}[case["dtype"]]
