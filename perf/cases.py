"""Measured cases of the verification library, through its public entry points.

A case names a call, a shape and the values' recipe.  Six calls:

  step       sd_verify_step, one whole chain verification step (segment caches)
  paged      sd_verify_step_paged, the same over a page pool
  sampled    sd_verify_step_sampled, with a warped target (T, top-k, top-p)
  tree       sd_verify_step_tree, a binary candidate tree
  attention  sd_verify_attention, one decoder layer's attention
  expand     sd_expand_layer, a draft tree grown layer by layer

Cache lengths are spread evenly between len_min and len_max (geometrically
with "spread": "log") and dealt to the requests in an order that the seed
draws, so a case's work does not depend on the seed.  Target logits are about
N(0, logit_scale^2), drafts are drawn from softmax(target + noise), and the
uniform draws are multiples of 2^-24, as everywhere in this repository.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2601_21622_amd as sd

_BASE = {"call": "step", "dtype": "bf16", "packed": True, "spread": "even", "logit_scale": 8.0, "noise": 1.0}


def _case(name, **kw):
    return dict(_BASE, name=name, **kw)


def listed():
    vicuna = dict(gamma=5, hq=32, hkv=32, dim=128, hidden=4096, vocab=32000)
    llama3 = dict(gamma=6, hq=32, hkv=8, dim=128, hidden=4096, vocab=128256)
    return [
        # The smallest call: one request of a tiny float32 target, all launches and host time.
        _case("tiny_f32_step", dtype="f32", packed=False, batch=1, gamma=4, hq=4, hkv=4, dim=64, hidden=256,
              vocab=1000, len_min=128, len_max=128),
        # A small float32 target (16 heads of 64) verifying a batch at full precision.
        _case("small_f32_step", dtype="f32", packed=False, batch=8, gamma=4, hq=16, hkv=16, dim=64, hidden=1024,
              vocab=32000, len_min=256, len_max=1024),
        # One interactive session on a 7B-shaped target: the latency of a lone user's step.
        _case("single_7b_step", batch=1, **vicuna, len_min=1024, len_max=1024),
        # An ordinary batch on a 7B-shaped target.
        _case("vicuna7b_step", batch=8, **vicuna, len_min=512, len_max=2048),
        # One draft serving many clients: 64 pooled requests of widely mixed lengths in 64-key pages.
        _case("pooled_paged_step", call="paged", page=64, batch=64, gamma=4, hq=32, hkv=32, dim=128, hidden=4096,
              vocab=32000, len_min=128, len_max=8192, spread="log"),
        # Odd sizes throughout: head dimension 64, 13 requests, a vocabulary no tile divides, row-major weights.
        _case("ragged_d64_step", packed=False, batch=13, gamma=3, hq=24, hkv=8, dim=64, hidden=1536, vocab=50021,
              len_min=37, len_max=3001),
        # An 8B-shaped grouped-query target with a large vocabulary, a full batch.
        _case("llama3_8b_step", batch=32, **llama3, len_min=4096, len_max=4096, logit_scale=16.0),
        # The largest: a 70B-shaped share with long contexts, its drafts mostly rejected.
        _case("llama70b_share_step", batch=16, gamma=8, hq=64, hkv=8, dim=128, hidden=8192, vocab=128256,
              len_min=16384, len_max=32768, logit_scale=16.0, noise=8.0),
        # Sampling with a nucleus cut over a large vocabulary.
        _case("llama3_8b_top_p", call="sampled", batch=32, **llama3, len_min=512, len_max=4096, logit_scale=4.0,
              temperature=1.0, top_k=0, top_p=0.9),
        # One grouped-query decoder layer of a half-full batch: the call a whole model makes once per layer.
        _case("llama3_8b_attention", call="attention", batch=16, **llama3, len_min=1000, len_max=8000),
        # A binary candidate tree of 31 nodes per request.
        _case("vicuna7b_tree31", call="tree", batch=8, **dict(vicuna, gamma=31), len_min=512, len_max=2048),
        # The draft side: a binary tree of depth 5 grown for a batch, one call per layer.
        _case("expand_tree", call="expand", batch=8, vocab=32000, top_k=2, depth=5),
    ]


# ---- drawn cases ------------------------------------------------------------

_MOST_BYTES, _MOST_FLOPS = 3.5e9, 2.8e11


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    call = rng.choices(["step", "paged", "sampled", "tree", "attention", "expand", "f32"],
                       [30, 10, 18, 12, 12, 8, 10])[0]
    if call == "expand":
        return {k: v for k, v in dict(_BASE, call=call, batch=_log(rng, 1, 64), vocab=_log(rng, 1000, 130000),
                                      top_k=rng.choice([2, 2, 3, 4, 8]), depth=rng.randint(2, 4)).items()}
    c = dict(_BASE)
    if call == "f32":
        c.update(dtype="f32", packed=False, batch=_log(rng, 1, 16), gamma=rng.randint(1, 7))
        c.update(hkv=rng.choice([4, 8, 16]), dim=rng.choice([64, 128]))
        c["hq"] = c["hkv"] * rng.choice([1, 1, 2, 4])
        c.update(hidden=32 * _log(rng, 8, 64), vocab=_log(rng, 1000, 50000))
        c["len_min"] = _log(rng, 16, 512)
        c["len_max"] = c["len_min"] + _log(rng, 1, 1500)
        return c
    c.update(call=call, batch=_log(rng, 1, 64), gamma=rng.choice([14, 30, 62, 12, 39]) if call == "tree"
             else rng.randint(1, 10), dim=rng.choice([64, 128, 128, 128]))
    if rng.random() < 0.4:
        c["hkv"] = rng.choice([8, 16, 32])
        c["hq"] = c["hkv"]
    else:
        c["hkv"] = rng.choice([2, 4, 8])
        most = 128 // (c["gamma"] + 1)
        c["hq"] = c["hkv"] * rng.choice([g for g in (2, 3, 4, 5, 8) if g <= most] or [1])
    c.update(hidden=rng.choice([32 * _log(rng, 32, 256), 256 * _log(rng, 4, 32)]), vocab=_log(rng, 4000, 130000),
             packed=rng.random() < 0.7, spread=rng.choice(["even", "log"]))
    c["len_min"] = c["gamma"] + 1 + _log(rng, 16, 4096)
    c["len_max"] = c["len_min"] + _log(rng, 1, 8192)
    if call == "paged":
        c["page"] = rng.choice([64, 128, 256])
    if call == "sampled":
        c["logit_scale"] = 4.0
        c["temperature"], c["top_k"], c["top_p"] = rng.choice(
            [(1.0, 0, 0.9), (0.8, 40, 0.9), (0.7, 50, 0.95), (0.9, 8, 1.0), (1.0, 0, 1.0), (0.6, 200, 0.95),
             (0.0, 0, 1.0)])
    return c


def draw(rng):
    while True:
        c = _draw_once(rng)
        w = work(c)
        if w["bytes"] <= _MOST_BYTES and w["flops"] <= _MOST_FLOPS:
            return c


# ---- inputs -----------------------------------------------------------------

def _lengths(c, seed=None):
    lo, hi, n = c["len_min"], c["len_max"], c["batch"]
    if n == 1:
        v = np.array([hi])
    elif c["spread"] == "log":
        v = np.rint(np.exp(np.linspace(math.log(lo), math.log(hi), n)))
    else:
        v = np.rint(np.linspace(lo, hi, n))
    v = v.astype(np.int32)
    return v if seed is None else np.random.default_rng(seed).permutation(v)


def _dims(c):
    return sd.Dims(c["batch"], c["gamma"], c["hq"], c["hkv"], c["dim"], c["hidden"], c["vocab"],
                   sd.SD_DTYPE_F32 if c["dtype"] == "f32" else sd.SD_DTYPE_BF16,
                   sd.SD_FLAG_PACKED_VOCAB if c["packed"] else 0)


def _parents(n):
    return np.array([i // 2 - 1 for i in range(n)], dtype=np.int32)


def _uniform(g, *shape):
    return torch.randint(0, 1 << 24, shape, generator=g, device="cuda").float() * 2.0 ** -24


def _inputs(c, seed):
    """Everything a step reads, in plain layouts (row-major weights, segment caches)."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    B, G, V = c["batch"], c["gamma"] + 1, c["vocab"]

    def normal(*shape, std=1.0, dtype=dt):
        return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std).to(dtype)

    x = {"kv_len": _lengths(c, seed)}
    seg = c["hkv"] * x["kv_len"].astype(np.int64) * c["dim"]
    x["kv_off"] = np.concatenate([[0], np.cumsum(seg)[:-1]]).astype(np.int64)
    x["q"] = normal(B, G, c["hq"], c["dim"])
    x["k"], x["v"] = normal(int(seg.sum())), normal(int(seg.sum()))
    if c["call"] == "attention":
        return x
    x["hidden"] = normal(B * G, c["hidden"])
    x["w"] = normal(V, c["hidden"], std=c["logit_scale"] / math.sqrt(c["hidden"]))
    x["u"] = _uniform(g, B, G)
    # A stand-in for the draft model: the target's logits plus noise.
    z = torch.matmul(x["hidden"], x["w"].t()).float()
    z += normal(B * G, V, std=c["noise"], dtype=torch.float32)
    if c["call"] == "tree":
        # Sibling j of a position proposes the draft's j-th ranked token there.
        top = torch.topk(z, 2, dim=1).indices.view(B, G, 2)
        par = _parents(c["gamma"])
        x["tokens"] = torch.stack([top[:, int(p) + 1, i % 2] for i, p in enumerate(par)], 1).int().contiguous()
        x["parent"] = torch.from_numpy(np.tile(par, (B, 1))).cuda()
    else:
        z = z.view(B, G, V)[:, :c["gamma"]].contiguous()
        if c["call"] == "sampled":
            z /= max(c["temperature"], 0.05)
            if c["top_k"]:
                z.masked_fill_(z < torch.topk(z, c["top_k"], dim=2).values[..., -1:], -math.inf)
        x["q_draft"] = torch.softmax(z, 2)
        gumbel = -torch.log(-torch.log(torch.rand(z.shape, generator=g, device="cuda").clamp_(1e-9, 1 - 1e-7)))
        x["draft"] = torch.argmax(z + gumbel, 2).int()
    return x


def _pages(c, x):
    """The segment caches moved into a pool whose requests grew a page at a time in turn."""
    P, Hkv, D = c["page"], c["hkv"], c["dim"]
    need = [-(-int(n) // P) for n in x["kv_len"]]
    pool = sd.KVPool(sum(need), P)
    for p in range(max(need)):
        for b, n in enumerate(x["kv_len"]):
            if p < need[b]:
                pool.reserve(b, min(int(n), (p + 1) * P))
    table = pool.block_table(range(c["batch"]), max(need))
    pool.close()
    out = []
    for name in ("k", "v"):
        pages = torch.zeros((sum(need), Hkv, P, D), dtype=x[name].dtype, device="cuda")
        for b, n in enumerate(x["kv_len"]):
            o, n = int(x["kv_off"][b]), int(n)
            rows = torch.zeros((Hkv, need[b] * P, D), dtype=x[name].dtype, device="cuda")
            rows[:, :n] = x[name][o:o + Hkv * n * D].view(Hkv, n, D)
            pages[torch.from_numpy(table[b, :need[b]].astype(np.int64)).cuda()] = (
                rows.view(Hkv, need[b], P, D).transpose(0, 1))
        out.append(pages)
    return out[0], out[1], sd.KVPages.of(torch.from_numpy(table).cuda(), P, sum(need))


def _expand_layers(c):
    """Expand descriptors of the layers of a full tree, and its node count."""
    k, layers, first, nodes = c["top_k"], [], 0, sum(c["top_k"] ** (i + 1) for i in range(c["depth"]))
    frontier0, F = -1, 1
    for _ in range(c["depth"]):
        layers.append(sd.Expand(c["batch"], F, c["vocab"], k, frontier0, first, nodes))
        frontier0, first, F = first, first + F * k, F * k
    return layers, nodes


def _draft_layers(c, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    return [torch.randn((c["batch"], e.frontier, c["vocab"]), generator=g, device="cuda") * 4.0
            for e in _expand_layers(c)[0]]


def prepare(case, seed):
    c = case
    if c["call"] == "expand":
        layers, nodes = _expand_layers(c)
        new = lambda dt: torch.zeros((c["batch"], nodes), dtype=dt, device="cuda")  # noqa: E731
        return {"call": "expand", "layers": list(zip(layers, _draft_layers(c, seed))), "tokens": new(torch.int32),
                "parent": new(torch.int32), "q_child": new(torch.float32)}
    x = _inputs(c, seed)
    dims = _dims(c)
    s = {"call": c["call"], "dims": dims, "scale": 1.0 / math.sqrt(c["dim"]), **x}
    B, G, V = c["batch"], c["gamma"] + 1, c["vocab"]

    def new(*shape, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device="cuda")

    s["attn"] = torch.empty_like(x["q"])
    s["ws"] = new(sd.sd_workspace_bytes(dims, int(x["kv_len"].max())), dtype=torch.uint8)
    if c["call"] == "attention":
        return s
    if c["packed"]:
        s["w"] = new(sd.sd_vocab_packed_bytes(dims) // 2, dtype=torch.bfloat16)
        sd.sd_pack_vocab(dims, x["w"], s["w"])
    if c["call"] == "paged":
        s["k"], s["v"], s["pages"] = _pages(c, x)
    s["logits"], s["lse"] = new(B * G, V), new(B * G)
    s["accept_len"], s["new_kv_len"] = new(B, dtype=torch.int32), new(B, dtype=torch.int32)
    s["out_tok"] = new(B, G, dtype=torch.int32)
    if c["call"] == "tree":
        s["out_node"] = new(B, G, dtype=torch.int32)
    if c["call"] == "sampled":
        s["sampling"] = sd.Sampling(c["temperature"], c["top_k"], c["top_p"])
        s["min_logit"] = new(B * G)
    return s


def run(s):
    call = s["call"]
    if call == "expand":
        for e, logits in s["layers"]:
            sd.sd_expand_layer(e, logits, s["tokens"], s["parent"], s["q_child"])
        return {k: s[k] for k in ("tokens", "parent", "q_child")}
    cache = (s["dims"], s["q"], s["k"], s["v"])
    if call == "attention":
        sd.sd_verify_attention(*cache, s["kv_off"], s["kv_len"], s["scale"], s["attn"], s["ws"])
        return {"attn": s["attn"]}
    outs = ["attn", "logits", "lse", "accept_len", "out_tok", "new_kv_len"]
    if call == "tree":
        sd.sd_verify_step_tree(*cache, s["kv_off"], s["kv_len"], s["parent"], s["scale"], s["hidden"], s["w"],
                               s["tokens"], s["u"], s["attn"], s["logits"], s["lse"], s["accept_len"], s["out_tok"],
                               s["out_node"], s["new_kv_len"], s["ws"])
        outs.append("out_node")
    elif call == "sampled":
        sd.sd_verify_step_sampled(s["dims"], s["sampling"], *cache[1:], s["kv_off"], s["kv_len"], s["scale"],
                                  s["hidden"], s["w"], s["q_draft"], s["draft"], s["u"], s["attn"], s["logits"],
                                  s["lse"], s["min_logit"], s["accept_len"], s["out_tok"], s["new_kv_len"], s["ws"])
        outs.append("min_logit")
    elif call == "paged":
        sd.sd_verify_step_paged(*cache, s["pages"], s["kv_len"], s["scale"], s["hidden"], s["w"], s["q_draft"],
                                s["draft"], s["u"], s["attn"], s["logits"], s["lse"], s["accept_len"], s["out_tok"],
                                s["new_kv_len"], s["ws"])
    else:
        sd.sd_verify_step(*cache, s["kv_off"], s["kv_len"], s["scale"], s["hidden"], s["w"], s["q_draft"], s["draft"],
                          s["u"], s["attn"], s["logits"], s["lse"], s["accept_len"], s["out_tok"], s["new_kv_len"],
                          s["ws"])
    return {k: s[k] for k in outs}


# ---- what a pass needs ------------------------------------------------------

def work(case):
    c = case
    if c["call"] == "expand":
        rows = c["batch"] * sum(c["top_k"] ** i for i in range(c["depth"]))
        return {"bytes": 4 * rows * c["vocab"] + 12 * rows * c["top_k"], "flops": 2 * rows * c["vocab"]}
    es = 4 if c["dtype"] == "f32" else 2
    B, G, V, K = c["batch"], c["gamma"] + 1, c["vocab"], c["hidden"]
    keys = int(_lengths(c).sum())
    n = 2 * es * keys * c["hkv"] * c["dim"] + 2 * es * B * G * c["hq"] * c["dim"]
    f = 4 * keys * G * c["hq"] * c["dim"]
    if c["call"] != "attention":
        # Weights and hidden rows read, logits written; the draft distribution of one position per request.
        n += es * K * (V + B * G) + 4 * B * G * V + (0 if c["call"] == "tree" else 4 * B * V)
        f += 2 * B * G * K * V
    return {"bytes": n, "flops": f}


def tolerance(case):
    if case["call"] == "expand":
        return {"rel": 1e-5}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}
    # bfloat16 attention outputs and probabilities; the logits are float32 sums of bfloat16 products.
    return {"rel": 1e-2, "max": 0.1, "differ": 0.01}


def _exact_attention(c, x):
    B, G, D, Hkv = c["batch"], c["gamma"] + 1, c["dim"], c["hkv"]
    group = c["hq"] // Hkv
    out = torch.empty((B, G, c["hq"], D), dtype=torch.float64, device="cuda")
    tail = torch.tril(torch.ones((G, G), dtype=torch.bool))
    if c["call"] == "tree":
        tail = torch.zeros((G, G), dtype=torch.bool)
        for g in range(G):
            p = g
            while p > 0:
                tail[g, p] = True
                p = int(_parents(c["gamma"])[p - 1]) + 1
            tail[g, 0] = True
    for b, L in enumerate(int(n) for n in x["kv_len"]):
        o = int(x["kv_off"][b])
        k, v = (x[n][o:o + Hkv * L * D].view(Hkv, L, D).double() for n in ("k", "v"))
        q = x["q"][b].double().view(G, Hkv, group, D).permute(1, 0, 2, 3).reshape(Hkv, G * group, D)
        sc = torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(D)
        see = torch.ones((G, L), dtype=torch.bool)
        see[:, L - G:] = tail
        sc.masked_fill_(~see.repeat_interleave(group, 0).cuda(), -math.inf)
        o = torch.matmul(torch.softmax(sc, 2), v)
        out[b] = o.view(Hkv, G, group, D).permute(1, 0, 2, 3).reshape(G, c["hq"], D)
    return out


def _exact_warp(c, logits):
    """Row normalisers and smallest kept logits of the warped target."""
    if c["temperature"] == 0.0:
        return torch.zeros_like(logits[:, 0]), torch.full_like(logits[:, 0], math.inf)
    z = logits / c["temperature"]
    cut = torch.full_like(z[:, 0], -math.inf)
    if c["top_k"]:
        cut = torch.topk(z, c["top_k"], dim=1).values[:, -1]
    if c["top_p"] < 1.0:
        s = torch.sort(z, dim=1, descending=True).values
        s.masked_fill_(s < cut[:, None], -math.inf)
        mass = torch.cumsum(torch.softmax(s, 1), 1)
        cut = s.gather(1, (mass < c["top_p"]).sum(1, keepdim=True).clamp_(max=s.shape[1] - 1))[:, 0]
    lse = torch.logsumexp(z.masked_fill(z < cut[:, None], -math.inf), 1)
    return lse, cut * c["temperature"]


def exact(case, seed):
    c = case
    if c["call"] == "expand":
        layers, nodes = _expand_layers(c)
        q = torch.empty((c["batch"], nodes), dtype=torch.float64, device="cuda")
        for e, z in zip(layers, _draft_layers(c, seed)):
            p = torch.topk(torch.softmax(z.double(), 2), c["top_k"], dim=2).values
            q[:, e.first_child:e.first_child + e.frontier * c["top_k"]] = p.reshape(c["batch"], -1)
        return {"tokens": None, "parent": None, "q_child": q}
    x = _inputs(c, seed)
    out = {"attn": _exact_attention(c, x)}
    if c["call"] == "attention":
        return out
    h, step = x["hidden"].double(), 8192
    logits = torch.cat([torch.matmul(h, x["w"][i:i + step].double().t().contiguous())
                        for i in range(0, c["vocab"], step)], 1)
    out.update(logits=logits, lse=torch.logsumexp(logits, 1), accept_len=None, out_tok=None, new_kv_len=None)
    if c["call"] == "tree":
        out["out_node"] = None
    if c["call"] == "sampled":
        out["lse"], out["min_logit"] = _exact_warp(c, logits)
    return out
