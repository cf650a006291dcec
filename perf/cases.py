"""The work that programs have this library do, as cases that can be timed and checked.

A case is one call (or the two or three calls that belong together) through the public
entry points of `paper_2505_23219_amd.binding`, on the shapes of this repository's named
workloads, of its benchmark's sweep and of its tests.  `listed()` are fixed cases, `draw()`
gives more of the same ranges; `prepare` makes the inputs from a seed, `run` is one pass,
`exact` the same outputs in 64 bits from plain torch.
"""
import hashlib
import math

import torch

from paper_2505_23219_amd import binding as B
from paper_2505_23219_amd import model
from paper_2505_23219_amd.workloads import ModelShape

ROPE_BASE, RMS_EPS = 10000.0, 1e-6


def listed():
    return [
        # The smallest model a program would run, one layer and its LM head over an 8-node
        # tree: launches and latency are all there is.
        {"name": "stack_tiny", "op": "stack", "nh": 4, "d": 64, "F": 688, "V": 1000, "L": 1, "M": 8, "kv": 128,
         "tree": "random"},
        # Plain decoding, one token at a time, in a 7B-shaped layer with a 2048-token context.
        {"name": "layer7b_decode", "op": "layer", "nh": 32, "d": 128, "F": 11008, "M": 1, "kv": 2048, "tree": "chain"},
        # The tree width that pays best in the paper (16 nodes), 1024 tokens of context.
        {"name": "layer7b_tree16", "op": "layer", "nh": 32, "d": 128, "F": 11008, "M": 16, "kv": 1024,
         "tree": "random"},
        # The widest tree the library takes: a 128-token draft sequence verified at once.
        {"name": "layer7b_chain128", "op": "layer", "nh": 32, "d": 128, "F": 11008, "M": 128, "kv": 2048,
         "tree": "chain"},
        # A small model whose sizes divide by nothing in particular (20 heads of 64, ragged
        # FFN, tree and context), as drafting and distilled models have them.
        {"name": "layer_ragged", "op": "layer", "nh": 20, "d": 64, "F": 3416, "M": 37, "kv": 777, "tree": "random"},
        # A 13B-shaped layer verifying a wide shallow tree over a long context.
        {"name": "layer13b_tree64", "op": "layer", "nh": 40, "d": 128, "F": 13824, "M": 64, "kv": 8192,
         "tree": "wide"},
        # The benchmark's step: 32 layers of a 7B shape and the LM head over a 64-node tree.
        {"name": "stack7b_tree64", "op": "stack", "nh": 32, "d": 128, "F": 11008, "V": 32000, "L": 32, "M": 64,
         "kv": 2048, "tree": "random"},
        # One linear layer called by itself, ragged in every direction, from a padded
        # activation buffer, fp32 result.
        {"name": "linear_ragged", "op": "linear", "M": 33, "N": 5003, "K": 4104, "pad": 24, "out16": False},
        # A wide projection of a small batch of rows, fp16 result.
        {"name": "linear_wide16", "op": "linear", "M": 16, "N": 12288, "K": 4096, "pad": 0, "out16": True},
        # Attention called by itself under a caller's verification pattern (several draft
        # sequences side by side), odd context length.
        {"name": "attention_masked", "op": "attention", "M": 48, "nh": 24, "d": 128, "kv": 3001, "mask": "sequences"},
        # Drafting: five heads, ten candidates each, on the last accepted node's hidden state.
        {"name": "draft7b", "op": "draft", "K": 5, "R": 10, "H": 4096, "V": 32000, "M": 64},
        # Acceptance from logits and commit of the accepted path in all 32 caches.
        {"name": "accept_commit7b", "op": "accept", "nh": 32, "d": 128, "V": 32000, "L": 32, "M": 64, "kv": 2048},
    ]


def _log(rng, lo, hi, step=1):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, v // step * step if step > 1 else v))


def draw(rng):
    op = rng.choice(["layer", "layer", "layer", "stack", "linear", "linear", "attention", "attention", "draft",
                     "accept"])
    M = _log(rng, 1, 128)
    if op in ("layer", "stack"):
        d = rng.choice([64, 128, 128])
        nh = _log(rng, 4, 40)
        F = max(8, int(nh * d * rng.uniform(2.2, 3.2)) // 8 * 8)
        c = {"op": op, "nh": nh, "d": d, "F": F, "M": M, "kv": _log(rng, 16, 8192),
             "tree": rng.choice(["chain", "random", "wide"])}
        if op == "stack":
            c.update(V=_log(rng, 1000, 32000), L=rng.randint(1, 8))
        return c
    if op == "linear":
        return {"op": op, "M": M, "N": _log(rng, 64, 32000), "K": _log(rng, 64, 13824, 8), "pad": 8 * rng.randint(0, 4),
                "out16": rng.random() < 0.5}
    if op == "attention":
        return {"op": op, "M": M, "nh": _log(rng, 2, 64), "d": rng.choice([64, 128, 128]), "kv": _log(rng, 16, 16384),
                "mask": rng.choice(["tree", "tree", "sequences"])}
    if op == "draft":
        return {"op": op, "K": rng.randint(1, 5), "R": rng.randint(1, 10), "H": _log(rng, 256, 4096, 8),
                "V": _log(rng, 1000, 32000), "M": M}
    return {"op": op, "nh": _log(rng, 4, 40), "d": rng.choice([64, 128]), "V": _log(rng, 1000, 64000),
            "L": rng.randint(1, 32), "M": M, "kv": _log(rng, 16, 4096)}


# ---- inputs -------------------------------------------------------------------------
def _gen(seed, *tags):
    g = torch.Generator(device="cuda")
    g.manual_seed(int.from_bytes(hashlib.sha256(repr((int(seed),) + tags).encode()).digest()[:7], "little"))
    return g


def _normal(shape, seed, *tags, std=1.0, mean=0.0):
    t = torch.randn(shape, generator=_gen(seed, *tags), device="cuda", dtype=torch.float32)
    return t.mul_(std).add_(mean).to(torch.float16)


def _parent(case, seed):
    """parent[] of the draft tree: a chain, a random tree of depth at most 5, or a wide
    shallow one (a root, M/2 children, grandchildren)."""
    M, kind = case["M"], case.get("tree", "random")
    r = torch.Generator().manual_seed(int(seed) * 7919 + M)
    parent, depth = [-1], [0]
    for i in range(1, M):
        if kind == "chain":
            p = i - 1
        else:
            if kind == "wide":
                ok = [0] if i <= M // 2 else list(range(1, M // 2 + 1))
            else:
                ok = [j for j in range(i) if depth[j] < 5]
            p = ok[int(torch.randint(len(ok), (1,), generator=r))]
        parent.append(p)
        depth.append(depth[p] + 1)
    return parent, depth


def _shape(case):
    return ModelShape("case", H=case["nh"] * case["d"], nh=case["nh"], d=case["d"], F=case["F"],
                      V=case.get("V", 1000), L=case.get("L", 1), rope_base=ROPE_BASE, rms_eps=RMS_EPS)


def _capacity(case):
    return (case["kv"] + case["M"] + 63) // 64 * 64


def _layer(case, seed, l):
    """Row-major fp16 weights of layer l: matrices N(0, 0.02), gains 1 + N(0, 0.02)."""
    H, F = case["nh"] * case["d"], case["F"]
    w = {n: _normal(s, seed, l, n, std=0.02) for n, s in
         (("Wqkv", (3 * H, H)), ("Wo", (H, H)), ("Wgu", (2 * F, H)), ("Wdown", (H, F)))}
    w.update({n: _normal((H,), seed, l, n, std=0.02, mean=1.0) for n in ("g_attn", "g_ffn")})
    return w


def _head(case, seed):
    H = case["nh"] * case["d"]
    return {"g_final": _normal((H,), seed, "g_final", std=0.02, mean=1.0),
            "Wlm": _normal((case["V"], H), seed, "Wlm", std=0.02)}


def _caches(case, seed, rows):
    """K [L, nh, cap, d] and V [L, nh, d, cap]: rows [0, rows) committed, N(0, 1), the rest zero."""
    L, nh, d, cap = case.get("L", 1), case["nh"], case["d"], _capacity(case)
    k = torch.zeros((L, nh, cap, d), dtype=torch.float16, device="cuda")
    v = torch.zeros((L, nh, d, cap), dtype=torch.float16, device="cuda")
    for l in range(L):
        k[l, :, :rows] = _normal((nh, rows, d), seed, l, "k")
        v[l, :, :, :rows] = _normal((nh, d, rows), seed, l, "v")
    return k, v


def _int32(values):
    return torch.tensor(values, dtype=torch.int32, device="cuda")


def _linear_inputs(case, seed):
    x = _normal((case["M"], case["K"] + case["pad"]), seed, "x")[:, :case["K"]]
    return x, _normal((case["N"], case["K"]), seed, "W", std=0.02)


def _attention_inputs(case, seed):
    M, nh, d = case["M"], case["nh"], case["d"]
    q = _normal((M, nh, d), seed, "q")
    k, v = _caches(case, seed, case["kv"] + M)
    if case["mask"] == "tree":
        parent, _ = _parent(case, seed)
        see = [0] * M
        for i in range(M):
            see[i] = (1 << i) | (see[parent[i]] if i else 0)
    else:       # draft sequences of 8 tokens side by side: a token sees its own sequence so far
        parent = None
        see = [sum(1 << j for j in range(i // 8 * 8, i + 1)) for i in range(M)]
    return q, k[0], v[0], parent, see


def _mask_words(see):
    def word(x):
        x &= (1 << 64) - 1
        return x - (1 << 64) if x >> 63 else x
    return torch.tensor([[word(s), word(s >> 64)] for s in see], dtype=torch.int64, device="cuda")


def _draft_inputs(case, seed):
    M, K, R, H, V = (case[n] for n in ("M", "K", "R", "H", "V"))
    # head accuracies fall with the head and, faster, with the candidate's rank
    acc = [[0.6 * 0.8 ** k * 0.35 ** r for r in range(R)] for k in range(K)]
    parent, rank, _ = B.ghd_tree_build(acc, M)
    M = len(parent)
    x = torch.randn((M, H), generator=_gen(seed, "x_final"), device="cuda", dtype=torch.float32) * 6.0
    # an accepted path: from a random node up to the root
    at, path = int(torch.randint(M, (1,), generator=torch.Generator().manual_seed(int(seed)))), []
    while at >= 0:
        path.insert(0, at)
        at = parent[at]
    res = [len(path), (int(seed) * 131 + 7) % V] + path + [0] * (M - len(path))
    return {"g": _normal((H,), seed, "g_final", std=0.02, mean=1.0),
            "W": _normal((K * V, H), seed, "heads", std=0.02), "x": x, "parent": parent, "rank": rank,
            "res": res, "last": path[-1]}


def _accept_inputs(case, seed):
    M, V = case["M"], case["V"]
    parent, _ = _parent(case, seed)
    logits = torch.randn((M, V), generator=_gen(seed, "logits"), device="cuda", dtype=torch.float32)
    amax = logits.argmax(1).tolist()
    r = torch.Generator().manual_seed(int(seed) + 3)
    # about half of the drafted tokens are what the model would have produced
    tokens = [int(torch.randint(V, (1,), generator=r)) for _ in range(M)]
    for i in range(1, M):
        if float(torch.rand(1, generator=r)) < 0.5:
            tokens[i] = amax[parent[i]]
    return logits, parent, tokens


def prepare(case, seed):
    """What a program holds before the call: packed weights, caches, tree, buffers, workspace."""
    op, s = case["op"], {"op": case["op"], "case": case}
    M = case["M"]
    if op in ("layer", "stack"):
        shape = _shape(case)
        s["cfg"] = B.make_cfg(shape, _capacity(case))
        s["k"], s["v"] = _caches(case, seed, case["kv"])
        s["parent"] = _int32(_parent(case, seed)[0])
        s["x16"] = _normal((M, shape.H), seed, "x")
        s["x"] = torch.empty((M, shape.H), dtype=torch.float32, device="cuda")
        s["ws"] = B.workspace(B.ghd_workspace_bytes(s["cfg"], M, case["kv"]))
        if op == "layer":
            s["w"] = model.upload_layer(_layer(case, seed, 0), shape.d)
        else:
            layers = [model.upload_layer(_layer(case, seed, l), shape.d) for l in range(shape.L)]
            s["stack"] = B.Stack(s["cfg"], layers, [(s["k"][l], s["v"][l]) for l in range(shape.L)],
                                 model.upload_head(_head(case, seed)))
            s["logits"] = torch.empty((M, shape.V), dtype=torch.float32, device="cuda")
    elif op == "linear":
        s["x"], W = _linear_inputs(case, seed)
        s["W"] = B.ghd_pack_weight(W)
        s["y"] = torch.empty((M, case["N"]), dtype=torch.float16 if case["out16"] else torch.float32, device="cuda")
        s["ws"] = B.workspace(B.lib().ghd_linear_workspace_bytes(M, case["N"], case["K"]))
    elif op == "attention":
        s["q"], s["k"], s["v"], parent, see = _attention_inputs(case, seed)
        s["parent"] = None if parent is None else _int32(parent)
        s["mask"] = _mask_words(see)
        s["ws"] = B.workspace(B.lib().ghd_attention_workspace_bytes(M, case["kv"], case["nh"], case["d"]))
    elif op == "draft":
        t = _draft_inputs(case, seed)
        s.update(g=t["g"], W=B.ghd_pack_weight(t["W"]), x=t["x"], parent=_int32(t["parent"]),
                 rank=_int32(t["rank"]), res=_int32(t["res"]))
        s["tokens"] = torch.empty(len(t["parent"]), dtype=torch.int32, device="cuda")
        s["ws"] = B.workspace(B.lib().ghd_draft_workspace_bytes(case["K"], case["R"], case["H"], case["V"]))
    else:
        shape = _shape(dict(case, F=8))
        s["logits"], parent, tokens = _accept_inputs(case, seed)
        s["parent"], s["tokens"] = _int32(parent), _int32(tokens)
        s["k"], s["v"] = _caches(case, seed, case["kv"] + M)
        # ghd_commit_path takes the caches of a Stack and no weight of it
        g = torch.ones(8, dtype=torch.float16, device="cuda")
        none = {n: g for n in ("g_attn", "Wqkv", "Wo", "g_ffn", "Wgu", "Wdown")}
        s["stack"] = B.Stack(B.make_cfg(shape, _capacity(case)), [none] * shape.L,
                             [(s["k"][l], s["v"][l]) for l in range(shape.L)], {"g_final": g, "Wlm": g})
        s["res"] = torch.zeros(2 + M, dtype=torch.int32, device="cuda")
        s["amax"] = torch.empty(M, dtype=torch.int32, device="cuda")
        s["ws"] = B.workspace(B.lib().ghd_accept_workspace_bytes(M))
    return s


def run(s):
    op, case = s["op"], s["case"]
    if op == "layer":
        s["x"].copy_(s["x16"])          # the tokens' hidden states, widened to the residual stream
        B.ghd_verify_layer(s["cfg"], s["w"], s["k"], s["v"], s["x"], s["parent"], case["kv"], ws=s["ws"])
        return {"x": s["x"], "k": s["k"], "v": s["v"]}
    if op == "stack":
        B.ghd_verify_stack(s["stack"], s["x16"], s["parent"], case["kv"], logits=s["logits"], x_out=s["x"],
                           ws=s["ws"])
        return {"logits": s["logits"], "x": s["x"], "k": s["k"], "v": s["v"]}
    if op == "linear":
        return B.ghd_linear_skinny(s["x"], s["W"], case["N"], ws=s["ws"], y=s["y"])
    if op == "attention":
        if case["mask"] == "tree":
            return B.ghd_tree_attention(s["q"], s["k"], s["v"], s["parent"], case["kv"], ws=s["ws"])
        return B.ghd_masked_attention(s["q"], s["k"], s["v"], s["mask"], case["kv"], ws=s["ws"])
    if op == "draft":
        tokens, topk, logits = B.ghd_draft_tokens(s["g"], s["W"], case["K"], case["R"], case["V"], RMS_EPS, s["x"],
                                                  s["res"], s["parent"], s["rank"], tokens=s["tokens"], ws=s["ws"])
        return {"tokens": tokens, "topk": topk, "logits": logits}
    res, amax = B.ghd_accept_greedy(s["logits"], s["tokens"], s["parent"], res=s["res"], amax=s["amax"], ws=s["ws"])
    B.ghd_commit_path(s["stack"], res, case["M"], case["kv"])
    return {"res": res, "amax": amax, "k": s["k"], "v": s["v"]}


# ---- what a pass cannot do without ----------------------------------------------------
def work(case):
    op, M = case["op"], case["M"]
    if op in ("layer", "stack"):
        nh, d, F, kv, L = case["nh"], case["d"], case["F"], case["kv"], case.get("L", 1)
        H = nh * d
        n_w = L * (4 * H * H + 3 * H * F) + (case["V"] * H if op == "stack" else 0)
        # weights, committed cache, the tree's rows written, hidden states in, residual stream out
        out = 4 * M * H + (4 * M * case["V"] if op == "stack" else 0)
        return {"bytes": 2 * n_w + 4 * L * (kv + M) * H + 2 * M * H + out,
                "flops": 2 * M * n_w + 4 * L * M * H * (kv + M)}
    if op == "linear":
        N, K = case["N"], case["K"]
        return {"bytes": 2 * N * K + 2 * M * K + (2 if case["out16"] else 4) * M * N, "flops": 2 * M * N * K}
    if op == "attention":
        H = case["nh"] * case["d"]
        return {"bytes": 4 * (case["kv"] + M) * H + 4 * M * H, "flops": 4 * M * H * (case["kv"] + M)}
    if op == "draft":
        n = case["K"] * case["V"]
        return {"bytes": 2 * n * case["H"] + 4 * n + 4 * case["H"], "flops": 2 * n * case["H"]}
    # the logits once; of the caches only the accepted rows move (about three of them here)
    return {"bytes": 4 * M * case["V"] + 3 * 8 * case["L"] * case["nh"] * case["d"], "flops": M * case["V"]}


def tolerance(case):
    op = case["op"]
    if op == "accept":
        return "exact"
    # About four times the distance from 64 bits that was measured.
    if op == "linear" and not case["out16"]:
        return {"rel": 1e-6}            # fp32 sums of fp16 products: 1.1e-7
    if op in ("linear", "draft"):
        return {"rel": 8e-4}            # rounded once to fp16 (the result, or the heads' input row): 2.1e-4
    if op == "attention":
        return {"rel": 1e-3}            # fp16 probabilities and fp16 result: 2.6e-4
    # fp16 inputs of every linear layer, through one layer (3.5e-4) or all of a stack's (2.1e-3)
    return {"rel": 1.4e-3 if op == "layer" else 8e-3}


# ---- the same in 64 bits ----------------------------------------------------------------
def _see(case, seed):
    parent, depth = _parent(case, seed)
    see = torch.zeros((case["M"], case["M"]), dtype=torch.bool)
    for i in range(case["M"]):
        j = i
        while j >= 0:
            see[i, j] = True
            j = parent[j]
    return see.cuda(), torch.tensor(depth, dtype=torch.float64, device="cuda")


def _attend(q, k, v, see, kv):
    """q [M, nh, d], k [nh, T, d], v [nh, d, T] in 64 bits, see [M, M]: -> [M, nh, d]."""
    s = torch.bmm(q.transpose(0, 1).contiguous(), k.transpose(1, 2).contiguous()) / math.sqrt(q.shape[2])
    s[:, :, kv:] = s[:, :, kv:].masked_fill(~see, -math.inf)
    p = torch.softmax(s, dim=2)
    return torch.bmm(p, v.transpose(1, 2).contiguous()).transpose(0, 1).contiguous()


def _norm(x, g):
    return x * torch.rsqrt(x.square().mean(1, keepdim=True) + RMS_EPS) * g.double()


def _exact_layer(case, seed, l, x, k, v, see, depth):
    """One decoder layer on x [M, H]; writes the tree's rows into k [nh, cap, d], v [nh, d, cap]."""
    M, nh, d, kv = case["M"], case["nh"], case["d"], case["kv"]
    H, F = nh * d, case["F"]
    w = _layer(case, seed, l)
    y = _norm(x, w["g_attn"]) @ w["Wqkv"].double().t()
    q, kn, vn = (y[:, i * H:(i + 1) * H].reshape(M, nh, d) for i in range(3))
    j = torch.arange(d // 2, dtype=torch.float64, device="cuda")
    ang = (kv + depth)[:, None] * ROPE_BASE ** (-2.0 * j / d)
    c, s = ang.cos()[:, None], ang.sin()[:, None]

    def rot(t):
        a, b = t[..., :d // 2], t[..., d // 2:]
        return torch.cat([a * c - b * s, b * c + a * s], dim=2)

    q, kn = rot(q), rot(kn)
    k[:, kv:kv + M] = kn.transpose(0, 1)
    v[:, :, kv:kv + M] = vn.permute(1, 2, 0)
    o = _attend(q, k[:, :kv + M], v[:, :, :kv + M], see, kv).reshape(M, H)
    x = x + o @ w["Wo"].double().t()
    gu = _norm(x, w["g_ffn"]) @ w["Wgu"].double().t()
    return x + (torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]) @ w["Wdown"].double().t()


def exact(case, seed):
    op, M = case["op"], case["M"]
    if op in ("layer", "stack"):
        see, depth = _see(case, seed)
        x = _normal((M, case["nh"] * case["d"]), seed, "x").double()
        k, v = (t.double() for t in _caches(case, seed, case["kv"]))
        for l in range(case.get("L", 1)):
            x = _exact_layer(case, seed, l, x, k[l], v[l], see, depth)
        if op == "layer":
            return {"x": x, "k": k, "v": v}
        h = _head(case, seed)
        return {"logits": _norm(x, h["g_final"]) @ h["Wlm"].double().t(), "x": x, "k": k, "v": v}
    if op == "linear":
        x, W = _linear_inputs(case, seed)
        return x.double() @ W.double().t()
    if op == "attention":
        q, k, v, _, see = _attention_inputs(case, seed)
        m = torch.tensor([[(s >> j) & 1 for j in range(M)] for s in see], dtype=torch.bool, device="cuda")
        T = case["kv"] + M
        return _attend(q.double(), k[:, :T].double(), v[:, :, :T].double(), m, case["kv"])
    if op == "draft":
        t = _draft_inputs(case, seed)
        n = _norm(t["x"][t["last"]:t["last"] + 1].double(), t["g"])
        W = t["W"].view(case["K"], case["V"], case["H"])
        return {"tokens": None, "topk": None,
                "logits": torch.stack([(n @ W[i].double().t())[0] for i in range(case["K"])])}
    return None
