"""Performance cases of the tree-verification library: what a speculative decoder has it do, call by call.

Four kinds of work, each through the package's public entry points and on inputs that already live on the GPU:

  draft   one tree drafted: D growth steps of W nodes (frontier rule or free attachment), then, if asked, pruning to
          the verifier's width
  verify  the tree attention of a verifier (or drafter) pass, one call per layer, each layer with its own tensors
  accept  greedy acceptance of the drafted tree and compaction of the accepted K/V rows of all layers
  step    a whole decode step: the three above in a row, either call by call or replayed from a HIP graph

A case is a dict of plain values; listed() names the fixed ones, draw() gives more of the same ranges.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2512_23858_amd as ygg
import ygg_workloads as wl

DEV = "cuda:0"
_CODE = {"f32": ygg.F32, "bf16": ygg.BF16, "fp8": ygg.FP8_E4M3}
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.uint8}
_KV_BYTES = {"f32": 4, "bf16": 2, "fp8": 1}


def _draft(name, batch, depth, width, vocab, attach=False, keep=0):
    """keep: nodes kept for verification by pruning after the last growth step (0: none)."""
    return dict(name=name, kind="draft", batch=batch, depth=depth, width=width, vocab=vocab, attach=attach, keep=keep)


def _verify(name, batch, heads, head_dim, depth, width, prefix, layers, dtype="bf16", shortest=0, lse=False):
    """heads: (query heads, K/V heads); prefix: longest sequence of the batch; shortest: the shortest (0: all alike)."""
    return dict(name=name, kind="verify", batch=batch, q_heads=heads[0], kv_heads=heads[1], head_dim=head_dim,
                depth=depth, width=width, prefix=prefix, shortest=shortest or prefix, layers=layers, dtype=dtype, lse=lse)


def _accept(name, batch, kv_heads, head_dim, depth, width, vocab, prefix, layers, agree, dtype="bf16", logits=True):
    """logits: the call finds the verifier's tokens itself; otherwise the program hands it the argmax."""
    return dict(name=name, kind="accept", batch=batch, q_heads=kv_heads, kv_heads=kv_heads, head_dim=head_dim,
                depth=depth, width=width, vocab=vocab, prefix=prefix, shortest=max(prefix // 2, 1), layers=layers,
                agree=agree, dtype=dtype, logits=logits)


def _step(name, batch, heads, head_dim, depth, width, vocab, prefix, layers, agree, dtype="bf16", graph=False):
    return dict(name=name, kind="step", batch=batch, q_heads=heads[0], kv_heads=heads[1], head_dim=head_dim,
                depth=depth, width=width, vocab=vocab, prefix=prefix, shortest=prefix, layers=layers, agree=agree,
                dtype=dtype, graph=graph, lse=False, attach=False, keep=0, logits=True)


def listed():
    return [
        # the smallest call sequence there is: a toy fp32 model, one layer; launches and host time are all of it
        _step("step tiny fp32", 1, (4, 4), 64, 3, 4, 1000, 128, 1, 0.7, dtype="f32"),
        # drafting beside a 7B verifier: six growth steps of one interactive request
        _draft("draft 7B", 1, 6, 8, 32000),
        # the same for a serving batch of sixteen requests
        _draft("draft 7B batch 16", 16, 6, 8, 32000),
        # free attachment over a 128k vocabulary, then pruning to three quarters of the tree
        _draft("draft attach and prune 8B", 1, 8, 16, 128256, attach=True, keep=96),
        # the attention of one verifier pass over all 32 layers, one request, short prompt: many small launches
        _verify("verify 7B", 1, (32, 32), 128, 6, 8, 1024, 32),
        # three ragged requests with sizes that fit no tile, grouped heads; log-sum-exps wanted too
        _verify("verify 8B ragged batch 3", 3, (32, 8), 128, 5, 7, 1531, 8, shortest=301, lse=True),
        # long context, widest tree: the matrix cores
        _verify("verify long context", 1, (32, 8), 128, 10, 32, 32768, 4),
        # a 70B-shaped serving batch of sixteen requests, 512 to 8192 tokens each
        _verify("verify 70B batch 16", 16, (64, 8), 128, 6, 8, 8192, 4, shortest=512),
        # K/V kept in 8 bits, eight requests of 4096 tokens, one query head per K/V head: the K/V stream
        _verify("verify 8-bit K/V batch 8", 8, (32, 32), 128, 6, 8, 4096, 2, dtype="fp8"),
        # the drafter's own attention over its tree (12 layers, 12 heads of 64)
        _verify("verify drafter", 1, (12, 12), 64, 8, 8, 2048, 12),
        # acceptance after an 8B verifier: argmax over 129 rows of a 128k vocabulary, K/V rows of 32 layers
        _accept("accept 8B", 1, 8, 128, 8, 16, 128256, 4096, 32, 0.6),
        # a whole decode step of the 8B model, captured once and replayed
        _step("step 8B graph", 1, (32, 8), 128, 8, 16, 128256, 4096, 32, 0.6, graph=True),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


_HEADS = [((32, 32), 128), ((40, 40), 128), ((32, 8), 128), ((64, 8), 128), ((12, 12), 64), ((32, 8), 64)]


def draw(rng):
    kind = rng.choice(["draft", "verify", "verify", "accept", "step"])
    batch = 1 if rng.random() < 0.4 else _log_int(rng, 2, 16)
    depth = rng.randint(2, 10)
    width = _log_int(rng, 2, 32)
    vocab = _log_int(rng, 1000, 128256)
    prefix = _log_int(rng, 64, 32768)
    heads, head_dim = rng.choice(_HEADS)
    agree = round(rng.uniform(0.4, 0.8), 3)
    dtype = rng.choice(["bf16", "bf16", "bf16", "fp8" if head_dim == 128 else "bf16", "f32"])
    if dtype == "f32":     # toy models and comparisons only
        heads, head_dim, batch, prefix, width = (4, 4), 64, min(batch, 2), min(prefix, 1024), min(width, 8)
    n_nodes = 1 + depth * width
    if kind == "draft":
        if batch * width * depth * vocab > 64 << 20:
            batch = max(1, (64 << 20) // (width * depth * vocab))
        attach = rng.random() < 0.4
        keep = rng.choice([0, max(1, (3 * n_nodes) // 4)])
        case = _draft("", batch, depth, width, vocab, attach, keep)
    elif kind == "verify":
        case = _verify("", batch, heads, head_dim, depth, width, prefix, rng.choice([2, 4, 8]), dtype,
                       shortest=rng.choice([0, max(1, prefix // 16)]), lse=rng.random() < 0.25)
    elif kind == "accept":
        if batch * n_nodes * vocab > 64 << 20:
            batch = max(1, (64 << 20) // (n_nodes * vocab))
        case = _accept("", batch, heads[1], head_dim, depth, width, vocab, min(prefix, 4096), rng.choice([1, 8, 32]), agree,
                       dtype, logits=rng.random() < 0.7)
    else:
        vocab = min(vocab, max(1000, (48 << 20) // (batch * n_nodes)))
        case = _step("", batch, heads, head_dim, depth, width, vocab, prefix, rng.choice([1, 4, 8]), agree, dtype,
                     graph=rng.random() < 0.5)
    while "prefix" in case and (_cost(case) > 4.5e-4 or _kv_bytes(case) > 3e9):   # stay below the largest listed cases
        if case["layers"] > 2:
            case["layers"] //= 2
        elif case["batch"] > 1:
            case["batch"] //= 2
        else:
            case["prefix"] = max(1, case["prefix"] // 2)
            case["shortest"] = min(case["shortest"], case["prefix"])
    del case["name"]
    return case


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 6e12, w["flops"] / 1.2e15)


def _kv_bytes(case):
    return 2.0 * case["layers"] * case["batch"] * case["prefix"] * case["kv_heads"] * case["head_dim"] * _KV_BYTES[case["dtype"]]


def _lens(case):
    """The batch's sequence lengths, evenly spread from the shortest to the longest (their order comes from the seed)."""
    return np.rint(np.linspace(case["prefix"], case["shortest"], case["batch"])).astype(np.int64)


def work(case):
    B, D, W = case["batch"], case["depth"], case["width"]
    N = 1 + D * W
    kind = case["kind"]
    nbytes = flops = 0.0
    if kind in ("draft", "step"):
        rows = B * (1 + (D - 1) * W)
        nbytes += 4.0 * rows * case["vocab"] + 12.0 * B * N + 12.0 * B * case["keep"]
        flops += 2.0 * rows * case["vocab"]
    if kind in ("verify", "step"):
        total = float(_lens(case).sum())
        kv, qo = _KV_BYTES[case["dtype"]], 4 if case["dtype"] == "f32" else 2
        row = case["head_dim"] * case["kv_heads"]
        nbytes += case["layers"] * (2.0 * (total + B * N) * row * kv + 2.0 * B * N * case["q_heads"] * case["head_dim"] * qo)
        keys = N * total + B * (1 + W * D * (D + 3) / 2)      # the prefix, then a node's ancestors and itself
        flops += case["layers"] * 4.0 * case["q_heads"] * case["head_dim"] * keys
    if kind in ("accept", "step"):
        if case["logits"]:
            nbytes += 4.0 * B * N * case["vocab"]
            flops += 1.0 * B * N * case["vocab"]
        accepted = 1 + min(D, case["agree"] / (1 - case["agree"]))
        nbytes += case["layers"] * 4.0 * B * accepted * case["kv_heads"] * case["head_dim"] * _KV_BYTES[case["dtype"]]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "accept":
        return "exact"                                        # tokens, lengths, paths and copied rows
    if case["kind"] == "draft" or case["dtype"] == "f32":
        return {"rel": 1e-5 if case["kind"] != "draft" else 1e-6, "max": 1e-4}     # fp32 sums; scores are fp64 rounded to fp32
    return {"rel": 1e-2, "max": 0.1}                          # bf16 softmax weights and outputs


# ---------------------------------------------------------------- what a program has in hand

def _shape(case, capacity):
    kv = "kv_heads" in case
    return ygg.Shape(batch=case["batch"], n_q_heads=case["q_heads"] if kv else 1, n_kv_heads=case["kv_heads"] if kv else 1,
                     head_dim=case["head_dim"] if kv else 64, depth=case["depth"], width=case["width"],
                     n_nodes=1 + case["depth"] * case["width"], vocab=case.get("vocab", 1),
                     kv_dtype=_CODE[case["dtype"]] if kv else ygg.BF16,
                     softmax_scale=1.0 / math.sqrt(case["head_dim"]) if kv else 1.0, kv_capacity=capacity,
                     max_seq_len=capacity - case["depth"] - 1)


def _ints(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)


def _normal(gen, shape, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(generator=gen)


def _codes(gen, layers, shape_cache, shape_tree):
    """K or V in 8 bits: N(0, 1) values, each layer's K/V head scaled so that its largest magnitude is 448."""
    heads = shape_cache[2]
    cache = torch.empty((layers, *shape_cache), dtype=torch.uint8, device=DEV)
    tree = torch.empty((layers, *shape_tree), dtype=torch.uint8, device=DEV)
    scale = torch.empty((layers, heads), dtype=torch.float32, device=DEV)
    for l in range(layers):
        c, t = _normal(gen, shape_cache, torch.float32), _normal(gen, shape_tree, torch.float32)
        s = torch.maximum(c.abs().amax(dim=(0, 1, 3)), t.abs().amax(dim=(0, 1, 3))) / 448.0
        scale[l] = s
        cache[l] = (c / s[:, None]).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
        tree[l] = (t / s[:, None]).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    return cache, tree, scale


def _kv(case, s, gen, capacity):
    B, N, Hkv, Dh, layers = case["batch"], 1 + case["depth"] * case["width"], case["kv_heads"], case["head_dim"], case["layers"]
    cache, tree = (B, capacity, Hkv, Dh), (B, N, Hkv, Dh)
    for x in "kv":
        if case["dtype"] == "fp8":
            s[x + "_cache"], s[x + "_tree"], s[x + "_scale"] = _codes(gen, layers, cache, tree)
        else:
            s[x + "_cache"] = _normal(gen, (layers, *cache), _TORCH[case["dtype"]])
            s[x + "_tree"] = _normal(gen, (layers, *tree), _TORCH[case["dtype"]])


def _best_tree(case, draft):
    """The tree that growth by the frontier rule makes of these logits, level by level (parents and tokens)."""
    B, D, W, V = case["batch"], case["depth"], case["width"], case["vocab"]
    parent = torch.full((B, 1 + D * W), -1, dtype=torch.int64, device=DEV)
    token = torch.zeros_like(parent)
    cum = torch.zeros((B, 1), dtype=torch.float64, device=DEV)
    for d in range(1, D + 1):
        score = (cum[:, :, None] + torch.log_softmax(draft[d - 1].double(), dim=-1)).view(B, -1)
        cum, flat = score.topk(W, dim=1)
        new = slice(1 + (d - 1) * W, 1 + d * W)
        parent[:, new] = flat // V + (0 if d == 1 else 1 + (d - 2) * W)
        token[:, new] = flat % V
    return parent.cpu().numpy(), token.cpu().numpy()


def _target(case, gen, host, parent, token):
    """The verifier's choice per node: one of the drafted children with probability `agree`, else something else."""
    B, V = case["batch"], case["vocab"]
    N = 1 + case["depth"] * case["width"]
    chosen = {}
    for b in range(B):
        for i in host.permutation(np.arange(1, N)):
            chosen[b, int(parent[b, i])] = int(token[b, i])
    hit = [(b, p, t) for (b, p), t in chosen.items() if host.random() < case["agree"]]
    at = torch.tensor(hit, dtype=torch.int64, device=DEV).reshape(-1, 3).T
    if not case["logits"]:
        best = torch.randint(0, V, (B, N), dtype=torch.int32, device=DEV, generator=gen)
        best[at[0], at[1]] = at[2].to(torch.int32)
        return best
    logits = _normal(gen, (B, N, V), torch.float32)
    logits[at[0], at[1], at[2]] = 8.0
    return logits


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    host = np.random.default_rng(seed)
    B, D, W = case["batch"], case["depth"], case["width"]
    N = 1 + D * W
    kind = case["kind"]
    capacity = (case["prefix"] + D + 1 + 255) // 256 * 256 + 256 if "prefix" in case else D + 2   # room to go on decoding
    shape = _shape(case, capacity)
    s = dict(case=case, shape=shape, graph=None)
    ygg.init()

    if kind in ("draft", "step"):
        s["draft"] = [_normal(gen, (B, 1 if d == 1 else W, case["vocab"]), torch.float32).mul_(3.0) for d in range(1, D + 1)]
        s["parent"] = torch.full((B, N), -1, dtype=torch.int32, device=DEV)
        s["token"] = torch.zeros((B, N), dtype=torch.int32, device=DEV)
        s["token"][:, 0] = torch.randint(0, case["vocab"], (B,), dtype=torch.int32, device=DEV, generator=gen)
        s["cum"] = torch.zeros((B, N), dtype=torch.float32, device=DEV)
        if case["attach"]:
            s["pool"] = torch.empty(ygg.attach_pool_bytes(shape), dtype=torch.uint8, device=DEV)
        s["ws_draft"] = ygg.new_workspace(shape, ygg.OP_ATTACH if case["attach"] else ygg.OP_EXPAND)
        if case["keep"]:
            for x in ("kept", "kept_parent", "kept_token"):
                s[x] = torch.zeros((B, case["keep"]), dtype=torch.int32, device=DEV)
            s["expected"] = torch.zeros((B,), dtype=torch.float32, device=DEV)
            s["best_width"] = torch.zeros((B,), dtype=torch.int32, device=DEV)
            s["t_verifier"] = torch.linspace(1.0, 2.0, N + 1, dtype=torch.float32, device=DEV)

    if kind != "draft":
        s["lens0"] = _ints(host.permutation(_lens(case)))
        s["lens"] = s["lens0"].clone()
        _kv(case, s, gen, capacity)
        if kind != "step":
            s["parent"] = _ints(np.stack([wl.level_tree(seed, D, W, "dirichlet", 0.5, sub=b) for b in range(B)]))

    if kind in ("verify", "step"):
        dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        rows = (case["layers"], B, N, case["q_heads"])
        s["q"] = _normal(gen, (*rows, case["head_dim"]), dt)
        s["out"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty(rows, dtype=torch.float32, device=DEV) if case["lse"] else None
        s["ws_attention"] = ygg.new_workspace(shape, ygg.OP_ATTENTION)
        names = ["q", "k_cache", "v_cache", "k_tree", "v_tree", "out"] + ["k_scale", "v_scale"] * (case["dtype"] == "fp8")
        s["layers"] = [{x: s[x][l] for x in names} | {"lse": s["lse"][l] if case["lse"] else None} for l in range(case["layers"])]

    if kind in ("accept", "step"):
        if kind == "step":
            parent, token = _best_tree(case, s["draft"])
        else:
            parent = s["parent"].cpu().numpy()
            token = np.stack([host.choice(case["vocab"], size=N, replace=False) for _ in range(B)])
            s["token"] = _ints(token)
        s["target"] = _target(case, gen, host, parent, token)
        s["accept_len"] = torch.zeros((B,), dtype=torch.int32, device=DEV)
        s["accept_path"] = torch.zeros((B, D + 1), dtype=torch.int32, device=DEV)
        s["bonus"] = torch.zeros((B,), dtype=torch.int32, device=DEV)
        s["ws_accept"] = ygg.new_workspace(shape, ygg.OP_ACCEPT, case["layers"])

    if case.get("graph"):
        _enqueue(s)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _enqueue(s)
        s["graph"] = graph
    return s


# ---------------------------------------------------------------- one pass

def _enqueue(s):
    case, shape = s["case"], s["shape"]
    kind = case["kind"]
    if kind in ("accept", "step"):
        s["lens"].copy_(s["lens0"])          # every pass starts from the same confirmed prefix
    if kind in ("draft", "step"):
        for d in range(1, case["depth"] + 1):
            if case["attach"]:
                ygg.equal_growth_attach(shape, d, s["draft"][d - 1], s["parent"], s["token"], s["cum"], s["pool"], s["ws_draft"])
            else:
                ygg.equal_growth_expand(shape, d, s["draft"][d - 1], s["parent"], s["token"], s["cum"], s["ws_draft"])
        if case["keep"]:
            ygg.prune_for_verification(shape, case["keep"], s["parent"], s["token"], s["cum"], s["kept"], s["kept_parent"],
                                       s["kept_token"], s["expected"], s["best_width"], t_verifier=s["t_verifier"], t_draft=1.0)
    if kind in ("verify", "step"):
        for x in s["layers"]:
            if case["dtype"] == "fp8":
                ygg.tree_attention_fp8kv(shape, x["q"], x["k_cache"], x["v_cache"], s["lens"], x["k_tree"], x["v_tree"],
                                         x["k_scale"], x["v_scale"], s["parent"], x["out"], x["lse"], s["ws_attention"])
            else:
                ygg.tree_attention(shape, x["q"], x["k_cache"], x["v_cache"], s["lens"], x["k_tree"], x["v_tree"],
                                   s["parent"], x["out"], x["lse"], s["ws_attention"])
    if kind in ("accept", "step"):
        ygg.accept_and_compact(shape, case["layers"], s["parent"], s["token"], s["k_tree"], s["v_tree"], s["k_cache"],
                               s["v_cache"], s["lens"], s["accept_len"], s["accept_path"], s["bonus"],
                               **{"target_logits" if case["logits"] else "target_tokens": s["target"]}, workspace=s["ws_accept"])


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _enqueue(state)
    kind = state["case"]["kind"]
    names = []
    if kind in ("draft", "step"):
        names += ["parent", "token", "cum"] + ["kept", "kept_parent", "kept_token", "expected", "best_width"] * bool(state["case"]["keep"])
    if kind in ("verify", "step"):
        names += ["out"] + ["lse"] * state["case"]["lse"]
    if kind in ("accept", "step"):
        names += ["accept_len", "accept_path", "bonus", "lens", "k_cache", "v_cache"]
    return {x: state[x] for x in names}
