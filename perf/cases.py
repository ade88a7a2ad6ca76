"""What this framework is timed on: the calls that a draft-then-verify serving program makes, from the smallest
step to the largest.

Five kinds of pass, all through the public entry points of the package:

  verify   one verification step of a target model: tree attention of every layer against that layer's own
           cache, acceptance over the logits, commit of the accepted path in every layer
  accept   the acceptance for drafts that were sampled from a draft distribution
  lm_head  acceptance straight from the last hidden states (the LM head inside the call)
  draft    the draft side of a step: Feature Sampler, draft decoder layer, top-k cut of the draft's logits
  cycle    one whole draft-then-verify cycle of a small batch, call after call as the README writes it

Geometries are those of the repository's own workloads (Vicuna 7B / 33B, LLaMA3 8B / 70B layers and heads);
`draw` spreads over the ranges around them, odd sizes among them. Inputs are random with the distributions the
repository's tests use: Q, K, V ~ N(0,1), logits ~ N(0, 3^2) with one entry of every row lifted by up to six
above the rest (a model is sure of some tokens and not of others, so paths of several nodes are accepted), drafts
from a perturbed target, trees cut from candidates whose conditional probabilities fall off geometrically.

A pass over a stack of layers repeats prepared calls over fixed buffers (how a serving loop calls this library,
and what bench.py times); the ragged batch and the cycle make plain calls, as a program does whose sizes
change from step to step.
"""
import math
import random

import numpy as np
import torch

import paper_2408_15562_amd as fspad

BF16, F32 = torch.bfloat16, torch.float32


# --------------------------------------------------------------------------------------------------- the cases

def _verify(name, **kw):
    case = {"name": name, "kind": "verify", "dtype": "bf16", "layers": 1, "batch": 1, "n_q_heads": 32, "n_kv_heads": 32,
            "head_dim": 128, "kv_min": 0, "kv_max": 0, "nodes_min": 0, "nodes_max": 26, "depth": 6, "topk": 4,
            "vocab": 32000, "accept": "greedy", "temperature": 1.0, "calls": "prepared", "shape_seed": 1}
    case.update(kw)
    case["kv_min"] = case["kv_min"] or case["kv_max"]
    case["nodes_min"] = case["nodes_min"] or case["nodes_max"]
    return case


def listed():
    return [
        # the smallest step there is: one fp32 layer, a thousand-word vocabulary (launches and latency)
        _verify("tiny fp32 step", dtype="f32", n_q_heads=8, n_kv_heads=8, head_dim=64, kv_max=256, depth=5, vocab=1000),
        # interactive decoding of a 7B model: one sequence, every layer of the stack, short tree
        _verify("7B stack greedy", layers=32, kv_max=2048),
        # the same with grouped heads, the default 60-node tree and sampling over a large vocabulary
        _verify("8B GQA stack sampling", layers=32, n_kv_heads=8, kv_max=4096, nodes_max=60, topk=10, vocab=128256,
                accept="sample"),
        # four sequences of a 33B model (20 of its 60 layers; each is the same work): the largest cache traffic
        _verify("33B layers 4 sequences", layers=20, batch=4, n_q_heads=52, n_kv_heads=52, kv_max=4096, nodes_max=60,
                topk=10),
        # long retrieval-augmented prompt of a 70B model (20 of its 80 layers)
        _verify("70B layers long prompt", layers=20, n_q_heads=64, n_kv_heads=8, kv_max=16384, nodes_max=60, topk=10,
                vocab=128256, accept="sample"),
        # a serving batch as it comes: 16 sequences of different lengths and tree sizes, temperature below 1
        _verify("ragged batch of 16", layers=4, batch=16, n_kv_heads=8, kv_min=131, kv_max=6011, nodes_min=17,
                nodes_max=60, topk=10, vocab=128256, accept="sample", temperature=0.7, calls="plain", shape_seed=7),
        # acceptance when the drafts were sampled (both distributions are read)
        {"name": "sampled drafts", "kind": "accept", "batch": 1, "nodes_min": 60, "nodes_max": 60, "depth": 6, "topk": 10,
         "vocab": 128256, "temperature": 1.0, "shape_seed": 1},
        # acceptance from hidden states: a 33B head for four sequences, weights as a model stores them ...
        {"name": "33B head greedy", "kind": "lm_head", "batch": 4, "nodes_min": 60, "nodes_max": 60, "depth": 6,
         "topk": 10, "hidden": 6656, "vocab": 32000, "accept": "greedy", "temperature": 1.0, "packed": False, "shape_seed": 1},
        # ... and an 8B head with a large vocabulary, sampling, weights repacked once ahead of time
        {"name": "8B head sampling", "kind": "lm_head", "batch": 1, "nodes_min": 60, "nodes_max": 60, "depth": 6,
         "topk": 10, "hidden": 4096, "vocab": 128256, "accept": "sample", "temperature": 1.0, "packed": True, "shape_seed": 1},
        # draft step of one sequence: the rows of one level of the tree through sampler, layer and top-k cut
        {"name": "draft step 4 rows", "kind": "draft", "batch": 1, "rows": 4, "hidden": 4096, "inter": 11008,
         "n_q_heads": 32, "n_kv_heads": 32, "head_dim": 128, "kv_max": 2048, "vocab": 32000, "topk": 4, "packed": True},
        # draft step of four sequences of a 33B model, weights as a model stores them
        {"name": "draft step 40 rows", "kind": "draft", "batch": 4, "rows": 10, "hidden": 6656, "inter": 17920,
         "n_q_heads": 52, "n_kv_heads": 52, "head_dim": 128, "kv_max": 4096, "vocab": 32000, "topk": 10, "packed": False},
        # one cycle end to end, written as the README writes it (one 7B layer stands for the stack)
        {"name": "one cycle plain calls", "kind": "cycle", "batch": 1, "rows": 4, "hidden": 4096, "inter": 11008,
         "n_q_heads": 32, "n_kv_heads": 32, "head_dim": 128, "kv_max": 2048, "nodes_min": 26, "nodes_max": 26, "depth": 6,
         "topk": 4, "vocab": 32000, "shape_seed": 1},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _vocab(rng):
    return rng.choice([32000, 50257, 128256, _log_int(rng, 1000, 152000)])


def _heads(rng, limit):
    q, kv = rng.choice([h for h in ((8, 8), (16, 16), (32, 32), (40, 40), (52, 52), (12, 2), (28, 4), (32, 8), (40, 8),
                                    (64, 8)) if h[0] <= limit])
    return q, kv


def draw(rng):
    """One more case of the ranges the listed ones stand for, never dearer than the largest of them."""
    kind = rng.choice(["verify", "verify", "verify", "verify", "accept", "lm_head", "lm_head", "draft", "draft", "cycle"])
    seed = rng.randrange(1 << 20)
    topk, depth = rng.choice([4, 5, 8, 10]), rng.randint(3, 6)
    n_max = min(rng.choice([64, 60, 60, 48, 26, rng.randint(1, 64)]), 1 + topk + (depth - 1) * topk * topk)
    n_min = rng.choice([n_max, n_max, rng.randint(1, n_max)])
    batch = _log_int(rng, 1, 16)
    if kind == "verify":
        f32 = rng.random() < 0.15
        hq, hkv = _heads(rng, 16 if f32 else 64)
        D = rng.choice([64, 128, 128])
        kv = _log_int(rng, 24, 700 if f32 else 16384)
        layers = 1 if f32 else _log_int(rng, 1, 32)
        accept, vocab = rng.choice(["greedy", "sample"]), _vocab(rng)
        if f32:
            batch = min(batch, 2)
        # keep the cache and the arithmetic of a pass below the largest listed case's
        while batch * layers * hkv * D * (kv + n_max) > 5e8 or batch * layers * hq * D * (kv + n_max) * n_max > 6e10:
            if layers > 1:
                layers = max(1, layers // 2)
            elif batch > 1:
                batch = max(1, batch // 2)
            else:
                kv //= 2
        return _verify("drawn", dtype="f32" if f32 else "bf16", layers=layers, batch=batch, n_q_heads=hq, n_kv_heads=hkv,
                       head_dim=D, kv_min=rng.choice([kv, max(1, kv // 8)]), kv_max=kv, nodes_min=n_min, nodes_max=n_max,
                       depth=depth, topk=topk, vocab=vocab, accept=accept,
                       temperature=rng.choice([1.0, 1.0, 0.7]), calls=rng.choice(["prepared", "plain"]), shape_seed=seed)
    if kind == "accept":
        return {"name": "drawn", "kind": kind, "batch": min(batch, 8), "nodes_min": n_min, "nodes_max": n_max, "depth": depth,
                "topk": topk, "vocab": _vocab(rng), "temperature": rng.choice([1.0, 0.7]), "shape_seed": seed}
    if kind == "lm_head":
        return {"name": "drawn", "kind": kind, "batch": min(batch, 5), "nodes_min": n_min, "nodes_max": n_max, "depth": depth,
                "topk": topk, "hidden": 256 * rng.choice([4, 8, 16, 16, 20, 26]), "vocab": _log_int(rng, 4000, 128256),
                "accept": rng.choice(["greedy", "sample"]), "temperature": rng.choice([1.0, 0.7]),
                "packed": rng.random() < 0.5, "shape_seed": seed}
    hidden = 256 * rng.choice([4, 8, 16, 16, 20, 26])
    D = 128 if hidden >= 2048 else 64
    hq = hidden // D
    side = {"batch": min(batch, 8), "rows": topk, "hidden": hidden, "inter": 256 * max(4, int(hidden * rng.uniform(2.3, 3.6) / 256)),
            "n_q_heads": hq, "n_kv_heads": rng.choice([h for h in (hq, 4, 8) if hq % h == 0]), "head_dim": D,
            "kv_max": _log_int(rng, 24, 8192), "vocab": _vocab(rng), "topk": topk}
    if kind == "draft":
        return {"name": "drawn", "kind": kind, "packed": rng.random() < 0.5, **side}
    side["vocab"], side["batch"] = min(side["vocab"], 64000), min(batch, 3)
    return {"name": "drawn", "kind": "cycle", "nodes_min": n_min, "nodes_max": n_max, "depth": depth, "shape_seed": seed, **side}


# ------------------------------------------------------------------------------------------------------ inputs

def _spread(case, lo, hi, salt):
    """One size per sequence between lo and hi (the first one hi), from the case alone."""
    r = random.Random(case["shape_seed"] * 7 + salt)
    return np.array([hi if b == 0 else r.randint(lo, hi) for b in range(case["batch"])], dtype=np.int32)


def _lens(case):
    return _spread(case, case["kv_min"], case["kv_max"], 1) if "kv_min" in case else np.full(case["batch"], case["kv_max"], np.int32)


def _nodes(case):
    return _spread(case, case["nodes_min"], case["nodes_max"], 2)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, dtype=BF16, scale=1.0):
    x = torch.empty(shape, dtype=dtype, device="cuda").normal_(generator=g)
    return x.mul_(scale) if scale != 1.0 else x


def _logits(g, B, N, V):
    x = _normal(g, (B, N, V), F32, 3.0)
    top = x.amax(dim=-1, keepdim=True) + 6.0 * torch.rand((B, N, 1), generator=g, device="cuda")
    return x.scatter_(2, torch.randint(V, (B, N, 1), generator=g, device="cuda"), top)


def _candidates(rng, depth, topk, vocab):
    """Candidates of `depth` draft steps: the top-k continuations of the k best nodes of each level."""
    par, tok, logp, joint, frontier = [-1], [int(rng.integers(vocab))], [0.0], [0.0], [0]
    for _ in range(depth):
        new = []
        for p in frontier:
            c = rng.uniform(0.2, 0.7) ** np.arange(topk)
            toks = rng.choice(vocab, size=topk, replace=False)
            for t, lp in zip(toks, np.log(c / c.sum())):
                par.append(p)
                tok.append(int(t))
                logp.append(float(lp))
                joint.append(joint[p] + float(lp))
                new.append(len(par) - 1)
        frontier = sorted(sorted(new, key=lambda i: -joint[i])[:topk])
    return par, tok, logp


def _tree_inputs(case, seed):
    """Candidates of every sequence on the GPU, as fspad_tree_build takes them."""
    rng = np.random.default_rng([seed, 11])
    per = [_candidates(rng, case["depth"], case["topk"], case["vocab"]) for _ in range(case["batch"])]
    par, tok, logp = (np.array([p[k] for p in per]) for k in range(3))
    cuda = lambda a, dt: torch.from_numpy(a.astype(dt)).cuda()  # noqa: E731
    return cuda(par, np.int32), cuda(tok, np.int32), cuda(logp, np.float32), torch.full((case["batch"],), par.shape[1], dtype=torch.int32, device="cuda")


def _trees(case, seed):
    """Trees of the case's node counts: parent [B,N] and mask on the device, node counts on both sides, sibling ranks."""
    n = _nodes(case)
    N = case["nodes_max"]
    cand = _tree_inputs(case, seed)
    parts = [fspad.fspad_tree_build(*(c[b:b + 1].contiguous() for c in cand), int(n[b]), N) for b in range(case["batch"])]
    parent, _, n_dev, mask, _ = (torch.cat(x) for x in zip(*parts))
    par = parent.cpu().numpy()
    rank = np.zeros_like(par)
    for b in range(par.shape[0]):
        seen = {}
        for i in range(1, int(n[b])):
            p = int(par[b, i])
            rank[b, i] = seen.get(p, 0)
            seen[p] = rank[b, i] + 1
    return {"parent": parent, "mask": mask, "n_dev": n_dev, "n": n, "rank": torch.from_numpy(rank).cuda().long()}


def _draft_tokens(g, logits, tree, sampled):
    """Every node's children carry the best (sampled: drawn without replacement) tokens of a perturbed copy of its row."""
    key = torch.empty_like(logits).normal_(generator=g).add_(logits)
    if sampled:
        key.sub_(torch.empty_like(logits).exponential_(generator=g).log_())   # + Gumbel noise
    top = key.topk(min(16, logits.shape[-1]), dim=-1).indices
    par = tree["parent"].long().clamp(min=0)
    tok = top.gather(1, par[:, :, None].expand(-1, -1, top.shape[2])).gather(2, tree["rank"][:, :, None].clamp(max=top.shape[2] - 1))
    return tok[:, :, 0].int().contiguous()


def _accept_outputs(B, N):
    z = lambda *s: torch.zeros(s, dtype=torch.int32, device="cuda")  # noqa: E731
    return z(B, N), z(B), z(B, N), z(B)


def _bytes(n):
    return torch.empty(max(16, n), dtype=torch.uint8, device="cuda")


def _prepare_verify(case, seed):
    g = _gen(seed)
    B, N, Hq, Hkv, D, V, layers = (case[k] for k in ("batch", "nodes_max", "n_q_heads", "n_kv_heads", "head_dim", "vocab", "layers"))
    dt = F32 if case["dtype"] == "f32" else BF16
    kv_len = _lens(case)
    cap = (int(kv_len.max()) + N + 63) // 64 * 64
    tree = _trees(case, seed)
    s = {"case": case, "kv_len": kv_len, "tree": tree}
    s["q"] = _normal(g, (layers, B, N, Hq, D), dt)
    s["k_tree"], s["v_tree"] = _normal(g, (layers, B, N, Hkv, D), dt), _normal(g, (layers, B, N, Hkv, D), dt)
    s["k_cache"], s["v_cache"] = _normal(g, (layers, B, Hkv, cap, D), dt), _normal(g, (layers, B, Hkv, cap, D), dt)
    s["out"] = torch.zeros((layers, B, N, Hq, D), dtype=dt, device="cuda")
    s["logits"] = _logits(g, B, N, V)
    s["tokens"] = _draft_tokens(g, s["logits"], tree, case["accept"] == "sample")
    s["uniforms"] = torch.rand((B, 2, N), generator=g, device="cuda")
    s["accepted"] = _accept_outputs(B, N)
    s["kv_len_out"] = torch.zeros(B, dtype=torch.int32, device="cuda")
    desc = fspad.make_attn_desc(s["q"][0], s["k_tree"][0], s["k_cache"][0])
    s["workspace"] = _bytes(fspad.fspad_tree_attn_workspace_bytes(desc, int(kv_len.max())))
    s["accept_workspace"] = _bytes(fspad.fspad_tree_accept_workspace_bytes(B, N, V))
    if case["calls"] == "prepared":
        s["attn_calls"] = [_attn(s, layer, True) for layer in range(layers)]
        s["accept_call"] = _accept(s, True)
        s["commit_calls"] = [_commit(s, layer, True) for layer in range(layers)]
    # the rows a commit may write: what it appended, and that it left the rest alone
    s["appended"] = [c[:, b, :, int(kv_len[b]):int(kv_len[b]) + N] for c in (s["k_cache"], s["v_cache"]) for b in range(B)]
    return s


def _attn(s, layer, prepare):
    t = s["tree"]
    return fspad.fspad_tree_attn(s["q"][layer], s["k_tree"][layer], s["v_tree"][layer], s["k_cache"][layer], s["v_cache"][layer],
                                 s["kv_len"], t["n"], t["mask"], out=s["out"][layer], workspace=s["workspace"], prepare=prepare)


def _accept(s, prepare):
    t, case = s["tree"], s["case"]
    kw = {"outputs": s["accepted"], "workspace": s["accept_workspace"], "prepare": prepare}
    if case["accept"] == "greedy":
        return fspad.fspad_tree_accept_greedy(s["logits"], s["tokens"], t["parent"], t["n_dev"], **kw)
    return fspad.fspad_tree_accept_sample(s["logits"], s["tokens"], t["parent"], t["n_dev"], case["temperature"], s["uniforms"], **kw)


def _commit(s, layer, prepare):
    return fspad.fspad_kv_commit(s["k_tree"][layer], s["v_tree"][layer], s["k_cache"][layer], s["v_cache"][layer], s["kv_len"],
                                 s["accepted"][0], s["accepted"][1], kv_len_out=s["kv_len_out"], prepare=prepare)


def _run_verify(s):
    layers = s["case"]["layers"]
    if s["case"]["calls"] == "prepared":
        for call in s["attn_calls"]:
            call()
        s["accept_call"]()
        for call in s["commit_calls"]:
            call()
    else:
        for layer in range(layers):
            _attn(s, layer, False)
        _accept(s, False)
        for layer in range(layers):
            _commit(s, layer, False)
    return [s["out"], s["accepted"], s["kv_len_out"], s["appended"]]


def _prepare_accept(case, seed):
    g = _gen(seed)
    B, N, V = case["batch"], case["nodes_max"], case["vocab"]
    s = {"case": case, "tree": _trees(case, seed)}
    s["logits"] = _logits(g, B, N, V)
    s["draft_logits"] = _normal(g, (B, N, V), F32).add_(s["logits"])
    gumbel = torch.empty_like(s["logits"]).exponential_(generator=g).log_().neg_()
    key = s["draft_logits"] / case["temperature"] + gumbel
    top = key.topk(min(16, V), dim=-1).indices
    par = s["tree"]["parent"].long().clamp(min=0)
    tok = top.gather(1, par[:, :, None].expand(-1, -1, top.shape[2])).gather(2, s["tree"]["rank"][:, :, None].clamp(max=top.shape[2] - 1))
    s["tokens"] = tok[:, :, 0].int().contiguous()
    s["uniforms"] = torch.rand((B, 2, N), generator=g, device="cuda")
    s["accepted"] = _accept_outputs(B, N)
    ws = _bytes(fspad.fspad_tree_accept_sample_draft_workspace_bytes(B, N, V))
    t = s["tree"]
    s["call"] = fspad.fspad_tree_accept_sample_draft(s["logits"], s["draft_logits"], s["tokens"], t["parent"], t["n_dev"],
                                                     case["temperature"], s["uniforms"], outputs=s["accepted"], workspace=ws, prepare=True)
    return s


def _head(case, g, tree, sampled):
    """Hidden states, head weights and draft tokens (from the perturbed logits that the head gives)."""
    B, N, Hd, V = case["batch"], case["nodes_max"], case["hidden"], case["vocab"]
    hidden = _normal(g, (B, N, Hd))
    weight = _normal(g, (V, Hd), BF16, 3.0 / math.sqrt(Hd))
    # every state leans towards one token's row (of length 3): that token's logit rises by 9 to 21
    lean = weight[torch.randint(V, (B, N), generator=g, device="cuda")].float()
    hidden = (hidden + lean * (1.0 + 4.0 / 3.0 * torch.rand((B, N, 1), generator=g, device="cuda"))).to(BF16)
    logits = torch.mm(hidden.view(B * N, Hd), weight.t()).float().view(B, N, V)
    return hidden, weight, _draft_tokens(g, logits, tree, sampled)


def _prepare_lm_head(case, seed):
    g = _gen(seed)
    B, N, V = case["batch"], case["nodes_max"], case["vocab"]
    t = _trees(case, seed)
    sampled = case["accept"] == "sample"
    hidden, weight, tokens = _head(case, g, t, sampled)
    if case["packed"]:
        weight = fspad.fspad_pack_weight(weight)
    uniforms = torch.rand((B, 2, N), generator=g, device="cuda")
    kw = {"outputs": _accept_outputs(B, N), "workspace": _bytes(fspad.fspad_tree_accept_lm_head_workspace_bytes(B, N, V)),
          "prepare": True, "packed": case["packed"], "vocab": V if case["packed"] else None}
    if sampled:
        call = fspad.fspad_tree_accept_sample_lm_head(hidden, weight, tokens, t["parent"], t["n_dev"], case["temperature"], uniforms, **kw)
    else:
        call = fspad.fspad_tree_accept_greedy_lm_head(hidden, weight, tokens, t["parent"], t["n_dev"], **kw)
    return {"case": case, "call": call}


def _layer_weights(case, g, packed):
    Hd, I, D = case["hidden"], case["inter"], case["head_dim"]
    attn, qkv = case["n_q_heads"] * D, (case["n_q_heads"] + 2 * case["n_kv_heads"]) * D
    shapes = {"w_qkv": (qkv, Hd), "w_o": (Hd, attn), "w_gate": (I, Hd), "w_up": (I, Hd), "w_down": (2 * Hd, I)}
    w = {k: _normal(g, shp, BF16, 1.0 / math.sqrt(shp[1])) for k, shp in shapes.items()}
    sampler = {"w_up": _normal(g, (I, Hd), BF16, 1.0 / math.sqrt(Hd)), "w_gate": _normal(g, (I, Hd), BF16, 1.0 / math.sqrt(Hd)),
               "w_down": _normal(g, (Hd, I), BF16, 1.0 / math.sqrt(I))}
    if packed:
        w = {k: fspad.fspad_pack_weight(v) for k, v in w.items()}
        sampler = {k: fspad.fspad_pack_weight(v) for k, v in sampler.items()}
    for k in ("gain_attn", "gain_mlp"):
        w[k] = (1.0 + 0.1 * torch.empty(Hd, device="cuda").normal_(generator=g)).to(BF16)
    return w, sampler


def _draft_side(case, seed, g, packed):
    """What the draft side has in hand before a step: weights, its own cache, the rows of one tree level."""
    B, R, Hd, Hkv, D, L = (case[k] for k in ("batch", "rows", "hidden", "n_kv_heads", "head_dim", "kv_max"))
    s = {"case": case, "kv_len": _lens(case), "n": np.full(B, R, np.int32)}
    s["weights"], s["sampler"] = _layer_weights(case, g, packed)
    s["f"], s["e"] = _normal(g, (B * R, Hd)), _normal(g, (B * R, Hd))
    s["draft_k"], s["draft_v"] = _normal(g, (B, Hkv, L + R, D)), _normal(g, (B, Hkv, L + R, D))
    # one level of the tree: a root and its children
    parent = np.zeros((B, R), np.int32)
    parent[:, 0] = -1
    mask = fspad.fspad_tree_build_mask(parent, s["n"])
    s["mask"] = torch.from_numpy(mask.view(np.int64)).cuda()
    s["positions"] = torch.from_numpy(s["kv_len"][:, None] + (parent >= 0).astype(np.int32)).cuda()
    s["draft_logits"] = _logits(g, 1, B * R, case["vocab"])[0]
    return s


def _prepare_draft(case, seed):
    g = _gen(seed)
    s = _draft_side(case, seed, g, case["packed"])
    B, R, Hd = case["batch"], case["rows"], case["hidden"]
    eta = torch.zeros((B * R, Hd), dtype=BF16, device="cuda")
    w = s["sampler"]
    s["calls"] = [
        fspad.fspad_feature_sampler(s["f"], s["e"], w["w_up"], w["w_gate"], w["w_down"], out=eta, packed=case["packed"], prepare=True),
        fspad.fspad_draft_layer(eta.view(B, R, Hd), s["positions"], s["weights"], s["draft_k"], s["draft_v"], s["kv_len"], s["n"],
                                s["mask"], case["n_q_heads"], case["n_kv_heads"], case["head_dim"], packed=case["packed"], prepare=True),
        fspad.fspad_draft_topk(s["draft_logits"], case["topk"], prepare=True)]
    return s


def _prepare_cycle(case, seed):
    g = _gen(seed)
    s = _draft_side(case, seed, g, False)
    B, N, Hq, Hkv, D = (case[k] for k in ("batch", "nodes_max", "n_q_heads", "n_kv_heads", "head_dim"))
    s["candidates"] = _tree_inputs(case, seed)
    s["n_keep"] = N
    s["tree"] = _trees({**case, "nodes_min": N}, seed)
    s["hidden"], s["head"], s["tokens"] = _head(case, g, s["tree"], False)
    cap = (case["kv_max"] + N + 63) // 64 * 64
    s["q"] = _normal(g, (B, N, Hq, D))
    s["k_tree"], s["v_tree"] = _normal(g, (B, N, Hkv, D)), _normal(g, (B, N, Hkv, D))
    s["k_cache"], s["v_cache"] = _normal(g, (B, Hkv, cap, D)), _normal(g, (B, Hkv, cap, D))
    s["appended"] = [c[:, :, case["kv_max"]:case["kv_max"] + N] for c in (s["k_cache"], s["v_cache"])]
    return s


def _run_cycle(s):
    case = s["case"]
    B, R, Hd, N = case["batch"], case["rows"], case["hidden"], case["nodes_max"]
    w = s["sampler"]
    eta = fspad.fspad_feature_sampler(s["f"], s["e"], w["w_up"], w["w_gate"], w["w_down"])
    layer = fspad.fspad_draft_layer(eta.view(B, R, Hd), s["positions"], s["weights"], s["draft_k"], s["draft_v"], s["kv_len"], s["n"],
                                    s["mask"], case["n_q_heads"], case["n_kv_heads"], case["head_dim"])
    top = fspad.fspad_draft_topk(s["draft_logits"], case["topk"])
    parent, _, n_nodes, mask, node_cand = fspad.fspad_tree_build(*s["candidates"], s["n_keep"], N)
    out = fspad.fspad_tree_attn(s["q"], s["k_tree"], s["v_tree"], s["k_cache"], s["v_cache"], s["kv_len"], s["tree"]["n"], mask)
    accepted = fspad.fspad_tree_accept_greedy_lm_head(s["hidden"], s["head"], s["tokens"], parent, n_nodes)
    fspad.fspad_kv_commit(s["k_tree"], s["v_tree"], s["k_cache"], s["v_cache"], s["kv_len"], accepted[0], accepted[1])
    return [eta, layer, top, (parent, n_nodes, mask, node_cand), out, accepted, s["appended"]]


def prepare(case, seed):
    return {"verify": _prepare_verify, "accept": _prepare_accept, "lm_head": _prepare_lm_head, "draft": _prepare_draft,
            "cycle": _prepare_cycle}[case["kind"]](case, seed)


def run(state):
    kind = state["case"]["kind"]
    if kind == "verify":
        return _run_verify(state)
    if kind == "draft":
        return [call() for call in state["calls"]]
    if kind == "cycle":
        return _run_cycle(state)
    return state["call"]()


# ----------------------------------------------------------------------------------------- what a pass needs

def _attn_work(kv_len, nodes, hq, hkv, D, item):
    """K and V of prefix and tree once per kv head, Q once, the output once; both products, mask not subtracted."""
    byts = flops = 0
    for L, n in zip(kv_len.tolist(), nodes.tolist()):
        byts += (2 * (L + n) * hkv * D + 2 * n * hq * D) * item
        flops += 4 * n * (L + n) * hq * D
    return byts, flops


def _draft_work(case):
    rows, Hd, I = case["batch"] * case["rows"], case["hidden"], case["inter"]
    hq, hkv, D = case["n_q_heads"], case["n_kv_heads"], case["head_dim"]
    weights = 3 * Hd * I + Hd * (hq + 2 * hkv) * D + Hd * hq * D + 4 * Hd * I
    byts, flops = _attn_work(np.full(case["batch"], case["kv_max"]), np.full(case["batch"], case["rows"]), hq, hkv, D, 2)
    byts += 2 * weights + 4 * rows * case["vocab"] + 2 * rows * Hd * 5
    return byts, flops + 2 * rows * weights


def work(case):
    kind, B = case["kind"], case["batch"]
    if kind == "draft":
        byts, flops = _draft_work(case)
        return {"bytes": byts, "flops": flops}
    nodes = _nodes(case)
    if kind == "accept":
        return {"bytes": 8 * int(nodes.sum()) * case["vocab"], "flops": 0}
    head_bytes, head_flops = 2 * case.get("hidden", 0) * (case["vocab"] + int(nodes.sum())), 2 * int(nodes.sum()) * case.get("hidden", 0) * case["vocab"]
    if kind == "lm_head":
        return {"bytes": head_bytes, "flops": head_flops}
    hq, hkv, D = case["n_q_heads"], case["n_kv_heads"], case["head_dim"]
    if kind == "cycle":
        a, f = _attn_work(_lens(case), np.full(B, case["nodes_max"]), hq, hkv, D, 2)
        d, df = _draft_work(case)
        return {"bytes": a + d + head_bytes, "flops": f + df + head_flops}
    a, f = _attn_work(_lens(case), nodes, hq, hkv, D, 4 if case["dtype"] == "f32" else 2)
    return {"bytes": case["layers"] * a + 4 * int(nodes.sum()) * case["vocab"], "flops": case["layers"] * f}


def tolerance(case):
    """About four times what the results differ by from a 64-bit evaluation (fp32 attention 3.9e-7 and at most
    2.1e-6; bf16 attention 2.3e-3 and 1.1e-2, its weights and results being rounded to bf16; the draft side 2.9e-3
    and 1.6e-2 over its five or six roundings). Tokens, paths and lengths from logits are exact; from hidden states
    a decision is only as good as fp32 sums of the logits."""
    if case["kind"] == "accept":
        return "exact"
    if case["kind"] == "lm_head":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}
    if case.get("dtype") == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    return {"rel": 1e-2, "max": 0.06}
