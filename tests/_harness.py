"""Test harness: feeds the same seeded inputs to the GPU library and to the CPU oracle."""
from __future__ import annotations

import numpy as np
import torch

import oracle
import paper_2408_15562_amd as fspad
from workloads import gen_draft_tokens, gen_lm_head, gen_lm_head_exact, gen_logits, gen_qkv, gen_trees, gen_uniforms

DEV = "cuda:0"
TOL = {"bf16": 2e-2, "f32": 1e-5}   # max-abs-error relative to the RMS of the oracle output
MARGIN = 1e-9                        # sampling decisions closer than this to a threshold are not compared


def to_dev(a: np.ndarray, dtype: str):
    t = torch.from_numpy(np.ascontiguousarray(a))
    return t.to(DEV, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)


class AttnCase:
    """One attention problem on both sides. Cache tensors are views into a larger allocation
    (Lcap > max kv_len, optional interleaved K/V heads) so that the strides are exercised."""

    def __init__(self, seed, B, N, Hq, Hkv, D, L, dtype="bf16", n_nodes=None, kv_len=None, depth=6, topk=10,
                 l_cap=None, interleave=False, parent=None):
        self.dtype, self.shape = dtype, (B, N, Hq, Hkv, D)
        kv_len = np.full(B, L, np.int32) if kv_len is None else np.asarray(kv_len, np.int32)
        self.kv_len = kv_len
        lmax = int(kv_len.max())
        l_cap = max(lmax, 1) if l_cap is None else l_cap
        q, kt, vt, kc, vc = gen_qkv(seed, B, N, Hq, Hkv, D, l_cap, dtype)
        if parent is None:
            topk = min(topk, max(1, N - 1))
            parent, n_nodes = gen_trees(seed, B, N, depth, topk, n_nodes=n_nodes)
        else:
            parent = np.asarray(parent, np.int32).reshape(B, N)
            n_nodes = np.full(B, N, np.int32) if n_nodes is None else np.asarray(n_nodes, np.int32)
        self.parent, self.n_nodes = parent, n_nodes
        self.host = dict(q=q, k_tree=kt, v_tree=vt, k_cache=kc, v_cache=vc)
        self.mask = fspad.fspad_tree_build_mask(parent, n_nodes)
        self.q, self.k_tree, self.v_tree = to_dev(q, dtype), to_dev(kt, dtype), to_dev(vt, dtype)
        if interleave:  # K and V heads interleaved in one buffer: [B, Hkv, 2, Lcap, D]
            both = torch.stack([to_dev(kc, dtype), to_dev(vc, dtype)], dim=2).contiguous()
            self.k_cache, self.v_cache = both[:, :, 0], both[:, :, 1]
        else:
            self.k_cache, self.v_cache = to_dev(kc, dtype), to_dev(vc, dtype)
        self.mask_dev = torch.from_numpy(self.mask.view(np.int64)).to(DEV)

    def run_gpu(self, out_dtype=torch.float32, scale=0.0, splits=0):
        # output and workspace hold NaN: an allocation may still hold the results of a call before, and an output or a
        # partial result that nobody wrote must not pass for one
        out = torch.full(self.q.shape, float("nan"), dtype=out_dtype, device=DEV)
        desc = fspad.make_attn_desc(self.q, self.k_tree, self.k_cache, out_dtype, scale, splits)
        need = fspad.fspad_tree_attn_workspace_bytes(desc, int(self.kv_len.max()))
        workspace = torch.full((max(need, 16),), 0xFF, dtype=torch.uint8, device=DEV)
        fspad.fspad_tree_attn(self.q, self.k_tree, self.v_tree, self.k_cache, self.v_cache, self.kv_len, self.n_nodes, self.mask_dev,
                              out=out, workspace=workspace, desc=desc)
        torch.cuda.synchronize()
        return out

    def run_oracle(self, scale=None, heads=None, nthreads=16):
        h = self.host
        B, N, Hq, Hkv, D = self.shape
        if heads is None:
            return oracle.tree_attn(h["q"], h["k_tree"], h["v_tree"], h["k_cache"], h["v_cache"], self.kv_len,
                                    self.n_nodes, self.parent, packed_mask=self.mask, scale=scale, nthreads=nthreads)
        # a subset of query heads: run them as an MHA problem over their own kv heads
        G = Hq // Hkv
        kvh = [x // G for x in heads]
        return oracle.tree_attn(h["q"][:, :, heads], h["k_tree"][:, :, kvh], h["v_tree"][:, :, kvh],
                                h["k_cache"][:, kvh], h["v_cache"][:, kvh], self.kv_len, self.n_nodes, self.parent,
                                packed_mask=self.mask, scale=scale, nthreads=nthreads)


def rel_err(gpu: torch.Tensor, ref: np.ndarray) -> float:
    """max over sequences of  max |gpu - ref| / RMS(ref over the sequence's live rows)
    (every sequence of a batch is an attention problem of its own, with its own output scale)."""
    g = gpu.detach().to(torch.float64).cpu().numpy()
    assert g.shape == ref.shape
    assert np.all(np.isfinite(g))
    worst = 0.0
    for b in range(ref.shape[0]):
        live = ref[b][np.abs(ref[b]).sum(axis=-1) > 0]
        rms = float(np.sqrt(np.mean(live ** 2))) if live.size else 1.0
        worst = max(worst, float(np.abs(g[b] - ref[b]).max() / rms))
    return worst


class AcceptCase:
    def __init__(self, seed, B, N, V, mode="greedy", depth=6, topk=10, peak=0.0, n_nodes=None, row_pad=0,
                 parent=None, logits=None, tokens=None, uniforms=None):
        if parent is None:
            topk = min(topk, max(1, N - 1))
            parent, n_nodes = gen_trees(seed, B, N, depth, topk, n_nodes=n_nodes)
        else:
            n_nodes = np.full(B, N, np.int32) if n_nodes is None else np.asarray(n_nodes, np.int32)
        self.parent, self.n_nodes = np.ascontiguousarray(parent, np.int32), n_nodes
        self.logits = gen_logits(seed, B, N, V, peak=peak) if logits is None else logits
        self.tokens = gen_draft_tokens(seed, self.logits, self.parent, n_nodes, mode) if tokens is None else tokens
        self.uniforms = gen_uniforms(seed, B, N) if uniforms is None else uniforms
        self.B, self.N, self.V = B, N, V
        if row_pad:  # rows that are not 16-byte aligned / padded strides
            buf = torch.full((B, N, V + row_pad), float("nan"), dtype=torch.float32, device=DEV)
            buf[:, :, :V] = torch.from_numpy(self.logits).to(DEV)
            self.logits_dev = buf[:, :, :V]
        else:
            self.logits_dev = torch.from_numpy(self.logits).to(DEV)
        self.tokens_dev = torch.from_numpy(self.tokens).to(DEV)
        self.parent_dev = torch.from_numpy(self.parent).to(DEV)
        self.n_nodes_dev = torch.from_numpy(np.asarray(n_nodes, np.int32)).to(DEV)
        self.uniforms_dev = torch.from_numpy(self.uniforms).to(DEV)

    def gpu_greedy(self):
        out = fspad.fspad_tree_accept_greedy(self.logits_dev, self.tokens_dev, self.parent_dev, self.n_nodes_dev)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in out]

    def gpu_sample(self, temperature=1.0):
        out = fspad.fspad_tree_accept_sample(self.logits_dev, self.tokens_dev, self.parent_dev, self.n_nodes_dev,
                                             temperature, self.uniforms_dev)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in out]

    def cpu_greedy(self):
        return list(oracle.accept_greedy(self.logits, self.tokens, self.parent, self.n_nodes))

    def cpu_sample(self, temperature=1.0):
        return list(oracle.accept_sample(self.logits, self.tokens, self.parent, self.n_nodes, temperature, self.uniforms))


def assert_accept_equal(gpu, cpu, keep=None):
    names = ("path", "path_len", "tokens", "n_tokens")
    for name, g, c in zip(names, gpu, cpu[:4]):
        if keep is not None:
            g, c = g[keep], c[keep]
        np.testing.assert_array_equal(g, c, err_msg=name)


class LmHeadCase:
    """Greedy acceptance from hidden states on both sides. The draft tokens are the top entries of a
    perturbed copy of the oracle's own logits, so that walks go several levels deep."""

    def __init__(self, seed, B, N, Hd, V, depth=6, topk=10, n_nodes=None, noise=1.0, exact=False):
        topk = min(topk, max(1, N - 1))
        self.parent, self.n_nodes = gen_trees(seed, B, N, depth, topk, n_nodes=n_nodes)
        self.hidden, self.w = (gen_lm_head_exact if exact else gen_lm_head)(seed, B, N, Hd, V)
        logits = (self.hidden.reshape(B * N, Hd) @ self.w.T).reshape(B, N, V)   # fp32: only steers the drafts
        self.tokens = gen_draft_tokens(seed, logits, self.parent, self.n_nodes, "greedy", noise)
        self.shape = (B, N, Hd, V)
        self.hidden_dev, self.w_dev = to_dev(self.hidden, "bf16"), to_dev(self.w, "bf16")
        self.tokens_dev = torch.from_numpy(self.tokens).to(DEV)
        self.parent_dev = torch.from_numpy(np.ascontiguousarray(self.parent, np.int32)).to(DEV)
        self.n_nodes_dev = torch.from_numpy(np.asarray(self.n_nodes, np.int32)).to(DEV)

    def packed_w(self):
        """the LM head in the library's tile order (flat: the vocabulary may not fill the last tile row)"""
        if not hasattr(self, "_packed"):
            self._packed = fspad.fspad_pack_weight(self.w_dev).reshape(-1)
        return self._packed

    def gpu(self, packed=False):
        out = fspad.fspad_tree_accept_greedy_lm_head(self.hidden_dev, self.packed_w() if packed else self.w_dev,
                                                     self.tokens_dev, self.parent_dev, self.n_nodes_dev, packed=packed,
                                                     vocab=self.shape[3] if packed else None)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in out]

    def cpu(self):
        return list(oracle.lm_head_greedy(self.hidden, self.w, self.tokens, self.parent, self.n_nodes))

    def gpu_sample(self, temperature=1.0, seed=0, packed=False):
        uni = gen_uniforms(seed, self.shape[0], self.shape[1])
        out = fspad.fspad_tree_accept_sample_lm_head(self.hidden_dev, self.packed_w() if packed else self.w_dev,
                                                     self.tokens_dev, self.parent_dev, self.n_nodes_dev, temperature,
                                                     torch.from_numpy(uni).to(DEV), packed=packed,
                                                     vocab=self.shape[3] if packed else None)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in out]

    def cpu_sample(self, temperature=1.0, seed=0):
        uni = gen_uniforms(seed, self.shape[0], self.shape[1])
        return list(oracle.lm_head_sample(self.hidden, self.w, self.tokens, self.parent, self.n_nodes, temperature, uni))


# fp32 accumulation of the logits: a target token is compared only where the oracle's winning logit
# leads the runner-up by more than this (logits ~ N(0, 3^2); K <= 8192 terms of fp32 rounding stay
# two orders of magnitude below it), and the winning logit itself must agree to LOGIT_TOL
LM_HEAD_MARGIN = 1e-3
LM_HEAD_LOGIT_TOL = 2e-4


def assert_lm_head_equal(gpu, cpu, require_decided=True):
    path, path_len, tokens, n_tokens, node_target, node_top = gpu
    c_path, c_len, c_tokens, c_ntok, c_target, c_top, c_margin = cpu
    live = c_target >= 0
    decided = live & (np.nan_to_num(c_margin, nan=0.0) > LM_HEAD_MARGIN)
    np.testing.assert_array_equal(node_target[decided], c_target[decided], err_msg="target tokens")
    assert (node_target[~live] == -1).all()
    np.testing.assert_allclose(node_top[live], c_top[live], rtol=0, atol=LM_HEAD_LOGIT_TOL * max(1.0, np.abs(c_top[live]).max()))
    assert np.isneginf(node_top[~live]).all()
    # an undecided row must still pick one of the entries within the margin: its logit is the oracle's top
    all_decided = bool((decided == live).all())
    if require_decided:
        assert all_decided, "seeded inputs with an undecided argmax: pick another seed"
    if all_decided:
        assert_accept_equal((path, path_len, tokens, n_tokens), (c_path, c_len, c_tokens, c_ntok))
    return all_decided


# sampling from hidden states: the kernel's exponentials are fp32 on fp32 logit sums, the oracle's fp64 on
# correctly rounded logits; a sequence is compared when every decision of its walk has a relative
# margin above this
LM_HEAD_SAMPLE_MARGIN = 1e-4


LM_HEAD_SAMPLE_STATS = {"sequences": 0, "compared": 0, "excluded": 0, "excluded_that_differ": 0}


def assert_lm_head_sample_equal(gpu, cpu, min_compared=0.75):
    """Sequences whose smallest decision margin is above LM_HEAD_SAMPLE_MARGIN must agree bit for bit.
    The others are not asserted on, but they are counted: how many of them actually differ is
    printed (and accumulated in LM_HEAD_SAMPLE_STATS), so that the exclusion is measured, not assumed."""
    margin = cpu[4]
    keep = margin >= LM_HEAD_SAMPLE_MARGIN
    assert keep.mean() >= min_compared, f"only {keep.sum()} of {keep.size} sequences are decided: pick another seed"
    assert_accept_equal(gpu, cpu, keep=keep)
    same = np.ones(keep.shape, dtype=bool)
    for g, c in zip(gpu, cpu[:4]):
        same &= (g.reshape(len(keep), -1) == c.reshape(len(keep), -1)).all(axis=1)
    differ = int((~same & ~keep).sum())
    LM_HEAD_SAMPLE_STATS["sequences"] += int(keep.size)
    LM_HEAD_SAMPLE_STATS["compared"] += int(keep.sum())
    LM_HEAD_SAMPLE_STATS["excluded"] += int((~keep).sum())
    LM_HEAD_SAMPLE_STATS["excluded_that_differ"] += differ
    print(f"lm_head sampling: {int(keep.sum())}/{keep.size} sequences above the margin (all equal); "
          f"{int((~keep).sum())} below it, of which {differ} differ from the oracle")
    return int(keep.sum())
