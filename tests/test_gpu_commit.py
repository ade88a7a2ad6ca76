"""GPU parity of the KV-cache commit against the CPU oracle, through the C ABI. Bar: the caches
are bit-identical to the oracle's everywhere (moved rows and untouched positions alike)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2408_15562_amd as fspad
from workloads import CONFIGS, gen_draft_tokens, gen_logits, gen_qkv, gen_trees

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    from tests import _harness
    return _harness


def _accepted_paths(seed, B, N, n_nodes=None):
    parent, n_nodes = gen_trees(seed, B, N, 6, min(10, max(1, N - 1)), n_nodes=n_nodes)
    logits = gen_logits(seed, B, N, 400, peak=4.0)
    tokens = gen_draft_tokens(seed, logits, parent, n_nodes, "greedy")
    path, path_len, _, _ = oracle.accept_greedy(logits, tokens, parent, n_nodes)
    return path, path_len


def _bits(t: torch.Tensor) -> np.ndarray:
    t = t.contiguous().cpu()
    return (t.view(torch.int16) if t.dtype == torch.bfloat16 else t.view(torch.int32)).numpy()


@pytest.mark.parametrize("B,N,Hkv,D,L", [(1, 1, 1, 64, 0), (2, 26, 32, 128, 300), (3, 60, 8, 128, 77), (5, 33, 2, 64, 129),
                                         (130, 26, 2, 64, 40)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("interleave", [False, True])
def test_commit_matches_oracle(H, B, N, Hkv, D, L, dtype, interleave):
    seed = 7000 + B + N + Hkv + D
    rng = np.random.default_rng(seed)
    kv_len = rng.integers(max(L - 30, 0), L + 1, B).astype(np.int32)
    cap = L + N + 3
    _, kt, vt, kc, vc = gen_qkv(seed, B, N, Hkv, Hkv, D, cap, dtype)
    path, path_len = _accepted_paths(seed, B, N)
    kt_d, vt_d = H.to_dev(kt, dtype), H.to_dev(vt, dtype)
    if interleave:
        both = torch.stack([H.to_dev(kc, dtype), H.to_dev(vc, dtype)], dim=2).contiguous()
        kc_d, vc_d = both[:, :, 0], both[:, :, 1]
    else:
        kc_d, vc_d = H.to_dev(kc, dtype), H.to_dev(vc, dtype)
    len_out = torch.full((B,), -5, dtype=torch.int32, device=H.DEV)
    fspad.fspad_kv_commit(kt_d, vt_d, kc_d, vc_d, kv_len, torch.from_numpy(path).to(H.DEV),
                          torch.from_numpy(path_len).to(H.DEV), len_out)
    torch.cuda.synchronize()
    k_ref, v_ref, len_ref = oracle.kv_commit(kt, vt, kc, vc, kv_len, path, path_len)
    assert np.array_equal(len_out.cpu().numpy(), len_ref)
    assert np.array_equal(_bits(kc_d), _bits(H.to_dev(k_ref, dtype)))
    assert np.array_equal(_bits(vc_d), _bits(H.to_dev(v_ref, dtype)))


def test_malformed_paths_move_nothing(H):
    """Lengths and node indices outside their ranges are not followed."""
    B, N, Hkv, D, L = 3, 8, 2, 64, 10
    _, kt, vt, kc, vc = gen_qkv(1, B, N, Hkv, Hkv, D, L + N, "bf16")
    kt_d, vt_d, kc_d, vc_d = [H.to_dev(a, "bf16") for a in (kt, vt, kc, vc)]
    before_k, before_v = _bits(kc_d).copy(), _bits(vc_d).copy()
    path = torch.tensor([[0, 99, -1, 0, 0, 0, 0, 0], [-3] * 8, [0] * 8], dtype=torch.int32, device=H.DEV)
    path_len = torch.tensor([3, 8, -2], dtype=torch.int32, device=H.DEV)
    fspad.fspad_kv_commit(kt_d, vt_d, kc_d, vc_d, np.full(B, L, np.int32), path, path_len)
    torch.cuda.synchronize()
    after_k = _bits(kc_d)
    expect = before_k.copy()
    expect[0, :, L] = _bits(kt_d)[0, 0]            # only the one valid entry of sequence 0 is moved
    assert np.array_equal(after_k, expect)
    changed_v = np.argwhere(np.any(_bits(vc_d) != before_v, axis=-1))
    assert {tuple(x) for x in changed_v.tolist()} <= {(0, g, L) for g in range(Hkv)}


def test_two_verification_steps_chained_on_the_device(H):
    """attention -> acceptance -> commit -> attention: the second step's output over the cache the
    library committed equals the oracle's second step over the cache the oracle committed."""
    c = CONFIGS["c0"]
    B, N, Hq, Hkv, D, L = 2, c.n_nodes, c.n_q_heads, c.n_kv_heads, c.head_dim, c.kv_len
    cap = L + 2 * N
    kv_len = np.array([L, L - 11], np.int32)
    _, _, _, kc, vc = gen_qkv(40, B, N, Hq, Hkv, D, cap, "bf16")
    kc_d, vc_d = H.to_dev(kc, "bf16"), H.to_dev(vc, "bf16")
    for step in range(2):
        seed = 41 + step
        parent, n_nodes = gen_trees(seed, B, N, c.tree_depth, c.tree_topk)
        mask = fspad.fspad_tree_build_mask(parent, n_nodes)
        q, kt, vt, _, _ = gen_qkv(seed, B, N, Hq, Hkv, D, 1, "bf16")
        logits = gen_logits(seed, B, N, 1000, peak=4.0)
        tokens = gen_draft_tokens(seed, logits, parent, n_nodes, "greedy")
        q_d, kt_d, vt_d = [H.to_dev(a, "bf16") for a in (q, kt, vt)]
        out = fspad.fspad_tree_attn(q_d, kt_d, vt_d, kc_d, vc_d, kv_len, n_nodes,
                                    torch.from_numpy(mask.view(np.int64)).to(H.DEV), out_dtype=torch.float32)
        acc = fspad.fspad_tree_accept_greedy(*[torch.from_numpy(a).to(H.DEV) for a in (logits, tokens, parent, n_nodes)])
        len_out = torch.empty(B, dtype=torch.int32, device=H.DEV)
        fspad.fspad_kv_commit(kt_d, vt_d, kc_d, vc_d, kv_len, acc[0], acc[1], len_out)
        torch.cuda.synchronize()
        ref = oracle.tree_attn(q, kt, vt, kc, vc, kv_len, n_nodes, parent, packed_mask=mask, nthreads=8)
        assert H.rel_err(out, ref) <= H.TOL["bf16"]
        path, path_len, _, _ = oracle.accept_greedy(logits, tokens, parent, n_nodes)
        kc, vc, new_len = oracle.kv_commit(kt, vt, kc, vc, kv_len, path, path_len)
        assert np.array_equal(len_out.cpu().numpy(), new_len)
        assert np.array_equal(_bits(kc_d), _bits(H.to_dev(kc, "bf16")))
        kv_len = new_len
    assert kv_len.min() > L - 11 + 1


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("Hkv", [32, 64, 65, 100])
def test_commit_of_wide_rows(H, dtype, Hkv):
    """Rows of one to four turns of a workgroup (1024 pieces of 16 bytes each), the last one ragged."""
    test_commit_matches_oracle(H, 2, 5, Hkv, 128, 20, dtype, False)
