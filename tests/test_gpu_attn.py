"""GPU parity of fspad_tree_attn against the CPU oracle, through the C ABI.

Bar: max-abs-error <= 2e-2 x RMS(oracle output) for bf16 inputs, <= 1e-5 x RMS for fp32.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from workloads import CONFIGS, chain_tree  # noqa: E402


@pytest.fixture(scope="module")
def H():
    from tests import _harness
    return _harness


def _check(H, case, tol, **kw):
    out = case.run_gpu(**kw)
    ref = case.run_oracle(scale=kw.get("scale") or None)
    err = H.rel_err(out, ref)
    assert err <= tol, f"rel err {err:.3e} > {tol}"
    # rows of unused tree slots are written as zeros
    for b, n in enumerate(case.n_nodes):
        assert torch.all(out[b, int(n):] == 0)
    return out, ref, err


def test_config0_tiny_fp32(H):
    c = CONFIGS["c0"]
    case = H.AttnCase(100, c.batch, c.n_nodes, c.n_q_heads, c.n_kv_heads, c.head_dim, c.kv_len, "f32",
                      depth=c.tree_depth, topk=c.tree_topk)
    _check(H, case, H.TOL["f32"])


@pytest.mark.parametrize("N,L,Hq,Hkv,D", [
    (1, 0, 2, 2, 64), (2, 1, 4, 1, 64), (26, 15, 4, 4, 128), (31, 17, 8, 2, 64), (33, 255, 2, 1, 128),
    (60, 256, 8, 8, 64), (64, 100, 4, 2, 128),
])
def test_fp32_sweep(H, N, L, Hq, Hkv, D):
    case = H.AttnCase(101 + N + L, 2, N, Hq, Hkv, D, L, "f32", l_cap=L + 3)
    _check(H, case, H.TOL["f32"])


@pytest.mark.parametrize("N", [1, 2, 16, 17, 26, 31, 32, 33, 48, 60, 63, 64])
@pytest.mark.parametrize("L", [0, 1, 31, 32, 33, 255, 1000])
def test_bf16_mha_sweep_nodes_and_lengths(H, N, L):
    case = H.AttnCase(7 * N + L, 2, N, 2, 2, 128, L, "bf16", l_cap=L + 5)
    _check(H, case, H.TOL["bf16"])


@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (4, 1), (8, 2), (8, 1), (16, 2)])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N", [5, 26, 60])
def test_bf16_gqa_and_head_dim(H, Hq, Hkv, D, N):
    case = H.AttnCase(13 * Hq + D + N, 1, N, Hq, Hkv, D, 200, "bf16")
    _check(H, case, H.TOL["bf16"])


@pytest.mark.parametrize("N,Hq,Hkv,D", [(60, 8, 2, 128), (40, 4, 1, 64), (26, 16, 2, 128), (64, 8, 1, 64)])
@pytest.mark.parametrize("L,splits", [(0, 0), (33, 0), (200, 0), (1000, 0), (1000, 7), (3000, 64)])
def test_bf16_shared_stage_kernel(H, N, Hq, Hkv, D, L, splits):
    """Grouped-query shapes with more than 128 rows per KV head take the kernel whose wavefronts
    share K/V blocks through LDS."""
    case = H.AttnCase(31 * N + L + 4, 2, N, Hq, Hkv, D, L, "bf16", l_cap=L + 9)
    _check(H, case, H.TOL["bf16"], **({"splits": splits} if splits else {}))


@pytest.mark.parametrize("splits", [1, 2, 3, 7, 16, 50, 333, 4096])
def test_bf16_workgroup_counts(H, splits):
    """Any number of workgroups cuts the flat block list differently (whole units, units cut in
    two or many segments, more workgroups than blocks); the result must not depend on it."""
    case = H.AttnCase(300 + splits, 2, 26, 4, 4, 128, 777, "bf16", kv_len=[777, 40])
    out, ref, _ = _check(H, case, H.TOL["bf16"], splits=splits)
    # run-to-run determinism (no floating-point atomics, fixed merge order)
    for _ in range(3):
        again = case.run_gpu(splits=splits)
        assert torch.equal(out, again)


@pytest.mark.parametrize("N,splits", [(26, 0), (26, 300), (26, 511), (17, 400), (26, 256)])
def test_bf16_small_tiles_above_and_below_one_workgroup_per_cu(H, N, splits):
    """32-row tiles with one workgroup per compute unit at most, and with two (more than 256
    workgroups), on a problem long enough for either: streams of 4 to 30 blocks per wave."""
    case = H.AttnCase(500 + N + splits, 2, N, 8, 8, 128, 2100, "bf16", kv_len=[2100, 1500])
    _check(H, case, H.TOL["bf16"], splits=splits)


@pytest.mark.parametrize("dtype,N,Hq,Hkv", [("bf16", 9, 2, 2), ("bf16", 40, 4, 1), ("f32", 9, 2, 2)])
def test_more_sequences_than_one_launch_takes(H, dtype, N, Hq, Hkv):
    """Sequences go to the kernels in slices of 128 (their lengths travel as kernel arguments): 130
    ragged sequences take two launches that reuse one workspace in stream order."""
    B = 130
    rng = np.random.default_rng(130 + N)
    kv_len = rng.integers(0, 90, B).astype(np.int32)
    n_nodes = rng.integers(1, N + 1, B).astype(np.int32)
    case = H.AttnCase(1300 + N, B, N, Hq, Hkv, 64, 90, dtype, kv_len=kv_len, n_nodes=n_nodes, topk=4)
    _check(H, case, H.TOL[dtype])


def test_bf16_shared_workspace_sees_no_stale_partials(H):
    """Two different problems of one shape alternate on one workspace, launched back to back: a
    merge that picked up the other problem's leftovers would not reproduce the result obtained
    on a private workspace."""
    import paper_2408_15562_amd as fspad
    cases = [H.AttnCase(340 + i, 1, 26, 8, 8, 128, 1500, "bf16") for i in range(2)]
    desc = fspad.make_attn_desc(cases[0].q, cases[0].k_tree, cases[0].k_cache, torch.float32, 0.0)
    shared = torch.empty(fspad.fspad_tree_attn_workspace_bytes(desc, 1500), dtype=torch.uint8, device=H.DEV)
    private = [c.run_gpu() for c in cases]
    for i, c in enumerate(cases):
        assert H.rel_err(private[i], c.run_oracle()) <= H.TOL["bf16"]
    for rep in range(6):
        for i, c in enumerate(cases):   # no host synchronisation in between: back-to-back launches
            out = fspad.fspad_tree_attn(c.q, c.k_tree, c.v_tree, c.k_cache, c.v_cache, c.kv_len, c.n_nodes,
                                        c.mask_dev, workspace=shared, out_dtype=torch.float32)
            assert torch.equal(out, private[i]), f"repetition {rep}, problem {i}"


@pytest.mark.parametrize("N,Hq,Hkv", [(26, 2, 2), (60, 2, 2), (60, 8, 2), (40, 4, 1)])
@pytest.mark.parametrize("splits", [0, 1])
def test_bf16_scores_that_keep_growing(H, N, Hq, Hkv, splits):
    """Keys whose scores climb along the prefix (by far more than the slack the kernel leaves before
    it moves a row's softmax shift) force the shift to move again and again in the middle of the
    stream, in some row tiles and not in others; a ramp in the other direction never moves it."""
    L = 1500
    for direction in (1.0, -1.0):
        case = H.AttnCase(900 + N + Hq, 1, N, Hq, Hkv, 128, L, "bf16")
        ramp = np.linspace(-1.0, 1.0, L)[None, None, :, None] * direction
        k = case.host["k_cache"]
        # rows of Q get different signs, so that growth happens for some rows only
        q = case.host["q"]
        q_dir = np.sign(q.sum(axis=-1, keepdims=True)) * np.ones_like(q) * 0.25
        k_new = (k * 0.3 + 4.0 * ramp * np.ones_like(k)).astype(np.float32)
        q_new = (q * 0.3 + q_dir).astype(np.float32)
        # round to bf16 on both sides
        case.host["k_cache"] = torch.from_numpy(k_new).to(torch.bfloat16).float().numpy()
        case.host["q"] = torch.from_numpy(q_new).to(torch.bfloat16).float().numpy()
        case.k_cache = H.to_dev(case.host["k_cache"], "bf16")
        case.q = H.to_dev(case.host["q"], "bf16")
        _check(H, case, H.TOL["bf16"], splits=splits)


def test_bf16_ragged_batch_and_strided_cache(H):
    case = H.AttnCase(400, 4, 60, 8, 2, 128, 0, "bf16", kv_len=[513, 0, 64, 1], n_nodes=[60, 1, 33, 17],
                      l_cap=600, interleave=True)
    _check(H, case, H.TOL["bf16"])
    _check(H, case, H.TOL["bf16"], splits=4)
    _check(H, case, H.TOL["bf16"], splits=40)


def test_bf16_output_is_rounded_fp32_output(H):
    case = H.AttnCase(401, 1, 26, 4, 4, 128, 300, "bf16")
    o32 = case.run_gpu(out_dtype=torch.float32)
    o16 = case.run_gpu(out_dtype=torch.bfloat16)
    assert torch.equal(o16, o32.to(torch.bfloat16))
    o16s = case.run_gpu(out_dtype=torch.bfloat16, splits=3)
    assert torch.equal(o16s, case.run_gpu(out_dtype=torch.float32, splits=3).to(torch.bfloat16))


def test_custom_scale(H):
    case = H.AttnCase(402, 1, 26, 4, 2, 64, 100, "bf16")
    _check(H, case, H.TOL["bf16"], scale=0.05)
    case32 = H.AttnCase(403, 1, 26, 4, 2, 64, 100, "f32")
    _check(H, case32, H.TOL["f32"], scale=0.05)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_zero_query_closed_form_on_gpu(H, dtype):
    """Q = 0 => every row is the plain mean of the visible value rows: catches mask and stride
    mistakes that a tolerance could hide."""
    case = H.AttnCase(404, 1, 60, 2, 1, 128, 100, dtype)
    case.q.zero_()
    out = case.run_gpu().double().cpu().numpy()
    v_pre = case.host["v_cache"][0, 0, :100].astype(np.float64)
    v_tree = case.host["v_tree"][0, :, 0].astype(np.float64)
    for i in range(60):
        anc, a = [], i
        while a >= 0:
            anc.append(a)
            a = int(case.parent[0, a])
        expect = (v_pre.sum(0) + v_tree[anc].sum(0)) / (100 + len(anc))
        tol = 2e-2 * np.sqrt(np.mean(expect ** 2)) if dtype == "bf16" else 1e-5
        assert np.abs(out[0, i] - expect).max() <= tol


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_chain_tree_is_causal_attention_on_gpu(H, dtype):
    import torch.nn.functional as F
    N, L, Hh, D = 33, 70, 2, 64
    case = H.AttnCase(405, 1, N, Hh, Hh, D, L, dtype, parent=chain_tree(N))
    out = case.run_gpu().double().cpu()
    h = case.host
    k_all = torch.from_numpy(np.concatenate([h["k_cache"][0, :, :L], h["k_tree"][0].transpose(1, 0, 2)], axis=1)).double()
    v_all = torch.from_numpy(np.concatenate([h["v_cache"][0, :, :L], h["v_tree"][0].transpose(1, 0, 2)], axis=1)).double()
    q_full = torch.zeros(Hh, L + N, D, dtype=torch.float64)
    q_full[:, L:] = torch.from_numpy(h["q"][0].transpose(1, 0, 2)).double()
    ref = F.scaled_dot_product_attention(q_full[None], k_all[None], v_all[None], is_causal=True)[0, :, L:]
    ref = ref.permute(1, 0, 2)
    rms = ref.pow(2).mean().sqrt().item()
    assert (out[0] - ref).abs().max().item() <= H.TOL[dtype] * rms


def test_config1_vicuna7b_layer_full(H):
    c = CONFIGS["c1"]
    case = H.AttnCase(500, c.batch, c.n_nodes, c.n_q_heads, c.n_kv_heads, c.head_dim, c.kv_len, "bf16",
                      depth=c.tree_depth, topk=c.tree_topk)
    _check(H, case, H.TOL["bf16"])
    out16 = case.run_gpu(out_dtype=torch.bfloat16)
    # bf16 output: the fp32 bound plus half a bf16 ulp of the largest output
    ref = case.run_oracle()
    assert H.rel_err(out16.float(), ref) <= H.TOL["bf16"] + 2.0 ** -8 * np.abs(ref).max() / np.sqrt(np.mean(ref ** 2))


def test_config2_llama3_8b_gqa_layer_full(H):
    c = CONFIGS["c2"]
    case = H.AttnCase(501, c.batch, c.n_nodes, c.n_q_heads, c.n_kv_heads, c.head_dim, c.kv_len, "bf16",
                      depth=c.tree_depth, topk=c.tree_topk)
    _check(H, case, H.TOL["bf16"])


def test_config3_one_layer_four_sequences_sampled_heads(H):
    """One layer of the Vicuna-33B-shaped stack at full size (B=4, 52 heads, L=4096, N=60), in the
    launch configuration the benchmark uses; the oracle checks all rows of 6 sampled heads."""
    c = CONFIGS["c3"]
    case = H.AttnCase(502, c.batch, c.n_nodes, c.n_q_heads, c.n_kv_heads, c.head_dim, c.kv_len, "bf16",
                      depth=c.tree_depth, topk=c.tree_topk)
    out = case.run_gpu()
    heads = [0, 7, 19, 33, 44, 51]
    ref = case.run_oracle(heads=heads)
    assert H.rel_err(out[:, :, heads], ref) <= H.TOL["bf16"]
    assert torch.isfinite(out).all()


@pytest.mark.parametrize("N,D,Hkv,kv_len", [
    (9, 128, 16, [8300] * 4), (26, 128, 16, [8300] * 4), (26, 128, 100, [1340] * 4), (40, 128, 16, [8300] * 4),
    (60, 64, 32, [8300] * 4), (26, 64, 32, [8300] * 4), (40, 64, 100, [2700] * 4), (9, 64, 32, [8300] * 4),
    (9, 128, 16, [16400, 3000, 14001, 2]), (26, 128, 16, [16400, 3000, 14001, 2]), (40, 128, 16, [16400, 3000, 14001, 2]),
    (60, 128, 16, [16400, 3000, 14001, 2]), (26, 64, 32, [16400, 3000, 14001, 2]), (60, 64, 32, [16400, 3000, 14001, 2])])
def test_keys_and_values_beyond_the_memory_side_cache(H, N, D, Hkv, kv_len):
    """More than 256 MB of keys and values in a call: the forms that read them with the non-temporal hint, for every row
    tile, of equally long and of ragged batches, and of whole units beyond the compute units. All kv heads share the
    keys and values of one (a head stride of zero), which the oracle sees for three of them."""
    import oracle
    B, L = 4, max(kv_len)
    assert sum(-(-x // 32) + -(-N // 32) for x in kv_len) * Hkv * 32 * D * 4 > 256 << 20
    case = H.AttnCase(510 + N + D, B, N, Hkv, Hkv, D, 1, "bf16", kv_len=[0] * B, n_nodes=[N, N, (N - 1) // 32 * 32 + 1, N], topk=4)
    rng = np.random.default_rng(N + D)
    kc, vc = [H.to_dev(rng.standard_normal((B, 1, L, D), dtype=np.float32), "bf16") for _ in range(2)]
    case.k_cache, case.v_cache, case.kv_len = kc.expand(B, Hkv, L, D), vc.expand(B, Hkv, L, D), np.asarray(kv_len, np.int32)
    assert case.k_cache.stride(1) == 0
    out = case.run_gpu()
    assert torch.isfinite(out).all()
    heads, h = [0, Hkv // 2, Hkv - 1], case.host
    kc3, vc3 = [np.repeat(t.float().cpu().numpy(), 3, axis=1) for t in (kc, vc)]
    ref = oracle.tree_attn(h["q"][:, :, heads], h["k_tree"][:, :, heads], h["v_tree"][:, :, heads], kc3, vc3, case.kv_len,
                           case.n_nodes, case.parent, packed_mask=case.mask, nthreads=16)
    assert H.rel_err(out[:, :, heads], ref) <= H.TOL["bf16"]


def test_config4_one_layer_long_context_sampled_heads(H):
    """One layer of the LLaMA3-70B-shaped stack (64/8 GQA, L=16384, N=60); oracle on 4 sampled heads."""
    c = CONFIGS["c4"]
    case = H.AttnCase(503, c.batch, c.n_nodes, c.n_q_heads, c.n_kv_heads, c.head_dim, c.kv_len, "bf16",
                      depth=c.tree_depth, topk=c.tree_topk)
    out = case.run_gpu()
    heads = [0, 13, 38, 63]
    ref = case.run_oracle(heads=heads)
    assert H.rel_err(out[:, :, heads], ref) <= H.TOL["bf16"]
    assert torch.isfinite(out).all()


def test_very_long_prefix(H):
    """150 000 prefix keys of one kv head under two query heads (4 689 blocks per unit, cut over every
    compute unit): the flat block arithmetic and the merge at the far end of their ranges."""
    case = H.AttnCase(505, 1, 64, 2, 1, 128, 150_000, "bf16")
    _check(H, case, H.TOL["bf16"])


def test_token_stride_of_two_megabytes(H):
    """A cache whose tokens lie 2^20 elements apart (the largest strides the descriptor accepts are of
    that order): byte offsets inside one sequence pass 4 GB, so every address has to be formed in 64
    bits. The keys and values themselves are the usual ones, viewed through the wide stride."""
    L, stride = 2100, 1 << 20
    case = H.AttnCase(506, 1, 40, 4, 2, 128, L, "bf16")
    wide = []
    for t in (case.k_cache, case.v_cache):          # [1, 2, L, 128] contiguous
        buf = torch.empty((2 * L * stride,), dtype=torch.bfloat16, device=H.DEV)
        view = buf.as_strided((1, 2, L, 128), (2 * L * stride, L * stride, stride, 1))
        view.copy_(t)
        wide.append(view)
    case.k_cache, case.v_cache = wide
    assert case.k_cache.stride(2) == stride and (L - 1) * stride * 2 > 4 * 2 ** 30
    _check(H, case, H.TOL["bf16"])
    del wide, case
    torch.cuda.empty_cache()


def test_missing_workspace_is_an_error_not_a_crash(H):
    import paper_2408_15562_amd as fspad
    case = H.AttnCase(504, 1, 26, 32, 32, 128, 2048, "bf16")
    tiny = torch.empty(16, dtype=torch.uint8, device=H.DEV)
    with pytest.raises(fspad.FspadError) as e:
        fspad.fspad_tree_attn(case.q, case.k_tree, case.v_tree, case.k_cache, case.v_cache, case.kv_len,
                              case.n_nodes, case.mask_dev, workspace=tiny)
    assert e.value.status == 5


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,Hq,Hkv", [(3, 4, 2), (26, 16, 16), (61, 16, 4)])
@pytest.mark.parametrize("L", [0, 7, 8, 9, 16, 17, 31, 32, 33, 64, 65, 255, 257, 700])
def test_fp32_nodes_per_workgroup(H, D, N, Hq, Hkv, L):
    """One and two nodes per workgroup (by heads x nodes), at the edges of the wavefronts' key tiles
    (16 or 32 keys, eight wavefronts; sixteen where few rows would take a second turn) and of the form of one wavefront (up to 8 or 16 keys, with more than 768 rows up
    to 32 or 64), with ragged trees. Tree rows that a node does not see may hold
    anything: the rows past n_nodes are NaN here."""
    case = H.AttnCase(900 + N + L, 2, N, Hq, Hkv, D, L, "f32", l_cap=L + 2, kv_len=[L, L // 2], n_nodes=[N, max(1, N // 2)])
    for t in (case.k_tree, case.v_tree):
        t[1, max(1, N // 2):] = float("nan")
    _check(H, case, H.TOL["f32"])


@pytest.mark.parametrize("Hq,Hkv,D", [(8, 2, 128), (16, 2, 64), (28, 4, 128)])
@pytest.mark.parametrize("N,n_nodes", [(60, [60, 5, 33, 17]), (64, [1, 16, 64, 32]), (48, [12, 12, 12, 12])])
@pytest.mark.parametrize("splits", [0, 3, 37])
def test_bf16_trees_smaller_than_the_largest(H, Hq, Hkv, D, N, n_nodes, splits):
    """Shared-stage kernel, trees of different sizes: a sequence has only the slab groups that its own tree
    fills, whole or cut; the output rows past them come out as zeros whatever was there."""
    case = H.AttnCase(800 + N + Hq, 4, N, Hq, Hkv, D, 300, "bf16", kv_len=[300, 40, 1, 213], n_nodes=n_nodes)
    _check(H, case, H.TOL["bf16"], **({"splits": splits} if splits else {}))
    ref = case.run_gpu()
    import paper_2408_15562_amd as fspad
    out = torch.full(case.q.shape, float("nan"), dtype=torch.bfloat16, device=H.DEV)
    fspad.fspad_tree_attn(case.q, case.k_tree, case.v_tree, case.k_cache, case.v_cache, case.kv_len, case.n_nodes, case.mask_dev,
                          out=out)
    assert torch.equal(out, ref.to(torch.bfloat16))


@pytest.mark.parametrize("Hq,Hkv,D", [(64, 8, 128), (12, 2, 64), (106, 53, 64)])
@pytest.mark.parametrize("N,n_nodes", [(26, [26, 11, 16, 23]), (32, [3, 32, 1, 9]), (64, [3, 3, 5, 2])])
@pytest.mark.parametrize("L", [0, 26, 300])
def test_bf16_units_equally_long_in_trees_of_different_sizes(H, Hq, Hkv, D, N, n_nodes, L):
    """Sequences of equally many key blocks whose trees fill different numbers of slab groups: units stay aligned with the
    workgroups (whole, or the same number of pieces each, also where full trees would have had fewer workgroups)."""
    kv_len = [L, max(0, L - 5), max(0, L - 9), max(0, L - 11)]
    case = H.AttnCase(850 + N + L, 4, N, Hq, Hkv, D, L, "bf16", kv_len=kv_len, n_nodes=n_nodes, l_cap=L + 1)
    _check(H, case, H.TOL["bf16"])


@pytest.mark.parametrize("B,Hkv,G,N,L", [(4, 40, 1, 5, 130), (4, 52, 1, 26, 33), (2, 40, 1, 40, 700), (2, 52, 1, 9, 1100),
                                         (2, 32, 1, 60, 300), (3, 8, 4, 40, 900), (5, 8, 1, 3, 64), (4, 39, 1, 4, 500),
                                         (13, 40, 1, 26, 70), (3, 40, 1, 60, 476), (2, 60, 1, 10, 600), (1, 64, 1, 26, 500),
                                         (4, 8, 4, 60, 220)])
def test_bf16_workgroups_aligned_with_units(H, B, Hkv, G, N, L):
    """Equally long units whose number does not divide the compute units: whole units on part of the chip,
    two or three pieces of each, short units kept whole (the last four: of 4 to 5 blocks per wavefront), (4 x 39,
    500 keys) just below the border, and (13 x 40) two workgroups per compute unit over more units than that."""
    case = H.AttnCase(700 + Hkv + N, B, N, Hkv * G, Hkv, 64, L, "bf16", n_nodes=[N] * B)
    _check(H, case, H.TOL["bf16"])


# Equal units in pieces: grouped heads of both head dims, one and two slabs a workgroup, 16-row tiles, 2, up to 8 and more pieces, trees of
# different sizes in equally many blocks.
@pytest.mark.parametrize("B,Hq,Hkv,N,D,L,n_nodes", [
    (3, 28, 4, 26, 128, 161, None), (1, 12, 2, 48, 128, 1500, None), (1, 12, 2, 48, 128, 5000, None), (2, 64, 8, 33, 128, 100, [33, 64 - 31]),
    (1, 12, 2, 60, 64, 91, None), (2, 28, 4, 40, 64, 1460, [40, 33]), (1, 16, 16, 26, 128, 700, None), (1, 32, 32, 8, 128, 700, None),
    (1, 8, 8, 26, 64, 700, None), (1, 8, 8, 60, 64, 288, None), (1, 28, 4, 10, 128, 3000, None), (2, 12, 2, 16, 128, 450, [16, 1])])
def test_bf16_equal_units_in_pieces(H, B, Hq, Hkv, N, D, L, n_nodes):
    case = H.AttnCase(B + Hq + N + L, B, N, Hq, Hkv, D, L, "bf16", n_nodes=None if n_nodes is None else np.array(n_nodes, np.int32))
    _check(H, case, H.TOL["bf16"])


@pytest.mark.parametrize("B,Hq,Hkv,N,D,L,workgroups", [
    (1, 32, 32, 26, 128, 2048, 256), (1, 32, 32, 4, 128, 2048, 256), (1, 32, 8, 60, 128, 4096, 256), (4, 32, 8, 60, 128, 330, 256),
    (8, 16, 16, 10, 64, 1200, 512), (2, 12, 2, 1, 128, 5030, 80), (1, 16, 16, 4, 128, 8300, 512), (2, 64, 8, 12, 128, 1188, 160)])
def test_bf16_equal_units_take_all_compute_units(H, B, Hq, Hkv, N, D, L, workgroups):
    """The built-in count is the one that fills the chip. The largest weight of every stream is exact in bf16, so fewer, longer streams are further
    from a 64-bit evaluation (4 to 17 % where the count was halved or the units left whole)."""
    case = H.AttnCase(B + Hq + N + L, B, N, Hq, Hkv, D, L, "bf16", n_nodes=[N] * B)
    assert torch.equal(case.run_gpu(), case.run_gpu(splits=workgroups))


@pytest.mark.parametrize("B,Hkv,G,N,D", [(8, 48, 1, 17, 128), (2, 200, 1, 32, 128), (8, 50, 2, 13, 128), (3, 128, 1, 33, 64),
                                         (10, 40, 3, 16, 64)])
@pytest.mark.parametrize("L", [0, 33, 300])
def test_bf16_more_whole_units_than_compute_units(H, B, Hkv, G, N, D, L):
    """32- and 48-row tiles, one whole unit per workgroup and two workgroups on a compute unit: trees of different
    sizes (of equally many blocks), both output types.

    The error of an output is at most 2^-8 of the weighted mean of |V| it is formed from (every weight is rounded to
    bf16, 2^-9, and the sum runs over the rounded ones). Among the 10^6 outputs of these cases are rows that few keys
    dominate, of ten times the RMS: each is held to the bar relative to its own value, where that is larger than the RMS."""
    n_nodes = [(N - 1) // 32 * 32 + 1 if b % 2 else N for b in range(B)]
    case = H.AttnCase(650 + B + N + L, B, N, Hkv * G, Hkv, D, L, "bf16", n_nodes=n_nodes, topk=4)
    out, ref = case.run_gpu(), case.run_oracle()
    got = out.double().cpu().numpy()
    for b in range(B):
        rms = np.sqrt(np.mean(ref[b, :n_nodes[b]] ** 2))
        assert np.all(np.abs(got[b] - ref[b]) <= H.TOL["bf16"] * np.maximum(rms, np.abs(ref[b])))
        assert np.sqrt(np.mean((got[b] - ref[b]) ** 2)) <= 2.0 ** -8 * rms
        assert np.all(got[b, n_nodes[b]:] == 0)
    assert torch.equal(case.run_gpu(out_dtype=torch.bfloat16), out.to(torch.bfloat16))


@pytest.mark.parametrize("Hq,Hkv,N,D", [(4, 4, 60, 128), (4, 4, 26, 64), (4, 4, 9, 128), (16, 2, 40, 128), (28, 4, 33, 64)])
@pytest.mark.parametrize("kv_len", [[2000, 0, 1, 33, 700, 5], [0, 31, 32, 0, 64, 1500], [3, 2, 1, 0, 0, 90]])
@pytest.mark.parametrize("splits", [0, 5, 40, 4096])
def test_bf16_ragged_batches_count_set_up(H, Hq, Hkv, N, D, kv_len, splits):
    """Long and very short sequences in one batch: units count for more than their blocks in the flat split, so that
    cuts fall inside a unit's set-up, workgroups get nothing but set-up, and units are cut anywhere."""
    case = H.AttnCase(600 + N + len(kv_len), 6, N, Hq, Hkv, D, max(kv_len), "bf16", kv_len=kv_len,
                      n_nodes=[N, 1, max(1, N // 2), N, 3, max(1, N // 3)])
    _check(H, case, H.TOL["bf16"], **({"splits": splits} if splits else {}))


@pytest.mark.parametrize("L,splits", [(0, 1), (5, 3), (64, 1), (95, 2), (160, 1), (256, 1), (289, 5), (1000, 1), (1000, 9), (1031, 40)])
@pytest.mark.parametrize("N,Hq,Hkv,scale", [(33, 4, 1, 0.0), (60, 8, 2, 1.0), (17, 8, 1, 0.3)])
@pytest.mark.parametrize("D", [64, 128])
def test_bf16_shared_stage_rings_and_segments(H, D, N, Hq, Hkv, scale, L, splits):
    """Segments of one to sixty blocks, odd and even, one or several to a workgroup: each length wraps the rings of K/V blocks
    (head dim 64: the stages) elsewhere and ends the two (three) key groups differently. Scale 1.0 spreads the scores over tens of powers of two, so that the
    shifts of the softmax keep moving along the stream. A tree smaller than the batch's largest leaves slabs without rows."""
    case = H.AttnCase(77 * N + L + splits, 2, N, Hq, Hkv, D, L, "bf16", l_cap=L + 3, n_nodes=[N, (N + 1) // 2])
    out, _, _ = _check(H, case, H.TOL["bf16"], splits=splits, **({"scale": scale} if scale else {}))
    assert torch.equal(out, case.run_gpu(splits=splits, **({"scale": scale} if scale else {})))


@pytest.mark.parametrize("blocks", range(13))
@pytest.mark.parametrize("N", [35, 64])
def test_bf16_shared_stage_first_and_last_blocks(H, N, blocks):
    """One workgroup per unit, so that a key group holds none to seven blocks: fewer than its ring, as many, more; the tree in one
    block or two and both halves of the ancestor words. The smaller tree leaves query rows past its end in a slab, and slabs without any."""
    case = H.AttnCase(900 + N + blocks, 2, N, 8, 2, 128, 32 * blocks, "bf16", n_nodes=[N, 19])
    _check(H, case, H.TOL["bf16"], splits=4)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,N,Hq,Hkv,lens,nodes", [
    (3, 60, 8, 2, (400, 90, 777), (60, 17, 33)),             # two classes of sequences, cut units
    (5, 64, 12, 1, (500, 3, 90, 301, 33), (64, 5, 22, 43, 11)),   # groups of 1 to 6: more than a launch has classes
    (9, 33, 32, 8, (90, 3, 40, 66, 0, 31, 64, 5, 77), (33, 9, 20, 33, 1, 16, 17, 30, 25)),   # short units, whole
    (40, 40, 8, 2, tuple(7 * i % 83 for i in range(40)), tuple(1 + 11 * i % 40 for i in range(40))),
    (4, 60, 8, 1, (2100, 1900, 2050, 2000), (60, 60, 60, 60)),   # four slab groups, equal classes
])
def test_bf16_shared_stage_classes(H, D, B, N, Hq, Hkv, lens, nodes):
    """Ragged batches of grouped heads: sequences whose trees fill different numbers of slab groups are planned in classes, short
    units stay whole; every output row is written either way, rows of unused nodes as zeros, at any number of workgroups
    (outputs and workspace are NaN before each call)."""
    case = H.AttnCase(900 + B + N + D, B, N, Hq, Hkv, D, max(lens), "bf16", l_cap=max(lens) + 2, kv_len=list(lens), n_nodes=list(nodes), topk=4)
    # The weights are rounded to bf16 (2^-9 of each) in numerator and sum alike: an output is off by at most 2^-9 (sum of
    # p |v| + |output|), under 2^-8 times the same attention over |v|; the rest is fp32. (A bar in terms of the whole batch's
    # RMS does not fit sequences of 3 and of 500 keys side by side: their outputs differ in size by a factor of ten.)
    import oracle
    h = case.host
    ref = case.run_oracle()
    bound = 1.05 * 2.0 ** -8 * oracle.tree_attn(h["q"], h["k_tree"], np.abs(h["v_tree"]), h["k_cache"], np.abs(h["v_cache"]), case.kv_len,
                                                case.n_nodes, case.parent, packed_mask=case.mask, nthreads=16) + 1e-5
    for splits in (0, 1, 5, 37):
        out = case.run_gpu(splits=splits)
        assert np.all(np.abs(out.double().cpu().numpy() - ref) <= bound), f"workgroups {splits}"
        for b, n in enumerate(case.n_nodes):
            assert torch.all(out[b, int(n):] == 0)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,Hq,Hkv,lens,nodes", [
    (26, 12, 2, (36, 19, 4, 4, 9, 32), (26,) * 6),                  # few units of 2 or 3 blocks
    (31, 16, 1, (219, 27, 100, 64), (31, 31, 9, 20)),               # up to 8 blocks, one to four slab groups
    (44, 12, 2, (91, 11), (44, 44)),
    (30, 16, 2, (287, 1, 150), (30, 30, 30)),                       # 10 blocks: the most that stay whole
    (20, 28, 4, tuple(6 + 2 * i for i in range(24)), (20,) * 24),   # more units than an even split of their blocks has workgroups
])
def test_bf16_short_ragged_units_stay_whole(H, D, N, Hq, Hkv, lens, nodes):
    """Units of up to five blocks per key group, of different lengths, that fit the chip are a workgroup's each: nothing is left
    in the workspace, and every output row is written."""
    import paper_2408_15562_amd as fspad
    case = H.AttnCase(960 + N + D, len(lens), N, Hq, Hkv, D, max(lens), "bf16", l_cap=max(lens) + 1, kv_len=list(lens), n_nodes=list(nodes), topk=4)
    desc = fspad.make_attn_desc(case.q, case.k_tree, case.k_cache)
    ws = torch.full((fspad.fspad_tree_attn_workspace_bytes(desc, max(lens)),), 0xA5, dtype=torch.uint8, device=H.DEV)
    out = torch.full(case.q.shape, float("nan"), dtype=torch.bfloat16, device=H.DEV)
    fspad.fspad_tree_attn(case.q, case.k_tree, case.v_tree, case.k_cache, case.v_cache, case.kv_len, case.n_nodes, case.mask_dev,
                          out=out, workspace=ws)
    assert torch.all(ws == 0xA5)
    ref, _, _ = _check(H, case, H.TOL["bf16"])
    assert torch.equal(out, ref.to(torch.bfloat16))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,Hq,Hkv,L", [(26, 4, 4, 200), (40, 8, 2, 33), (60, 8, 2, 1000)])
def test_bf16_non_finite_query_rows_stay_apart(H, D, N, Hq, Hkv, L):
    """A query row of NaN, or with an infinity, makes its own output NaN and leaves every other row as it is, also those that share
    a wavefront with it (whose softmax shifts move together)."""
    case = H.AttnCase(980 + N + D, 2, N, Hq, Hkv, D, L, "bf16", l_cap=L + 1, n_nodes=[N, N])
    ref = case.run_oracle()
    clean = case.q.clone()
    bad = torch.zeros(clean.shape[:3], dtype=torch.bool, device=H.DEV)
    case.q[0, 3, 1] = float("nan")
    case.q[0, 7, Hq - 1, 5] = float("inf")
    case.q[1, N - 1, 0, D - 1] = float("-inf")
    bad[0, 3, 1] = bad[0, 7, Hq - 1] = bad[1, N - 1, 0] = True
    spoilt = case.q
    for splits in (0, 1, 5):
        case.q = spoilt
        out = case.run_gpu(splits=splits)
        case.q = clean
        assert torch.all(torch.isnan(out[bad]))
        assert H.rel_err(torch.where(bad[..., None], case.run_gpu(splits=splits), out), ref) <= H.TOL["bf16"]
