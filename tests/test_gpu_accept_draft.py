"""GPU parity of fspad_tree_accept_sample_draft (acceptance for sampled drafts) against the CPU
oracle, through the C ABI.

Bar: path, lengths and emitted tokens bit-exact. Both sides decide in fp64 but sum in different
orders: a sequence whose closest decision sits within 1e-9 of its threshold is not compared
(such sequences must be rare)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from workloads import gen_logits, gen_sampled_drafts, gen_trees, gen_uniforms  # noqa: E402

DEV = "cuda:0"
MARGIN = 1e-9


def _case(seed, B, N, V, T, peak=0.0, noise=1.0, n_nodes=None, row_pad=0, depth=6, topk=10):
    topk = min(topk, max(1, N - 1))
    parent, n_nodes = gen_trees(seed, B, N, depth, topk, n_nodes=n_nodes)
    logits = gen_logits(seed, B, N, V, peak=peak)
    draft_logits, tokens = gen_sampled_drafts(seed, logits, parent, n_nodes, T, noise)
    return parent, n_nodes, logits, draft_logits, tokens


def _padded(a, pad):
    if not pad:
        return torch.from_numpy(a).to(DEV)
    B, N, V = a.shape
    buf = torch.full((B, N, V + pad), float("nan"), dtype=torch.float32, device=DEV)
    buf[:, :, :V] = torch.from_numpy(a).to(DEV)
    return buf[:, :, :V]


def _run(seed, B, N, V, T, useed=0, min_compared=None, **kw):
    import paper_2408_15562_amd as fspad
    parent, n_nodes, logits, draft_logits, tokens = _case(seed, B, N, V, T, **kw)
    uni = gen_uniforms(useed, B, N)
    pad = kw.get("row_pad", 0)
    # workspace (NaN) and outputs hold what no call leaves there: statistics that nobody formed, or words that nobody wrote, show
    ws = torch.full((fspad.fspad_tree_accept_sample_draft_workspace_bytes(B, N, V),), 0xFF, dtype=torch.uint8, device=DEV)
    out = [torch.full(shape, -77, dtype=torch.int32, device=DEV) for shape in ((B, N), (B,), (B, N), (B,))]
    fspad.fspad_tree_accept_sample_draft(_padded(logits, pad), _padded(draft_logits, pad), torch.from_numpy(tokens).to(DEV),
                                         torch.from_numpy(parent).to(DEV), torch.from_numpy(n_nodes).to(DEV), T,
                                         torch.from_numpy(uni).to(DEV), outputs=out, workspace=ws)
    torch.cuda.synchronize()
    ref = oracle.accept_sample_draft(logits, draft_logits, tokens, parent, n_nodes, T, uni)
    keep = ref[4] >= MARGIN
    assert keep.sum() >= (max(1, B - 1) if min_compared is None else min_compared), ref[4]
    for name, g, c in zip(("path", "path_len", "tokens", "n_tokens"), out, ref[:4]):
        np.testing.assert_array_equal(g.cpu().numpy()[keep], c[keep], err_msg=name)
    return ref


@pytest.mark.parametrize("B,N,V", [(1, 1, 7), (3, 2, 1000), (2, 26, 1000), (1, 26, 32000), (2, 60, 32000),
                                   (1, 64, 8192), (1, 60, 128256), (4, 33, 8193), (2, 17, 1001), (3, 9, 1023)])
@pytest.mark.parametrize("peak,noise", [(0.0, 1.0), (3.0, 0.5)])
@pytest.mark.parametrize("T", [1.0, 0.7])
def test_matches_oracle(B, N, V, peak, noise, T):
    _run(5000 + B + N + V, B, N, V, T, peak=peak, noise=noise)


@pytest.mark.parametrize("B,N,V", [(260, 4, 600), (1, 6, 200000), (1, 5, 300001), (40, 8, 5000), (256, 3, 700)])
def test_both_launch_forms(B, N, V):
    """The library spreads a sequence over several workgroups when the shape allows it and keeps one
    workgroup a sequence otherwise: more sequences than the chip-wide form takes; vocabularies that
    put 16 and 32 entries into a thread; batches that leave a sequence five workgroups, or one."""
    _run(6100 + B + V, B, N, V, 0.9, peak=2.0, noise=0.5, min_compared=B - max(1, B // 40))


@pytest.mark.parametrize("B,N", [(1, 64), (3, 26)])
@pytest.mark.parametrize("V", [20, 40, 51, 53, 60, 93, 120, 137])
def test_smallest_vocabularies(B, N, V):
    """Around the vocabulary from which the exchange area fits in the workspace's rows."""
    _run(6300 + V, B, N, V, 0.9, peak=1.0, noise=0.7, topk=8, min_compared=max(1, B - 1))


def test_small_vocabularies_take_the_form_of_larger_ones():
    """64 nodes: a vocabulary of 120 entries takes no longer than one of 1000, which it does in the general form."""
    import paper_2408_15562_amd as fspad
    N, T, took = 64, 1.0, {}
    for V in (120, 1000):
        parent, n_nodes, logits, draft_logits, tokens = _case(68, 1, N, V, T, peak=2.0)
        parent[:], n_nodes[:], tokens[:] = 0, N, V    # the root rejects 63 children
        parent[:, 0] = -1
        dev = [torch.from_numpy(a).to(DEV) for a in (logits, draft_logits, tokens, parent, n_nodes, gen_uniforms(1, 1, N))]
        out = [torch.empty(shape, dtype=torch.int32, device=DEV) for shape in ((1, N), (1,), (1, N), (1,))]
        ws = torch.empty(fspad.fspad_tree_accept_sample_draft_workspace_bytes(1, N, V), dtype=torch.uint8, device=DEV)
        graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
            for _ in range(20):
                fspad.fspad_tree_accept_sample_draft(*dev[:5], T, dev[5], outputs=out, workspace=ws)
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            took[V] = min(took.get(V, np.inf), a.elapsed_time(b))
    assert took[120] < 1.1 * took[1000], took   # (the general form: 1.22 of it, this one 0.96)


def test_one_workspace_call_after_call():
    """The chip-wide form exchanges its sums through the workspace and has an earlier launch of every
    call set these places to zero: calls that follow one another through one workspace (a larger problem, then a
    smaller one, then the first again) each match the oracle."""
    import paper_2408_15562_amd as fspad
    shapes = [(2, 40, 20000), (1, 12, 3000), (2, 40, 20000)]
    ws = torch.empty(max(fspad.fspad_tree_accept_sample_draft_workspace_bytes(*sh) for sh in shapes), dtype=torch.uint8, device=DEV)
    ws.fill_(0xAB)   # nothing in it is assumed to be zero
    for i, (B, N, V) in enumerate(shapes):
        parent, n_nodes, logits, draft_logits, tokens = _case(6400 + i, B, N, V, 0.8, peak=2.0, noise=0.5)
        uni = gen_uniforms(i, B, N)
        out = fspad.fspad_tree_accept_sample_draft(torch.from_numpy(logits).to(DEV), torch.from_numpy(draft_logits).to(DEV),
                                                   torch.from_numpy(tokens).to(DEV), torch.from_numpy(parent).to(DEV),
                                                   torch.from_numpy(n_nodes).to(DEV), 0.8, torch.from_numpy(uni).to(DEV), workspace=ws)
        torch.cuda.synchronize()
        ref = oracle.accept_sample_draft(logits, draft_logits, tokens, parent, n_nodes, 0.8, uni)
        keep = ref[4] >= MARGIN
        assert keep.sum() >= 1
        for name, g, c in zip(("path", "path_len", "tokens", "n_tokens"), out, ref[:4]):
            np.testing.assert_array_equal(g.cpu().numpy()[keep], c[keep], err_msg=f"call {i}: {name}")


def test_walks_accept_reject_and_draw():
    """A drafter close to a peaked target: accepted chains several levels deep, rejections with
    siblings left (the residual max(p - q, 0) applied more than once at a node), draws at inner
    nodes and at leaves."""
    lens = []
    for useed in range(4):
        ref = _run(77, 32, 40, 3000, 1.0, useed=useed, peak=3.0, noise=0.3, min_compared=30)
        lens += ref[1].tolist()
    assert max(lens) >= 4 and len(set(lens)) >= 3


def test_ragged_trees_and_padded_rows():
    _run(78, 5, 60, 5000, 0.9, peak=2.0, n_nodes=[60, 1, 17, 33, 2], row_pad=4, min_compared=4)


def test_drafter_equal_to_the_target_accepts_whole_chains():
    import paper_2408_15562_amd as fspad
    B, N, V = 3, 12, 2000
    logits = gen_logits(9, B, N, V)
    chain = np.tile(np.arange(-1, N - 1, dtype=np.int32), (B, 1))
    tokens = np.random.default_rng(9).integers(0, V, (B, N)).astype(np.int32)
    uni = gen_uniforms(9, B, N)
    dl = torch.from_numpy(logits).to(DEV)
    out = fspad.fspad_tree_accept_sample_draft(dl, dl.clone(), torch.from_numpy(tokens).to(DEV), torch.from_numpy(chain).to(DEV),
                                               torch.full((B,), N, dtype=torch.int32, device=DEV), 1.0,
                                               torch.from_numpy(uni).to(DEV))
    torch.cuda.synchronize()
    assert out[1].cpu().tolist() == [N] * B
    assert np.array_equal(out[2].cpu().numpy()[:, : N - 1], tokens[:, 1:])


def test_point_mass_drafts_agree_with_the_topk_acceptance_on_gpu():
    """On chains whose draft distribution is a point mass on the drafted token, the call gives what
    fspad_tree_accept_sample gives."""
    import paper_2408_15562_amd as fspad
    B, N, V = 4, 10, 3000
    logits = gen_logits(11, B, N, V, peak=3.0)
    chain = np.tile(np.arange(-1, N - 1, dtype=np.int32), (B, 1))
    nn = torch.full((B,), N, dtype=torch.int32, device=DEV)
    tokens = np.argsort(-logits, axis=2)[:, :, 0].astype(np.int32)          # child c carries its parent's best token
    tokens = np.concatenate([np.zeros((B, 1), np.int32), tokens[:, :-1]], axis=1)
    ql = np.full((B, N, V), -1e30, dtype=np.float32)
    for b in range(B):
        for c in range(1, N):
            ql[b, c - 1, tokens[b, c]] = 0.0
    for useed in range(3):
        uni = torch.from_numpy(gen_uniforms(useed, B, N)).to(DEV)
        args = (torch.from_numpy(tokens).to(DEV), torch.from_numpy(chain).to(DEV), nn, 0.8, uni)
        a = fspad.fspad_tree_accept_sample(torch.from_numpy(logits).to(DEV), *args)
        d = fspad.fspad_tree_accept_sample_draft(torch.from_numpy(logits).to(DEV), torch.from_numpy(ql).to(DEV), *args)
        torch.cuda.synchronize()
        ref = oracle.accept_sample(logits, tokens, chain, np.full(B, N, np.int32), 0.8, uni.cpu().numpy())
        keep = torch.from_numpy(ref[4] >= MARGIN).to(DEV)
        for x, y in zip(a, d):
            assert torch.equal(x[keep], y[keep])


def test_bad_arguments_are_errors():
    import paper_2408_15562_amd as fspad
    B, N, V = 1, 4, 100
    logits = torch.zeros((B, N, V), dtype=torch.float32, device=DEV)
    tok = torch.zeros((B, N), dtype=torch.int32, device=DEV)
    par = torch.tensor([[-1, 0, 0, 1]], dtype=torch.int32, device=DEV)
    nn = torch.tensor([4], dtype=torch.int32, device=DEV)
    uni = torch.zeros((B, 2, N), dtype=torch.float32, device=DEV)
    for t in (0.0, -1.0, float("inf"), float("nan")):
        with pytest.raises(fspad.FspadError):
            fspad.fspad_tree_accept_sample_draft(logits, logits, tok, par, nn, t, uni)
    with pytest.raises(fspad.FspadError):
        fspad.fspad_tree_accept_sample_draft(logits, logits, tok, par, nn, 1.0, uni,
                                             workspace=torch.empty(16, dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()


@pytest.mark.parametrize("draw", range(10))
def test_random_shape(draw):
    """Batch, tree size, vocabulary, temperature, drafter noise and target peakedness at random."""
    rng = np.random.default_rng([616, draw])
    B = int(rng.integers(1, 7))
    N = int(rng.integers(1, 65))
    V = int(rng.choice([3, 64, 65, 1000, 4097, 20000, 50257]))
    T = float(rng.choice([0.5, 1.0, 1.7]))
    n_nodes = [int(rng.integers(1, N + 1)) for _ in range(B)]
    _run(6000 + draw, B, N, V, T, useed=draw, peak=float(rng.choice([0.0, 2.0, 4.0])), noise=float(rng.choice([0.2, 1.0, 3.0])),
         n_nodes=n_nodes, row_pad=int(rng.choice([0, 0, 4])), depth=8, topk=int(rng.integers(3, 11)), min_compared=max(1, B - 1))


@pytest.mark.parametrize("B,V", [(2, 60000), (1, 128256), (6, 128256), (260, 600)])
def test_plus_infinity_leaves_a_row_without_mass(B, V):
    """A logit of +infinity leaves no entry of its row with mass, whichever workgroup holds it: token 0 comes out, as the oracle
    says, of a leaf's row and of an inner row whose child is rejected, in every form of the call."""
    import paper_2408_15562_amd as fspad
    N = 3
    rng = np.random.default_rng(V)
    for at in (0, V // 2, V - 1):
        logits = rng.normal(0, 2, (B, N, V)).astype(np.float32)
        draft_logits = rng.normal(0, 2, (B, N, V)).astype(np.float32)
        logits[:, :, at] = np.inf
        parent = np.tile(np.array([-1, 0, 0], np.int32), (B, 1))
        n_nodes = np.where(np.arange(B) % 2, 3, 1).astype(np.int32)     # roots alone, and roots with two children
        tokens = rng.integers(1, V - 1, (B, N)).astype(np.int32)
        uni = gen_uniforms(at, B, N)
        out = fspad.fspad_tree_accept_sample_draft(*(torch.from_numpy(a).to(DEV) for a in (logits, draft_logits, tokens, parent, n_nodes)),
                                                   0.9, torch.from_numpy(uni).to(DEV))
        torch.cuda.synchronize()
        with np.errstate(invalid="ignore"):
            ref = oracle.accept_sample_draft(logits[:2], draft_logits[:2], tokens[:2], parent[:2], n_nodes[:2], 0.9, uni[:2])
        assert (ref[2][:, 0] == 0).all() and (ref[1] == 1).all()
        assert (out[1].cpu().numpy() == 1).all() and (out[2].cpu().numpy()[:, 0] == 0).all()


@pytest.mark.parametrize("B,N,V,pad", [(6, 20, 1025, 0), (6, 20, 33001, 1), (2, 26, 128256, 0), (260, 4, 600, 0), (3, 9, 90, 3)])
@pytest.mark.parametrize("T", [1.0, 0.7])
def test_rows_with_nan_and_infinity(B, N, V, pad, T):
    """NaNs of both kinds and -infinity among the target's and the draft's entries (not at the children's tokens, which were drawn), in all of a
    wavefront's and of a chunk's, draft rows of leaves all NaN (nobody asks for them); roots whose target row is nothing but NaN or -infinity,
    which reject their children and give token 0, compared whatever the oracle's margin."""
    import paper_2408_15562_amd as fspad
    parent, n_nodes, logits, draft_logits, tokens = _case(7300 + V, B, N, V, T, peak=2.0, noise=0.5)
    rng = np.random.default_rng(V)
    own = np.zeros((B, N, V), bool)
    b, c = np.nonzero(parent >= 0)
    own[b, parent[b, c], tokens[b, c]] = True
    for x in (logits, draft_logits):
        hit = rng.random((B, N, V), dtype=np.float32)
        x[(hit < 0.05) & ~own] = np.nan
        x.view(np.uint32)[(hit > 0.05) & (hit < 0.08) & ~own] = 0x7fa00001
        x[(hit > 0.08) & (hit < 0.2) & ~own] = -np.inf
        part = np.zeros((B, N, V), bool)
        part[:, ::3, 256:512] = True
        part[:, 1::3, 1024:min(10240, V // 2)] = True
        x[part & ~own] = (np.nan, -np.inf)[x is logits]
    leaf = np.ones((B, N), bool)
    leaf[b, parent[b, c]] = False
    draft_logits[leaf] = np.nan
    nothing = np.arange(B) % 3 < 2 if B > 2 else np.arange(B) < 1
    for i in np.nonzero(nothing)[0]:
        logits[i, 0] = (np.nan, -np.inf)[i % 2]
    uni = gen_uniforms(5, B, N)
    out = fspad.fspad_tree_accept_sample_draft(_padded(logits, pad), _padded(draft_logits, pad), *(torch.from_numpy(a).to(DEV) for a in (tokens, parent, n_nodes)),
                                               T, torch.from_numpy(uni).to(DEV))
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        ref = oracle.accept_sample_draft(logits, draft_logits, tokens, parent, n_nodes, T, uni)
    assert (ref[1][nothing] == 1).all() and (ref[2][nothing, 0] == 0).all()
    keep = ref[4] >= MARGIN
    assert keep[~nothing].sum() >= max(1, (~nothing).sum() - 1)
    keep[nothing] = True
    for name, g, r in zip(("path", "path_len", "tokens", "n_tokens"), out, ref[:4]):
        np.testing.assert_array_equal(g.cpu().numpy()[keep], r[keep], err_msg=name)


def test_captured_call_replays_like_eager():
    import paper_2408_15562_amd as fspad
    B, N, V, T = 3, 30, 5000, 1.0
    parent, n_nodes, logits, draft_logits, tokens = _case(91, B, N, V, T, peak=2.0, noise=0.5)
    dev = [torch.from_numpy(a).to(DEV) for a in (logits, draft_logits, tokens, parent, n_nodes, gen_uniforms(1, B, N))]
    outs = tuple(torch.empty(s, dtype=torch.int32, device=DEV) for s in ((B, N), (B,), (B, N), (B,)))
    ws = torch.empty(fspad.fspad_tree_accept_sample_draft_workspace_bytes(B, N, V), dtype=torch.uint8, device=DEV)

    def step():
        fspad.fspad_tree_accept_sample_draft(dev[0], dev[1], dev[2], dev[3], dev[4], T, dev[5], outputs=outs, workspace=ws)

    def snapshot():
        torch.cuda.synchronize()
        return [t.clone() for t in outs]

    def scrub():
        for t in outs:
            t.fill_(-9)
        ws.random_()
        torch.cuda.synchronize()

    step()
    eager = snapshot()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        scrub()
        with torch.cuda.graph(graph, stream=side):
            step()
    for _ in range(3):
        scrub()
        graph.replay()
        for a, b in zip(eager, snapshot()):
            assert torch.equal(a, b)


@pytest.fixture(scope="module")
def late_call():
    """The same entry point of the build whose chip-wide walks have late workgroups: from the late_from-th of every sequence on they
    count themselves in when the others have gone on, or late_us after their start."""
    import ctypes

    from paper_2408_15562_amd import build
    lib = ctypes.CDLL(build.build_late(force=False))
    f = lib.fspad_tree_accept_sample_draft
    vp = ctypes.c_void_p
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int32] * 3 + [vp, vp, ctypes.c_int64] + [vp] * 3 + [ctypes.c_float] + [vp] * 6 + [ctypes.c_size_t, vp]

    def call(late_from, late_us, B, N, V, T, dev, outputs, workspace):
        ctypes.c_int32.in_dll(lib, "fspad_test_late_from").value = late_from
        ctypes.c_int64.in_dll(lib, "fspad_test_late_ticks").value = int(100 * late_us)
        logits, draft_logits, tokens, parent, n_nodes, uni = dev
        return f(B, N, V, logits.data_ptr(), draft_logits.data_ptr(), logits.stride(1), tokens.data_ptr(), parent.data_ptr(),
                 n_nodes.data_ptr(), T, uni.data_ptr(), *(t.data_ptr() for t in outputs), workspace.data_ptr(), workspace.numel(),
                 torch.cuda.current_stream().cuda_stream)
    return call


def _late_case(seed, B, N, V, T, noise, pad=0, wide=False):
    """Inputs on the device, outputs of the full walk, and a workspace of NaN."""
    import paper_2408_15562_amd as fspad
    parent, n_nodes, logits, draft_logits, tokens = _case(seed, B, N, V, T, peak=2.0, noise=noise)
    if wide:   # every node a child of the root, and none of them accepted
        parent, n_nodes = np.zeros((B, N), np.int32), np.full(B, N, np.int32)
        parent[:, 0] = -1
        tokens[:, 1::2] = V
        tokens[:, 2::2] = draft_logits[:, 0].argmax(1)[:, None]
        logits[np.arange(B), 0, tokens[:, 2]] = -20.0
    uni = gen_uniforms(3, B, N)
    dev = [_padded(logits, pad), _padded(draft_logits, pad)] + [torch.from_numpy(a).to(DEV) for a in (tokens, parent, n_nodes, uni)]
    full = fspad.fspad_tree_accept_sample_draft(*dev[:5], T, dev[5])
    ws = torch.full((fspad.fspad_tree_accept_sample_draft_workspace_bytes(B, N, V),), 0xFF, dtype=torch.uint8, device=DEV)
    return dev, full, ws, oracle.accept_sample_draft(logits, draft_logits, tokens, parent, n_nodes, T, uni)


@pytest.mark.parametrize("B,N,V,pad", [(1, 26, 2000, 0), (2, 40, 20000, 4), (1, 60, 128256, 0), (3, 30, 50257, 1), (40, 8, 5000, 0),
                                       (5, 20, 128256, 0), (1, 12, 300001, 0), (2, 1, 4097, 0)])
@pytest.mark.parametrize("noise", [0.3, 1.0])
@pytest.mark.parametrize("there", [1, 2, 3, 7, 62])
def test_walk_by_the_workgroups_that_are_there(late_call, B, N, V, pad, noise, there):
    """Shares of 4, 8, 16 and 32 entries per thread, rows of any alignment, one workgroup or several that take all shares: the outputs
    of the full walk (the same arithmetic) and of the oracle. Who comes late finds the count closed and touches nothing.
    A second call through the same workspace does the same."""
    T = 0.9
    dev, full, ws, ref = _late_case(8100 + B + N + V, B, N, V, T, noise, pad)
    keep = ref[4] >= MARGIN
    assert keep.sum() >= max(1, B - 1)
    for _ in range(2):
        out = [torch.full(shape, -77, dtype=torch.int32, device=DEV) for shape in ((B, N), (B,), (B, N), (B,))]
        assert late_call(there, 50e3, B, N, V, T, dev, out, ws) == 0
        torch.cuda.synchronize()
        for name, g, f, c in zip(("path", "path_len", "tokens", "n_tokens"), out, full, ref[:4]):
            assert torch.equal(g, f), name
            np.testing.assert_array_equal(g.cpu().numpy()[keep], c[keep], err_msg=name)


@pytest.mark.parametrize("B,N,V", [(1, 33, 60000), (2, 20, 300001)])
@pytest.mark.parametrize("there", [1, 5])
def test_many_rejections_by_the_workgroups_that_are_there(late_call, B, N, V, there):
    """More rounds than places to exchange in, on shares whose entries are formed anew in every one."""
    T = 1.0
    dev, full, ws, ref = _late_case(8500 + V, B, N, V, T, 1.0, wide=True)
    assert ref[1].tolist() == [1] * B
    out = [torch.full(shape, -77, dtype=torch.int32, device=DEV) for shape in ((B, N), (B,), (B, N), (B,))]
    assert late_call(there, 50e3, B, N, V, T, dev, out, ws) == 0
    torch.cuda.synchronize()
    for g, f in zip(out, full):
        assert torch.equal(g, f)


def test_workgroups_that_come_as_the_count_is_closed(late_call):
    """Starts from 0 to some 70 us late, the first workgroup's wait (20 us here) among them: whether the count is closed before,
    after or while they come, the outputs are those of the full walk."""
    B, N, V, T = 3, 40, 60000, 0.9
    dev, full, ws, _ = _late_case(8600, B, N, V, T, 0.7)
    for there in (40, 58):
        for late_us in [0, 5, 10] + list(range(15, 45)) + [50, 60, 70]:
            out = [torch.full(shape, -77, dtype=torch.int32, device=DEV) for shape in ((B, N), (B,), (B, N), (B,))]
            assert late_call(there, late_us, B, N, V, T, dev, out, ws) == 0
            torch.cuda.synchronize()
            for g, f in zip(out, full):
                assert torch.equal(g, f), (there, late_us)


def test_a_walk_without_all_of_its_workgroups_is_not_a_walk_alone(late_call):
    """Where a fourth of the workgroups are there, the call takes a small part of what one of them alone takes: all of them go on."""
    B, N, V, T = 1, 33, 128256, 1.0
    dev, full, ws, _ = _late_case(8700, B, N, V, T, 1.0, wide=True)
    out = [torch.full(shape, -77, dtype=torch.int32, device=DEV) for shape in ((B, N), (B,), (B, N), (B,))]
    took = {}
    for there in (1, 16):
        for _ in range(3):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            assert late_call(there, 50e3, B, N, V, T, dev, out, ws) == 0
            b.record()
            torch.cuda.synchronize()
            took[there] = min(took.get(there, np.inf), a.elapsed_time(b))
        for g, f in zip(out, full):
            assert torch.equal(g, f)
    assert took[16] < 0.25 * took[1], took   # (63 shares: 4 of them at most instead of 63, and the waits shorter likewise)


def test_calls_on_two_streams_at_once():
    """Calls in flight on two streams, each with a workspace of its own (the chip holds the 236 workgroups of both): the outputs of
    calls that follow one another. (What a walk does without some of its workgroups: the tests with late ones.)"""
    import paper_2408_15562_amd as fspad
    B, N, V, T = 4, 40, 60000, 1.0
    streams, preps, outs = [torch.cuda.Stream() for _ in range(2)], [], []
    for i, stream in enumerate(streams):
        parent, n_nodes, logits, draft_logits, tokens = _case(8300 + i, B, N, V, T, peak=2.0, noise=0.7)
        dev = [torch.from_numpy(a).to(DEV) for a in (logits, draft_logits, tokens, parent, n_nodes, gen_uniforms(i, B, N))]
        alone = fspad.fspad_tree_accept_sample_draft(*dev[:5], T, dev[5])
        out = [torch.full(shape, -77, dtype=torch.int32, device=DEV) for shape in ((B, N), (B,), (B, N), (B,))]
        ws = torch.empty(fspad.fspad_tree_accept_sample_draft_workspace_bytes(B, N, V), dtype=torch.uint8, device=DEV)
        preps.append(fspad.fspad_tree_accept_sample_draft(*dev[:5], T, dev[5], outputs=out, workspace=ws, stream=stream, prepare=True))
        outs.append((out, alone))
    torch.cuda.synchronize()
    for _ in range(20):
        for call in preps:
            call()
    torch.cuda.synchronize()
    for out, alone in outs:
        for a, b in zip(out, alone):
            assert torch.equal(a, b)
