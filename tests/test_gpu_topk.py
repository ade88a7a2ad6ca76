"""GPU parity of fspad_draft_topk against the CPU oracle, through the C ABI.

Bar: tokens bit-exact (order included; ties to the lower token), log-probabilities within 4e-6
absolute (fp32 exponentials summed in fp64 on the GPU, fp64 throughout in the oracle)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from workloads import gen_logits  # noqa: E402

DEV = "cuda:0"
ATOL = 4e-6


def _run(x, k, **kw):
    import paper_2408_15562_amd as fspad
    tok, lp = fspad.fspad_draft_topk(x, k, **kw)
    torch.cuda.synchronize()
    return tok.cpu().numpy(), lp.cpu().numpy()


def _check(host, k, dev=None):
    tok, lp = _run(torch.from_numpy(host).to(DEV) if dev is None else dev, k)
    r_tok, r_lp = oracle.draft_topk(host, k)
    np.testing.assert_array_equal(tok, r_tok)
    fin = np.isfinite(r_lp)
    np.testing.assert_allclose(lp[fin], r_lp[fin], rtol=0, atol=ATOL)
    assert np.array_equal(np.isneginf(lp), np.isneginf(r_lp))


@pytest.mark.parametrize("rows,V,k", [
    (1, 1, 1), (1, 5, 5), (3, 1000, 4), (4, 1024, 10), (2, 1025, 16), (10, 32000, 10), (40, 32000, 4),
    (1, 32000, 16), (10, 128256, 10), (100, 4099, 10), (700, 777, 3),
])
def test_shapes(rows, V, k):
    """One chunk and many, chunk tails, every chunk size the planner picks, k from 1 to the maximum."""
    x = gen_logits(50 + rows + V, 1, rows, V)[0]
    _check(x, k)


def test_ties_resolve_to_the_lower_token():
    rng = np.random.default_rng(4)
    x = rng.integers(-3, 4, size=(6, 20000)).astype(np.float32)     # seven distinct values: ties everywhere
    x[:, ::7] *= -0.0                                                # zeros of both signs
    _check(x, 16)


def test_nan_and_infinite_entries():
    x = gen_logits(9, 1, 5, 9000)[0]
    x[0, :] = -np.inf                       # nothing finite: tokens 0..k-1, logp -inf
    x[1, 100:8000] = np.nan                 # NaN ranks as -inf and adds nothing to the normaliser
    x[2, :8990] = -np.inf                   # fewer finite entries (10) than k in all chunks but one
    x[3, 5] = np.nan
    _check(x, 12)


def test_strided_and_unaligned_rows():
    host = gen_logits(10, 1, 7, 3001)[0]
    buf = torch.full((7, 3001 + 6), float("nan"), dtype=torch.float32, device=DEV)
    buf[:, 1:3002] = torch.from_numpy(host).to(DEV)
    _check(host, 10, dev=buf[:, 1:3002])    # rows start 4 bytes off a 16-byte boundary


def test_peaked_rows_and_large_values():
    x = gen_logits(11, 1, 8, 32000, peak=12.0)[0]
    x[4] *= 20.0                             # logits in the hundreds: the shift by the maximum matters
    x[5] -= 1000.0
    _check(x, 10)


@pytest.mark.parametrize("V,equal", [(1023, 0), (1024, 17), (1025, 255), (8191, 256), (8192, 257), (20481, 1000), (40, 40)])
def test_entries_at_the_bound(V, equal):
    """The best entries next to each other (sorted rows, both ways) and as many equal ones at the top as a workgroup sets
    aside, one more and one less; whole chunks and chunks that end within a thread's four entries."""
    rng = np.random.default_rng(V)
    x = np.sort(gen_logits(60 + V, 1, 600, V)[0], axis=1)     # (600 rows: the widest chunks)
    x[1::2] = x[1::2, ::-1].copy()
    for row in range(2, 600, 3):
        x[row, rng.permutation(V)[:equal]] = x[row].max() + 1.0
    for part in (x, x[:3]):                                   # (3 rows: the narrowest)
        _check(np.ascontiguousarray(part), 16)


def _masked(rows, V):
    """Rows of a masked vocabulary: none, one, 5, k + 1 finite entries, 300 equal ones at the top, constant rows, half of the vocabulary, and as many large entries
    as a workgroup sets aside, and more, all with threads of one group (neighbours of four, every 128th)."""
    x = gen_logits(70 + V, 1, rows, V)[0]
    rng = np.random.default_rng(V)
    for row in range(rows):
        kind = row % 9
        if kind < 5:
            keep = rng.permutation(V)[:(0, 1, 5, 17, 300)[kind]]
            values = x[row, keep] if kind < 4 else np.float32(2.0)
            x[row] = -np.inf
            x[row, keep] = values
        elif kind == 5:
            x[row] = 0.5
        elif kind == 6:
            x[row, (V + 1) // 2:] = -np.inf
        else:
            x[row, (np.arange(V) // 4) % 32 == 7] += 100.0 if kind == 7 else np.float32(np.inf)
    return x


@pytest.mark.parametrize("rows,V", [(9, 257), (9, 1000), (27, 1025), (9, 8193), (18, 32000), (600, 8192), (9, 128256)])
@pytest.mark.parametrize("k", [1, 10, 16])
def test_masked_vocabularies(rows, V, k):
    """More entries at the bound than a workgroup sets aside: equal ones, which the lower tokens win, and different ones that one group of threads holds."""
    x = _masked(rows, V)
    x[np.isposinf(x)] = 300.0
    _check(x, min(k, V))


def test_masked_vocabularies_take_about_what_ordinary_rows_take():
    """Rows with five finite entries, of which every chunk but a few is nothing but -infinity (one round for each of the k entries: 3.8 times)."""
    import paper_2408_15562_amd as fspad
    rows, V, k = 10, 128256, 16
    x = torch.randn((rows, V), device=DEV)
    masked = torch.full_like(x, -np.inf)
    masked[:, 17::V // 5] = 1.0
    out = torch.empty((rows, k), dtype=torch.int32, device=DEV), torch.empty((rows, k), dtype=torch.float32, device=DEV)
    ws = torch.empty(fspad.fspad_draft_topk_workspace_bytes(rows, V, k), dtype=torch.uint8, device=DEV)
    took = []
    for logits in (x, masked):
        graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
            for _ in range(20):
                fspad.fspad_draft_topk(logits, k, outputs=out, workspace=ws)
        best = np.inf
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        took.append(best)
    assert took[1] < 2.0 * took[0], took


def test_output_feeds_the_tree_build():
    """A draft step on the device: cut each expanded node's output, append the candidates, build."""
    import paper_2408_15562_amd as fspad
    V, k, n_keep = 5000, 4, 12
    x = gen_logits(12, 1, 1 + k, V)[0]                     # outputs at the root and at its k children
    tok, lp = _run(torch.from_numpy(x).to(DEV), k)
    r_tok, r_lp = oracle.draft_topk(x, k)
    m = 1 + k + k * k
    par = np.full((1, m), -1, np.int32)
    par[0, 1:1 + k] = 0
    for j in range(k):
        par[0, 1 + k + j * k:1 + k + (j + 1) * k] = 1 + j

    def cands(t, l):
        return (np.concatenate([[0], t[0], t[1:].reshape(-1)])[None].astype(np.int32),
                np.concatenate([[0.0], l[0], l[1:].reshape(-1)])[None].astype(np.float32))
    g_tok, g_lp = cands(tok, lp)
    o_tok, o_lp = cands(r_tok, r_lp)
    dev = [torch.from_numpy(a).to(DEV) for a in (par, g_tok, g_lp, np.array([m], np.int32))]
    out = fspad.fspad_tree_build(*dev, n_keep, 16)
    torch.cuda.synchronize()
    ref = oracle.tree_build(par, o_tok, o_lp, [m], n_keep, 16)
    # the two candidate sets differ by rounding in logp only; with continuous data the kept set is the same
    assert np.array_equal(out[0].cpu().numpy(), ref[0]) and np.array_equal(out[1].cpu().numpy(), ref[1])


def test_missing_workspace_is_an_error():
    import paper_2408_15562_amd as fspad
    x = torch.zeros((2, 5000), dtype=torch.float32, device=DEV)
    with pytest.raises(fspad.FspadError):
        fspad.fspad_draft_topk(x, 4, workspace=torch.empty(16, dtype=torch.uint8, device=DEV))
