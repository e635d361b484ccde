"""Selection of units of 16385 to 32768 pages, of which only the quads that can hold a selected page are looked at closely: the
result of the size-agnostic kernels at the edges of what the list of quads holds."""
import functools

import numpy as np
import pytest
import torch

from paper_2605_18071_amd import workloads as W
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2605_18071_amd import kvd as K
    from tests import gpu_rig as R


@pytest.mark.parametrize("pages,same,k,kw", [
    (16385, 1, 1, dict()),                                # no ties, one page
    (32768, 1, 1024, dict()),                             # as many pages as are listed this way
    (32768, 1, 1025, dict()),                             # one more
    (32767, 40, 700, dict(sink_pages=3, recent_pages=5)),    # pages no multiple of 4; a short list in the decisive bucket
    (20000, 600, 333, dict(sink_pages=333)),              # forced pages only
    (20000, 600, 333, dict(sink_pages=2, recent_pages=330, dtype="f16")),
    (24576, 2500, 64, dict()),                            # 2500 pages alike: the list of tied pages is too short for them
    (28672, 9000, 500, dict()),                           # more quads alike than are listed
    (29999, 15000, 1000, dict(sink_pages=3, recent_pages=5)),    # two scores
    (30001, 30001, 90, dict()),                           # one score for all
    (25000, 1, 300, dict(values=True)),                   # scores of both infinities and none
    (25000, 1, 300, dict(none=True)),                     # scores that are no numbers
])
def test_equals_the_size_agnostic_kernels(pages, same, k, kw, monkeypatch):
    kw, values, none = dict(kw), kw.get("values"), kw.get("none")
    kw.pop("values", None), kw.pop("none", None)
    w = small("held", **{**dict(ctx=4 * pages, page=4, topk_pages=k, capacity=min(k + 40, pages), batch=2, n_kv_heads=1, n_q_heads=4,
                                heavy_count=0, steps=3), **kw})
    seq = [w.ctx, w.ctx - w.ctx // 5 - 3]                  # the second may be small enough for the other form
    fused = R.Rig(w, seq_lens=seq, build_index=False)
    monkeypatch.setenv("KVD_GENERIC_SELECT", "1")
    plain = R.Rig(w, seq_lens=seq, micro_batches=1, build_index=False)
    gen = torch.Generator(device=R.DEV)
    gen.manual_seed(70_000 + pages + k)
    rows = max(1, pages // same)
    base = torch.randn(w.units, rows, 128, device=R.DEV, generator=gen)
    summ = base[:, torch.randperm(pages, device=R.DEV, generator=gen) % rows].to(w.torch_dtype)
    if values:
        summ[:, 5::700, 0] = float("inf")
    if values or none:
        summ[:, 7::3000, 1] = float("nan")
    for r in (fused, plain):
        r.summaries.copy_(summ.view(r.summaries.shape))
    for t, q in enumerate(W.query_stream(w, fused.q0, w.steps, R.DEV)):
        fused.step(0, t, q[0])
        plain.step(0, t, q[0])
        assert np.array_equal(fused.n_scores, plain.n_scores, equal_nan=True), t
        for what in ("n_sel_pages", "n_hit_mask", "n_sel_slots", "n_counts"):
            assert np.array_equal(getattr(fused, what), getattr(plain, what)), (what, t)
    fused.close()
    plain.close()


@pytest.mark.parametrize("pages,k,kw,at", [
    (20000, 2, dict(), {5000: 3e38, 8000: 2e38, 8001: 2e38, 8002: -2e38, 8003: -2e38}),     # pairs that overflow to both infinities
    (20000, 2, dict(), {5000: 3e38, 8000: -2e38, 8001: -2e38, 8002: 2e38, 8003: 2e38}),
    (20000, 2, dict(), {5000: 3e38, 8000: 2e38, 8001: 2e38, 8002: -np.inf}),                # one pair does, beside a page of minus infinity
    (20000, 4, dict(sink_pages=2), {5000: 3e38, 2: 2e38, 3: 2e38}),                         # ... beside forced pages
    (20000, 4, dict(recent_pages=2), {5000: 3e38, -4: 2e38, -3: 2e38}),
    (20002, 2, dict(), {5000: 3e38, -2: 2e38, -1: 2e38}),                                   # ... at the end of the sequence
    (20000, 40, dict(sink_pages=3), {p: np.inf for p in range(3001, 15000)}),               # more quads than are listed, all in the first bucket
    (32767, 1024, dict(recent_pages=9), {**{p: 2e38 for p in range(5, 9500)}, 9000: 3e38}),  # ... in a later one
    (30000, 700, dict(sink_pages=1), {p: 1e38 + 1e36 * (p % 300) for p in range(1, 30000, 3)}),   # ... of which few are in doubt
    (16385, 3, dict(), {5000: -1e38, 16384: 3e38, 8000: 3e38, 8001: 3.2e38, 8002: -3e38, 8003: -3e38}),   # the range overflows
])
def test_scores_whose_sums_overflow(pages, k, kw, at, monkeypatch):
    """Scores near the largest number: the best k pages in the order of (score, page), as a step's stage and alone."""
    monkeypatch.setattr(K, "Kvd", functools.partial(K.Kvd, softmax_scale=1.0))
    w = small("held-overflow", **{**dict(ctx=4 * pages, page=4, topk_pages=k, capacity=k + 5, batch=1, n_kv_heads=2, n_q_heads=4,
                                         heavy_count=0, steps=1), **kw})
    rig = R.Rig(w, build_index=False)
    gen = np.random.default_rng(pages + k)
    values = torch.from_numpy(gen.random((w.units, pages), dtype=np.float32) * np.float32(9e37)).to(w.torch_dtype)
    for page, v in at.items():
        values[:, page] = float(v)
    rig.summaries.zero_()
    rig.summaries.view(w.units, pages, 128)[:, :, 0] = values.to(R.DEV)
    q = torch.zeros((w.batch, w.n_q_heads, 128), dtype=w.torch_dtype, device=R.DEV)
    q[:, :, 0] = 1.0                                        # a page's score is the first element of its summary
    scores = values.float().numpy()
    want = np.empty((w.units, k), np.int32)
    for u in range(w.units):
        forced = list(range(w.sink_pages)) + list(range(pages - w.recent_pages, pages))
        free = np.arange(w.sink_pages, pages - w.recent_pages)
        best = free[np.lexsort((free, -scores[u, free]))][:k - len(forced)]
        want[u] = np.sort(np.concatenate([np.array(forced, int), best]))
    rig.step(0, 0, q)
    assert np.array_equal(rig.n_scores, scores) and np.array_equal(rig.n_sel_pages, want)
    alone = torch.full((w.units, k), -7, dtype=torch.int32, device=R.DEV)
    rig.kvd.score_select(0, q, alone)
    assert np.array_equal(alone.cpu().numpy(), want)
    rig.close()


@pytest.mark.parametrize("lens", [(9000, 60001), (68000, 40000), (65536, 65537)])
def test_a_captured_selection_of_sequences_that_grow_and_are_cut(lens):
    """The kernel that a capture records is that of the lengths at that time; it selects the same of others."""
    w = small("held-captured", ctx=4 * 17001, page=4, topk_pages=200, capacity=240, batch=2, n_kv_heads=1, n_q_heads=4, heavy_count=0, steps=3)
    rig, eager = R.Rig(w, seq_lens=[lens[0]] * 2), R.Rig(w, seq_lens=[lens[0]] * 2)
    q = torch.zeros((w.batch, w.n_q_heads, 128), dtype=w.torch_dtype, device=R.DEV)
    s = torch.cuda.Stream()
    rig.kvd.score_select(0, q, rig.sel_pages, rig.scores, stream=s)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        rig.kvd.score_select(0, q, rig.sel_pages, rig.scores, stream=s)
    for t, query in enumerate(W.query_stream(w, rig.q0, w.steps, R.DEV)):
        for n in (lens[0], lens[1], lens):
            n = list(n) if isinstance(n, tuple) else [n, n]
            for r in (rig, eager):
                r.kvd.set_seq_lens(n)
            q.copy_(query[0])
            rig.sel_pages.fill_(-7)
            torch.cuda.synchronize()
            graph.replay()
            eager.kvd.score_select(0, query[0], eager.sel_pages, eager.scores)
            torch.cuda.synchronize()
            assert torch.equal(rig.scores, eager.scores) and torch.equal(rig.sel_pages, eager.sel_pages), (t, n)
    rig.close()
    eager.close()


@pytest.mark.parametrize("same,k,kw", [(1, 1024, dict()), (40, 300, dict(sink_pages=2, recent_pages=7)), (9000, 64, dict())])
def test_shorter_sequences_beside_a_long_one(same, k, kw, monkeypatch):
    """Sequences on both sides of the number of pages from which they are selected by quads too."""
    monkeypatch.delenv("KVD_GENERIC_SELECT", raising=False)
    w = small("held-mixed", **{**dict(ctx=4 * 16386, page=4, topk_pages=k, capacity=k + 9, batch=6, n_kv_heads=1, n_q_heads=4, heavy_count=0,
                                      steps=2), **kw})
    seq = [w.ctx, 4 * 12288, 4 * 12288 + 1, 4 * 12289, 4 * 15000 - 1, 4 * 700]
    fused = R.Rig(w, seq_lens=seq, build_index=False)
    monkeypatch.setenv("KVD_GENERIC_SELECT", "1")
    plain = R.Rig(w, seq_lens=seq, micro_batches=1, build_index=False)
    gen = torch.Generator(device=R.DEV)
    gen.manual_seed(same + k)
    rows = max(1, w.n_pages // same)
    base = torch.randn(w.units, rows, 128, device=R.DEV, generator=gen)
    summ = base[:, torch.randperm(w.n_pages, device=R.DEV, generator=gen) % rows].to(w.torch_dtype)
    for r in (fused, plain):
        r.summaries.copy_(summ.view(r.summaries.shape))
    for t, q in enumerate(W.query_stream(w, fused.q0, w.steps, R.DEV)):
        fused.step(0, t, q[0])
        plain.step(0, t, q[0])
        for what in ("n_scores", "n_sel_pages", "n_hit_mask", "n_sel_slots", "n_counts"):
            assert np.array_equal(getattr(fused, what), getattr(plain, what), equal_nan=what == "n_scores"), (what, t)
    fused.close()
    plain.close()
