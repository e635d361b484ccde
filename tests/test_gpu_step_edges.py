"""The step's launch forms at the edges of what they hold: selections around the sizes of a wave's registers and with ties that
end in each of the three ways in which the decisive bucket is resolved, several splits per attention workgroup in launches of
several layers, and the merge on both sides of the splits that it fetches at once."""
import numpy as np
import pytest
import torch

from paper_2605_18071_amd import kvd as K
from paper_2605_18071_amd import workloads as W
from tests import helpers as H
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests import gpu_rig as R


@pytest.mark.parametrize("pages,same,k,kw", [
    (2048, 40, 100, dict()),                              # every 2048 / 40 th page has the same score: a short list in the decisive bucket
    (2049, 300, 100, dict(sink_pages=3, recent_pages=5)),
    (2050, 1, 1, dict()),                                 # no ties, one page
    (4096, 1500, 333, dict(sink_pages=1)),                # more candidates than the list holds
    (3001, 32, 20, dict()),                               # lists that a wave ranks by itself and that the threads share
    (3300, 33, 20, dict()),
    (4097, 65, 64, dict(dtype="f16")),
    (8192, 64, 256, dict(recent_pages=2)),
    (8193, 2000, 700, dict()),
    (12001, 1024, 512, dict(sink_pages=7, recent_pages=9, dtype="f16")),
    (16383, 1025, 90, dict()),
    (16384, 300, 2048, dict()),
])
def test_selection_equals_the_size_agnostic_kernels(pages, same, k, kw, monkeypatch):
    w = small("selection-edges", **{**dict(ctx=4 * pages, page=4, topk_pages=k, capacity=min(k + 40, pages), batch=2, n_kv_heads=1,
                                           n_q_heads=4, heavy_count=0, steps=3), **kw})
    seq = [w.ctx, w.ctx - w.ctx // 5 - 3]
    one = R.Rig(w, seq_lens=seq, micro_batches=-1, build_index=False)
    monkeypatch.setenv("KVD_GENERIC_SELECT", "1")
    plain = R.Rig(w, seq_lens=seq, micro_batches=1, build_index=False)
    gen = torch.Generator(device=R.DEV)
    gen.manual_seed(90_000 + pages)
    rows = max(1, pages // same)
    base = torch.randn(w.units, rows, 128, device=R.DEV, generator=gen)
    summ = base[:, torch.randperm(pages, device=R.DEV, generator=gen) % rows].to(w.torch_dtype)
    for r in (one, plain):
        r.summaries.copy_(summ.view(r.summaries.shape))
    assert one.kvd.step_form() == -1
    for t, q in enumerate(W.query_stream(w, one.q0, w.steps, R.DEV)):
        one.step(0, t, q[0])
        plain.step(0, t, q[0])
        for what in ("n_scores", "n_sel_pages", "n_hit_mask", "n_sel_slots", "n_counts"):
            assert np.array_equal(getattr(one, what), getattr(plain, what)), (what, t)
    one.close()
    plain.close()


@pytest.mark.parametrize("mb", [-1, 1], ids=["single-launch", "kernel-chain"])
@pytest.mark.parametrize("pages,pool,same,kw", [
    (300, 30, 1, dict()),
    (512, 511, 1, dict()),                                # all pages but one: the key of the last but one
    (2049, 60, 40, dict(dtype="f16")),                    # ties at the pool's edge
    (4097, 1500, 300, dict(sink_pages=2)),
    (8193, 100, 1, dict()),
    (8200, 3000, 8200, dict()),                           # one score for all: more than the list holds
    (16384, 16383, 2000, dict()),
    (9001, 64, 1, dict(values=True)),                     # scores of both infinities and none
])
def test_pool_of_the_best_pages_equals_the_size_agnostic_kernels(pages, pool, same, kw, mb, monkeypatch):
    kw, values = dict(kw), kw.get("values")
    kw.pop("values", None)
    w = small("pool-edges", **{**dict(ctx=4 * pages, page=4, topk_pages=24, capacity=40, batch=2, n_kv_heads=2, n_q_heads=4,
                                      heavy_count=0, steps=6, policy="lookahead", lookahead_pool=pool, rho=0.2), **kw})
    seq = [w.ctx, w.ctx - 7]
    fused = R.Rig(w, seq_lens=seq, micro_batches=mb, build_index=False)
    monkeypatch.setenv("KVD_GENERIC_SELECT", "1")
    plain = R.Rig(w, seq_lens=seq, micro_batches=1, build_index=False)
    gen = torch.Generator(device=R.DEV)
    gen.manual_seed(91_000 + pages)
    rows = max(1, pages // same)
    base = torch.randn(w.units, rows, 128, device=R.DEV, generator=gen)
    summ = base[:, torch.randperm(pages, device=R.DEV, generator=gen) % rows].to(w.torch_dtype)
    if values:
        summ[:, 5::700, 0] = float("inf")
        summ[:, 7::3000, 1] = float("nan")
    for r in (fused, plain):
        r.summaries.copy_(summ.view(r.summaries.shape))
    evicted = 0
    for t, q in enumerate(W.query_stream(w, fused.q0, w.steps, R.DEV)):
        fused.step(0, t, q[0])
        plain.step(0, t, q[0])
        evicted += fused.n_counts[:, 2]
        assert np.array_equal(fused.n_scores, plain.n_scores, equal_nan=True), t
        for what in ("n_sel_pages", "n_hit_mask", "n_sel_slots", "n_counts"):
            assert np.array_equal(getattr(fused, what), getattr(plain, what)), (what, t)
        assert np.array_equal(np.sort(fused.n_evicted), np.sort(plain.n_evicted)), t
    assert (evicted > 0).all() or same == pages
    fused.close()
    plain.close()


@pytest.mark.parametrize("layers,kw", [
    (8, dict(batch=8, n_kv_heads=4, n_q_heads=32, topk_pages=128)),                       # 8 splits of 16 pages, eight heads
    (6, dict(batch=10, n_kv_heads=4, n_q_heads=4, topk_pages=101)),                       # 5 splits, the last one shorter
    (4, dict(batch=7, n_kv_heads=8, n_q_heads=32, topk_pages=127, dtype="f16")),
    (5, dict(batch=6, n_kv_heads=4, n_q_heads=20, topk_pages=333, page=8, ctx=8 * 500)),  # packed pages, uneven shares of the splits
    (3, dict(batch=3, n_kv_heads=2, n_q_heads=14, topk_pages=43, page=64, ctx=64 * 60)),
    (9, dict(batch=2, n_kv_heads=2, n_q_heads=4, topk_pages=64, page=4, ctx=4 * 8197)),   # 8 layers share a launch, one is left
])
def test_splits_shared_by_the_workgroups_of_several_layers(layers, kw):
    """Outputs bit for bit those of the layers one by one: the splits and the order of their sums are the same."""
    w = small("several-splits", **{**dict(ctx=16 * 200, heavy_count=3, steps=3, n_layers=layers, physical_layers=1,
                                          capacity=kw["topk_pages"] + 10), **kw})
    seq = [w.ctx - 37 * b for b in range(w.batch)]
    one, together = R.Rig(w, seq_lens=seq, micro_batches=-1), R.Rig(w, seq_lens=seq, micro_batches=-1)
    shape = (layers, w.batch, w.n_q_heads, w.head_dim)
    a, b = (torch.empty(shape, dtype=torch.float32, device=R.DEV) for _ in range(2))
    for t, q in enumerate(W.query_stream(w, one.q0, w.steps, R.DEV)):
        b.fill_(float("nan"))
        for l in range(layers):
            one.kvd.step(l, t, q[l], a[l])
        together.kvd.step_layers(0, layers, t, q.contiguous(), b)
        torch.cuda.synchronize()
        assert torch.equal(a, b), t
    for l in range(layers):
        for x, y in zip(one.kvd.cache_export(l), together.kvd.cache_export(l)):
            assert torch.equal(x, y), l
    one.close()
    together.close()


@pytest.mark.parametrize("groups", [1, 3])
@pytest.mark.parametrize("layers,kw", [
    (4, dict(batch=16, n_kv_heads=4, n_q_heads=8, topk_pages=128)),                       # 4 splits, all in one workgroup but for the last layer's
    (4, dict(batch=7, n_kv_heads=4, n_q_heads=8, topk_pages=128)),                        # 8 splits, four to a workgroup
    (5, dict(batch=5, n_kv_heads=4, n_q_heads=8, topk_pages=130, capacity=150, rho=0.3)), # 11 splits; most pages miss
    (6, dict(batch=9, n_kv_heads=4, n_q_heads=28, topk_pages=100, page=8, ctx=8 * 300, dtype="f16")),
])
def test_the_last_layers_splits_have_a_workgroup_each(layers, groups, kw):
    """... while the others' workgroups take three or more, also with the units of a layer in groups, the last of them
    smaller: outputs bit for bit those of the layers one by one."""
    w = small("last-layer", **{**dict(ctx=16 * 200, heavy_count=3, steps=3, n_layers=layers, physical_layers=1,
                                      capacity=kw["topk_pages"] + 10), **kw})
    one, together = R.Rig(w, micro_batches=-1), R.Rig(w, micro_batches=-1)
    together.kvd.set_step_shape(groups=groups, multi_layer=True)
    a, b = (torch.empty((layers, w.batch, w.n_q_heads, w.head_dim), dtype=torch.float32, device=R.DEV) for _ in range(2))
    for t, q in enumerate(W.query_stream(w, one.q0, w.steps, R.DEV)):
        b.fill_(float("nan"))
        for l in range(layers):
            one.kvd.step(l, t, q[l], a[l])
        together.kvd.step_layers(0, layers, t, q.contiguous(), b)
        torch.cuda.synchronize()
        assert torch.equal(a, b), t
    for l in range(layers):
        for x, y in zip(one.kvd.cache_export(l), together.kvd.cache_export(l)):
            assert torch.equal(x, y), l
    one.close()
    together.close()


@pytest.mark.parametrize("mb", [-1, 1], ids=["single-launch", "kernel-chain"])
@pytest.mark.parametrize("splits,kw", [
    (8, dict()),
    (9, dict()),                                          # more than eight: the partials go through LDS
    (16, dict(n_q_heads=2)),
    (17, dict(n_q_heads=16)),
    (31, dict(dtype="f16")),
    (32, dict(page=4, ctx=4 * 600)),
    (33, dict()),
    (64, dict(n_q_heads=14)),
])
def test_merge_of_many_splits_equals_one_split(splits, kw, mb):
    w = small("merge-edges", **{**dict(ctx=16 * 600, topk_pages=257, capacity=300, heavy_count=3, steps=2), **kw})
    many, one = R.Rig(w, micro_batches=mb, attn_splits=splits), R.Rig(w, micro_batches=mb, attn_splits=1)
    assert many.kvd.step_form() == mb
    for t, q in enumerate(W.query_stream(w, many.q0, w.steps, R.DEV)):
        many.step(0, t, q[0])
        one.step(0, t, q[0])
        assert np.array_equal(many.n_sel_pages, one.n_sel_pages), t
        # (the probabilities that multiply V keep 16 bits in bf16 and 11 in fp16, relative to each split's own maximum)
        err = H.attn_rel_err(many.n_out.reshape(-1, 128), one.n_out.reshape(-1, 128))
        assert err <= (2.0 ** -14 if w.dtype == "bf16" else 2.0 ** -11), (t, err)
        assert np.abs(many.n_lse - one.n_lse).max() <= 1e-4, t
    many.close()
    one.close()


@pytest.mark.parametrize("mb", [-1, 1], ids=["single-launch", "kernel-chain"])
@pytest.mark.parametrize("splits,kw", [
    (9, dict()),
    (9, dict(n_q_heads=2)),                                # a head has fewer dims than the workgroup threads
    (17, dict(n_q_heads=16)),
    (33, dict(dtype="f16")),
])
def test_merge_of_many_splits_reads_no_other_units_partials(splits, kw, mb):
    """The merge fetches partials 16 or 32 at a time, more than there are; what lies behind a unit's partials is the next
    unit's, and here that holds infinities and NaN in every other unit."""
    w = small("merge-bounds", **{**dict(ctx=16 * 600, topk_pages=257, capacity=300, heavy_count=3, steps=3, batch=4), **kw})
    many, one = R.Rig(w, micro_batches=mb, attn_splits=splits), R.Rig(w, micro_batches=mb, attn_splits=1)
    for r in (many, one):
        r.store[:, 1::2, :, :, 1] = float("inf")           # V of every second sequence, whatever its pages
        r.store[:, 1::2, :, :, 1, :, ::2] = float("nan")
    for t, q in enumerate(W.query_stream(w, many.q0, w.steps, R.DEV)):
        many.step(0, t, q[0])
        one.step(0, t, q[0])
        assert not np.isfinite(many.n_out[1::2]).any()
        got, want = many.n_out[::2].reshape(-1, 128), one.n_out[::2].reshape(-1, 128)
        assert np.isfinite(got).all() and np.isfinite(many.n_lse).all(), t
        # (as in the test above)
        assert H.attn_rel_err(got, want) <= (2.0 ** -14 if w.dtype == "bf16" else 2.0 ** -11), t
    many.close()
    one.close()


@pytest.mark.parametrize("splits", [9, 17, 33])
def test_merge_of_many_splits_in_used_scratch(splits):
    """The call without a context works in one array of the library: first 64 splits of values that are no numbers, then
    fewer splits of ordinary ones, whose last unit's partials have the old ones right behind them."""
    w = small("merge-scratch", ctx=16 * 300, topk_pages=129, capacity=140, heavy_count=3, steps=1, batch=2)
    rig = R.Rig(w, micro_batches=1, attn_splits=1)
    q = next(W.query_stream(w, rig.q0, 1, R.DEV))[0].contiguous()
    rig.step(0, 0, q)
    seq = torch.tensor(rig.seq_lens, dtype=torch.int32, device=R.DEV)
    shape = dict(batch=w.batch, n_q_heads=w.n_q_heads, n_kv_heads=w.n_kv_heads, page_size=w.page, topk_pages=w.topk_pages,
                 capacity_max=w.capacity, kv_dtype=w.torch_dtype)
    bad, got = torch.full_like(rig.pool[0], float("nan")), torch.empty_like(rig.out)
    K.sparse_decode_attn_noalloc(q, bad, rig.sel_pages, rig.sel_slots, seq, got, None, attn_splits=64, **shape)
    K.sparse_decode_attn_noalloc(q, rig.pool[0], rig.sel_pages, rig.sel_slots, seq, got, None, attn_splits=splits, **shape)
    torch.cuda.synchronize()
    got = got.cpu().numpy().reshape(-1, 128)
    assert np.isfinite(got).all()
    assert H.attn_rel_err(got, rig.n_out.reshape(-1, 128)) <= 2.0 ** -14
    rig.close()


def few_large_units(**kw):
    """4 units of more than 8192 pages: with the form left to the library a layer steps as a chain of kernels, and several
    share a launch."""
    return small("few-large", **{**dict(ctx=16 * 8200, topk_pages=100, capacity=150, batch=2, n_kv_heads=2, n_q_heads=8, n_layers=9,
                                        physical_layers=1, heavy_count=5, steps=4, rho=0.3), **kw})


@pytest.mark.parametrize("kw", [dict(), dict(policy="lookahead", dtype="f16", n_q_heads=14), dict(page=8, ctx=8 * 8301, n_layers=3),
                                dict(index_centroids=300, index_iterations=2, n_layers=2)],
                         ids=["lru", "lookahead-f16", "packed", "clusters"])
def test_layers_that_share_a_launch_only_together(kw):
    """Outputs, directory, trace and counters are those of the layers one by one: the launch has the chain's splits.  Of nine
    layers eight share a launch and the last one goes as a single layer, in the first one's scratch."""
    w = few_large_units(**kw)
    L = w.n_layers
    one, together = R.Rig(w, seq_lens=[w.ctx - 5, w.ctx - 700]), R.Rig(w, seq_lens=[w.ctx - 5, w.ctx - 700])
    assert one.kvd.step_form() == together.kvd.step_form() == 1
    shape = (L, w.batch, w.n_q_heads, w.head_dim)
    a, b = (torch.empty(shape, dtype=torch.float32, device=R.DEV) for _ in range(2))
    la, lb = (torch.empty(shape[:-1], dtype=torch.float32, device=R.DEV) for _ in range(2))
    for t, q in enumerate(W.query_stream(w, one.q0, w.steps, R.DEV)):
        b.fill_(float("nan"))
        for l in range(L):
            one.kvd.step(l, t, q[l], a[l], la[l])
        n = L if t % 2 == 0 else L - 1                       # with and without the one that is left over
        together.kvd.step_layers(0, n, t, q[:n].contiguous(), b, lb)
        if n < L:
            together.kvd.step(n, t, q[n], b[n], lb[n])
        traces = []
        for r in (one, together):
            r.kvd.step_trace(r.sel_pages, r.sel_slots, r.hit_mask, r.evicted, r.counts, r.scores)
            torch.cuda.synchronize()
            scores = r.scores.flatten()[:w.units * (w.index_centroids or w.n_pages)]
            traces.append([x.clone() for x in (r.sel_pages, r.sel_slots, r.hit_mask, r.evicted.sort().values, r.counts, scores)])
        assert torch.equal(a, b) and torch.equal(la, lb), t
        for i, (x, y) in enumerate(zip(*traces)):
            assert torch.equal(x, y), (t, i)
    for l in range(L):
        for x, y in zip(one.kvd.cache_export(l), together.kvd.cache_export(l)):
            assert torch.equal(x, y), l
    s1, s2 = one.kvd.stats(), together.kvd.stats()
    assert (s1.steps, s1.hits, s1.misses, s1.evictions) == (s2.steps, s2.hits, s2.misses, s2.evictions) and s1.evictions > 0
    one.close()
    together.close()


def test_layers_that_share_a_launch_only_together_recover_from_a_wait():
    w = few_large_units(n_layers=3)
    rig, cold = R.Rig(w), R.Rig(w)
    out, want = (torch.empty((3, w.batch, w.n_q_heads, w.head_dim), dtype=torch.float32, device=R.DEV) for _ in range(2))
    qs = [q.contiguous() for q in W.query_stream(w, rig.q0, w.steps, R.DEV)]
    rig.kvd.step_layers(0, 3, 0, qs[0], out)
    rig.kvd.set_wait_limit_us(0)
    rig.kvd.step_layers(0, 3, 1, qs[1], out)                 # workgroups that have to wait give up
    torch.cuda.synchronize()
    for call in (rig.kvd.stats, lambda: rig.kvd.step_layers(0, 3, 2, qs[2], out)):
        with pytest.raises(K.KvdError) as e:
            call()
        assert e.value.status == K.ERR_STATE
    # told once; the layers go on from empty windows, each as a chain (the limit is still 0: nothing waits any more)
    for t in (2, 3):
        rig.kvd.step_layers(0, 3, t, qs[t], out)
        for l in range(3):
            cold.kvd.step(l, t, qs[t][l], want[l])
        torch.cuda.synchronize()
        rig.kvd.stats()
        assert rig.kvd.step_form() == 1 and torch.equal(out, want), t
        for l in range(3):
            for x, y in zip(rig.kvd.cache_export(l), cold.kvd.cache_export(l)):
                assert torch.equal(x, y), (t, l)
    rig.close()
    cold.close()


@pytest.mark.parametrize("call", ["resolve", "attention", "tiered"])
def test_calls_after_a_wait_that_ran_out_report_it(call, tmp_path):
    """What the failed launch left (directories half updated, tickets not at zero) is not worked on by the stage calls and
    the tiered step either: they report the failure once, and the next call starts from empty windows."""
    w = few_large_units(n_layers=2, ctx=16 * 8193)
    rig = R.Rig(w)
    if call == "tiered":
        rig.attach_tier(str(tmp_path / "pages"), extent_pages=8, pool_extents=4000)
        rig.kvd.bind_host_store(rig.store)
    out = torch.empty((2, w.batch, w.n_q_heads, w.head_dim), dtype=torch.float32, device=R.DEV)
    qs = [q.contiguous() for q in W.query_stream(w, rig.q0, w.steps, R.DEV)]
    rig.kvd.score_select(0, qs[1][0], rig.sel_pages)
    rig.kvd.step_layers(0, 2, 0, qs[0], out)
    rig.kvd.set_wait_limit_us(0)
    rig.kvd.step_layers(0, 2, 1, qs[1], out)
    torch.cuda.synchronize()
    run = {"resolve": lambda: rig.kvd.cache_resolve(0, 2, rig.sel_pages, rig.sel_slots),
           "attention": lambda: rig.kvd.sparse_decode_attn(0, qs[1][0], rig.sel_pages, rig.sel_slots, rig.out),
           "tiered": lambda: rig.kvd.step_tiered(0, 2, qs[1][0], rig.out)}[call]
    rig.sel_slots.fill_(-1)
    with pytest.raises(K.KvdError) as e:
        run()
    assert e.value.status == K.ERR_STATE
    assert rig.kvd.step_form() == 1 and all((rig.kvd.cache_export(l)[0] == -1).all() for l in range(2))
    run()
    torch.cuda.synchronize()
    rig.kvd.stats()
    rig.close()
