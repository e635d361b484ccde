"""Units of more pages or slots than the register-resident selection holds: the form of the same kernel that
reads the scores once per pass, from just above the sizes of the other form to its own limits, and just beyond them."""
import pytest
import torch

from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests import gpu_rig as R


@pytest.mark.parametrize("pages,k,cap,kw", [
    (16385, 300, 700, dict()),                                                            # one page more than the registers hold
    (16388, 2048, 2100, dict(policy="lookahead", sink_pages=5, recent_pages=9)),          # the largest k, forced pages
    (300, 40, 4097, dict()),                                                              # few pages, one slot more
    (6000, 500, 5000, dict(policy="lookahead", lookahead_pool=700)),                      # victims among more than 4096 slots
    (33001, 600, 1300, dict(policy="lookahead", dtype="f16", lookahead_pool=900)),        # pages no multiple of 4
    (65536, 700, 1500, dict(sink_pages=3, recent_pages=3)),                               # the largest
    (65537, 100, 220, dict()),                                                            # beyond: the size-agnostic kernels
    (20000, 64, 16385, dict()),
])
def test_step_parity(pages, k, cap, kw):
    w = small("big", **{**dict(ctx=4 * pages, page=4, topk_pages=k, capacity=cap, batch=2, n_kv_heads=1, n_q_heads=4,
                               heavy_count=32, steps=4), **kw})
    rig = R.Rig(w, seq_lens=[w.ctx - 1, w.ctx - w.ctx // 3])
    assert rig.kvd.step_form() == 1
    units = [R.OracleUnit(rig, 0, b, 0, lazy=True) for b in range(w.batch)]
    rep = R.run_steps(rig, units, w.steps, check_dir_every=2, progress=f"big-{pages}-{cap}")
    assert rep.unit_steps == w.steps * w.units
    assert rep.tie_divergences <= 2 and rep.victim_tie_divergences <= 2
    rig.close()


@pytest.mark.parametrize("policy", ["lru", "lookahead"])
def test_degenerate_scores_and_victims(policy):
    """All scores equal (more candidates in the decisive bucket than the list holds: radix refinement), and window
    content that all looks alike to the victim choice."""
    w = small("big-ties", ctx=4 * 17000, page=4, topk_pages=96, capacity=4200, heavy_count=0, batch=1, n_kv_heads=2,
              n_q_heads=4, policy=policy, steps=1)
    rig = R.Rig(w)
    warm = list(range(12000, 16200))
    rig.kvd.cache_warm(0, warm * w.units, [len(warm)] * w.units)
    units = [R.OracleUnit(rig, 0, 0, h, lazy=True) for h in range(w.n_kv_heads)]
    for ou in units:
        ou.window.warm(warm, stamp=-1)
    zero = torch.zeros((w.batch, w.n_q_heads, w.head_dim), dtype=w.torch_dtype, device=R.DEV)
    rep = R.StepReport()
    for t in (100, 101):
        rig.step(0, t, zero)
        for ou in units:
            R.compare_unit(rig, ou, t, zero, rep)
    assert rep.tie_divergences == 0 and rep.victim_tie_divergences == 0
    rig.close()


def test_stages_one_by_one():
    w = small("big-stages", ctx=4 * 17001, page=4, topk_pages=200, capacity=500, batch=2, n_kv_heads=1, n_q_heads=7, steps=3)
    rig, whole = R.Rig(w, seq_lens=[w.ctx, w.ctx - 999]), R.Rig(w, seq_lens=[w.ctx, w.ctx - 999])
    for t, q in enumerate(R.W.query_stream(w, rig.q0, w.steps, R.DEV)):
        rig.kvd.score_select(0, q[0], rig.sel_pages, rig.scores)
        rig.kvd.cache_resolve(0, t, rig.sel_pages, rig.sel_slots, rig.hit_mask, rig.evicted, rig.counts)
        rig.kvd.sparse_decode_attn(0, q[0], rig.sel_pages, rig.sel_slots, rig.out, rig.lse)
        whole.step(0, t, q[0])
        torch.cuda.synchronize()
        assert torch.equal(rig.sel_pages, whole.sel_pages) and torch.equal(rig.sel_slots, whole.sel_slots)
        assert torch.equal(rig.hit_mask, whole.hit_mask) and torch.equal(rig.counts, whole.counts)
        assert torch.equal(rig.out, whole.out) and torch.equal(rig.lse, whole.lse)
    rig.close()
    whole.close()


@pytest.mark.parametrize("mb,pool", [(1, 0), (2, 0), (1, 700)])
def test_hierarchical_index_with_more_slots_than_the_registers_hold(mb, pool):
    """Selection through the centroids, victims by the score of their cluster among 4300 slots, all taken."""
    w = small("big-hier", ctx=4 * 6000, page=4, topk_pages=500, capacity=4300, batch=2, n_kv_heads=1, n_q_heads=4,
              heavy_count=32, steps=4, policy="lookahead", lookahead_pool=pool, index_centroids=1200, index_iterations=2)
    rig = R.Rig(w, seq_lens=[w.ctx - 1, w.ctx - 4 * 900], micro_batches=mb)
    assert rig.kvd.step_form() == mb
    warm = list(range(700, 5000))
    rig.kvd.cache_warm(0, warm * w.units, [len(warm)] * w.units)
    units = [R.OracleUnit(rig, 0, b, 0) for b in range(w.batch)]
    for ou in units:
        ou.window.warm(warm, stamp=-1)
    rep = R.run_steps(rig, units, w.steps, check_dir_every=2, progress=f"big-hier-{mb}-{pool}")
    assert rep.unit_steps == w.steps * w.units and rig.kvd.stats().evictions > w.units
    assert rep.tie_divergences <= 2 and rep.victim_tie_divergences <= 4
    rig.close()


def test_every_way_through_a_step_gives_the_same(tmp_path):
    """Two groups on streams, the tier behind the window and the profiled step against the plain chain of kernels."""
    w = small("big-ways", ctx=4 * 17000, page=4, topk_pages=200, capacity=500, batch=2, n_kv_heads=1, n_q_heads=4, steps=4)
    plain, groups, tiered, profiled = (R.Rig(w, seq_lens=[w.ctx - 2, w.ctx // 2], micro_batches=mb) for mb in (1, 2, 1, 1))
    tiered.attach_tier(str(tmp_path / "kv.bin"), extent_pages=8, pool_extents=600, max_run_extents=8)
    profiled.kvd.set_profiling(1)
    for t, q in enumerate(R.W.query_stream(w, plain.q0, w.steps, R.DEV)):
        for rig in (plain, groups, tiered, profiled):
            rig.step(0, t, q[0])
        for rig in (groups, tiered, profiled):
            for name in ("sel_pages", "sel_slots", "hit_mask", "counts", "out", "lse"):
                assert torch.equal(getattr(rig, name), getattr(plain, name)), name
    for rig in (plain, groups, tiered, profiled):
        rig.close()
