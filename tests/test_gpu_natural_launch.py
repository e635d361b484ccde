"""Pages kept in natural order (sizes that are neither 4, 8 nor a multiple of 16): with the choice of form left to the library
the step is one launch.  It is compared with the chain of kernels, whose stages the oracle checks."""
import pytest
import torch

from paper_2605_18071_amd import kvd as K
from paper_2605_18071_amd import workloads as W
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests import gpu_rig as R


def fresh(w, seq, mb):
    return R.Rig(w, seq_lens=seq, micro_batches=mb)


@pytest.mark.parametrize("page,pages,k,kw", [
    (1, 700, 520, dict()),                                             # more entries than one split stages
    (2, 2049, 60, dict(dtype="f16")),                                  # two pages to a KiB piece of the copy
    (3, 300, 17, dict(sink_pages=1, recent_pages=2)),                  # a page ends in half a piece
    (12, 513, 33, dict(n_q_heads=14, policy="lookahead")),
    (24, 400, 85, dict(dtype="f16", n_q_heads=14, sink_pages=2, recent_pages=4)),
    (33, 90, 20, dict(policy="lookahead", lookahead_pool=25)),
    (20, 600, 40, dict(index_centroids=70)),
    (255, 40, 5, dict()),
    (3, 4000, 150, dict(n_q_heads=6, dtype="f16")),                    # each number of pages that a thread holds, and what it holds them in
    (20, 8000, 40, dict(n_q_heads=10, heavy_count=3, steps=3)),
    (20, 7000, 40, dict(n_q_heads=16, heavy_count=3, steps=3, dtype="f16")),
    (6, 8200, 30, dict(batch=5)),                                      # 10 units of more than 8192 pages
])
def test_equals_the_chain(page, pages, k, kw):
    w = small("natural-launch", **{**dict(ctx=page * pages, page=page, topk_pages=k, capacity=k + k // 2 + 2, batch=3, n_kv_heads=2, n_q_heads=4,
                                          heavy_count=3, steps=5, rho=0.5), **kw})
    seq = [max(1, w.ctx - page // 2 - b * (w.ctx // 3)) for b in range(w.batch)]
    one, chain = fresh(w, seq, 0), fresh(w, seq, 1)
    misses = 0
    for t, q in enumerate(W.query_stream(w, one.q0, w.steps, R.DEV)):
        one.out.fill_(float("nan"))
        one.step(0, t, q[0])
        chain.step(0, t, q[0])
        misses += int(chain.n_counts[:, 1].sum())
        for what in ("sel_pages", "sel_slots", "hit_mask", "counts"):
            assert torch.equal(getattr(one, what), getattr(chain, what)), (what, t)
        # 24 bits of P and fp32 sums in both, in another order where the splits differ
        assert float((one.out - chain.out).norm() / chain.out.norm()) < 1e-6
        assert float((one.lse - chain.lse).abs().max()) < 1e-4
    assert misses > 0 and torch.equal(one.pool, chain.pool)
    one.close()
    chain.close()


@pytest.mark.parametrize("layers,pages,kw", [(5, 300, dict()), (3, 8300, dict(batch=1, n_kv_heads=2)), (10, 60, dict(dtype="f16", page=12))])
def test_layers_in_a_launch_equal_layers_one_by_one(layers, pages, kw):
    """Bit for bit; 3 layers of two units of 8300 pages step one by one as a chain, whose splits the shared launch has."""
    w = small("natural-layers", **{**dict(page=6, topk_pages=25, capacity=37, batch=3, n_kv_heads=2, n_q_heads=4, heavy_count=3, steps=4,
                                          n_layers=layers, physical_layers=2, rho=0.5), **kw})
    w = w.replace(ctx=w.page * pages)
    seq = [w.ctx - 5 * b for b in range(w.batch)]
    one, together = fresh(w, seq, 0), fresh(w, seq, 0)
    shape = (layers, w.batch, w.n_q_heads, w.head_dim)
    a, b = (torch.empty(shape, dtype=torch.float32, device=R.DEV) for _ in range(2))
    for t, q in enumerate(W.query_stream(w, one.q0, w.steps, R.DEV)):
        b.fill_(float("nan"))
        for l in range(layers):
            one.kvd.step(l, t, q[l], a[l])
        together.kvd.step_layers(0, layers, t, q, b)
        torch.cuda.synchronize()
        assert torch.equal(a, b), t
    assert torch.equal(one.pool, together.pool)
    one.close()
    together.close()


def test_a_pool_that_starts_inside_a_cache_line_and_a_wait_that_runs_out():
    """Slots that share cache lines take the chain, which has no waits; elsewhere a wait that runs out is reported once and
    the context goes on as a chain."""
    w = small("natural-limits", page=12, ctx=12 * 300, topk_pages=40, capacity=60, batch=2, n_kv_heads=2, n_q_heads=4, steps=3)
    rig, shifted, chain = fresh(w, [w.ctx] * 2, 0), fresh(w, [w.ctx] * 2, 0), fresh(w, [w.ctx] * 2, 1)
    room = torch.zeros(rig.pool.numel() + 64, dtype=w.torch_dtype, device=R.DEV)
    shifted.kvd.bind_slot_pool(room[8:8 + rig.pool.numel()].view(rig.pool.shape))
    for r in (rig, shifted, chain):
        r.kvd.set_wait_limit_us(0)
    qs = list(W.query_stream(w, rig.q0, w.steps, R.DEV))
    for t, q in enumerate(qs):
        shifted.step(0, t, q[0])
        chain.step(0, t, q[0])
        assert torch.equal(shifted.sel_slots, chain.sel_slots) and torch.equal(shifted.out, chain.out)
    rig.kvd.step(0, 0, qs[0][0], rig.out, rig.lse)
    torch.cuda.synchronize()
    with pytest.raises(K.KvdError):
        rig.kvd.step(0, 0, qs[0][0], rig.out, rig.lse)
    for t, q in enumerate(qs):
        rig.step(0, t, q[0])
        chain.step(0, t + 3, q[0])
        assert torch.equal(rig.sel_pages, chain.sel_pages) and torch.equal(rig.out, chain.out)
    for r in (rig, shifted, chain):
        r.close()


def test_the_form_that_runs_is_the_one_reported():
    """Form 0 where the library's choice is one launch: setting what is reported changes nothing, a calibration times the chain
    and the launch apart and leaves the form that it names, and a launch's timeline can be had."""
    w = small("natural-form", page=12, ctx=12 * 300, topk_pages=40, capacity=60, batch=3, n_kv_heads=2, n_q_heads=4, heavy_count=3, steps=4)
    seq = [w.ctx] * w.batch
    rig, same, chain = fresh(w, seq, 0), fresh(w, seq, 0), fresh(w, seq, 1)
    assert rig.kvd.step_form() == 0 and chain.kvd.step_form() == 1
    qs = [q[0] for q in W.query_stream(w, rig.q0, w.steps, R.DEV)]
    for t, q in enumerate(qs):
        same.kvd.set_step_form(same.kvd.step_form())
        assert same.kvd.step_form() == 0
        rig.step(0, t, q)
        same.step(0, t, q)
        chain.step(0, t, q)
        assert torch.equal(rig.out, same.out) and torch.equal(rig.sel_slots, chain.sel_slots)
    with pytest.raises(K.KvdError):
        rig.kvd.set_step_form(-1)
    # the timeline of the launch
    with pytest.raises(K.KvdError):
        chain.kvd.step_timeline()
    rig.kvd.set_profiling(2)
    rig.step(0, w.steps, qs[0])
    rec = rig.kvd.step_timeline()
    rig.kvd.set_profiling(0)
    role = rec[:, 4] & 0xff
    assert int((role == 1).sum()) == w.units and bool((rec[:, 3] >= rec[:, 0]).all()) and int((role == 2).sum()) % w.units == 0
    # the calibration
    for r in (rig, chain):
        chosen, ms = r.kvd.calibrate_step_form(0, w.steps + 1, torch.stack(qs).contiguous(), 5, r.out)
        assert set(ms) == {0, 1, 2} and all(v > 0 for v in ms.values())
        assert chosen == min(ms, key=ms.get) and r.kvd.step_form() == chosen
    rig.kvd.set_step_form(0)
    same.kvd.set_step_form(1)
    assert rig.kvd.step_form() == 0 and same.kvd.step_form() == 1
    for r in (rig, same, chain):
        r.close()
    # what the library's choice takes as a chain is one
    few = small("natural-few", page=6, ctx=6 * 8300, topk_pages=25, capacity=37, batch=1, n_kv_heads=2, n_q_heads=4, steps=2)
    rig = fresh(few, [few.ctx], 0)
    assert rig.kvd.step_form() == 1
    q = torch.stack([q[0] for q in W.query_stream(few, rig.q0, 2, R.DEV)]).contiguous()
    assert set(rig.kvd.calibrate_step_form(0, 0, q, 2, rig.out)[1]) == {1}
    rig.close()


@pytest.mark.parametrize("shape", [(1, 5, 2, 1), (2, 7, 3, 2), (0, 0, 8, 0), (3, 200, 1, 4), (0, 0, 0, 0)])
def test_the_launch_shape_that_is_reported_runs(shape):
    w = small("natural-shape", page=20, ctx=20 * 1100, topk_pages=35, capacity=50, batch=3, n_kv_heads=2, n_q_heads=4, heavy_count=3,
              n_layers=3, steps=3, rho=0.5)
    seq = [w.ctx - 5 * b for b in range(w.batch)]
    rig, one, chain = fresh(w, seq, 0), fresh(w, seq, 0), fresh(w, seq, 1)
    for r in (rig, one):
        r.kvd.set_step_shape(*shape)
    rig.kvd.set_step_shape(*shape, multi_layer=True)
    for multi in (False, True):
        got = rig.kvd.step_shape(multi_layer=multi)
        assert all(a == b for a, b in zip(got, shape) if b > 0) or shape[1] > got[1], got
    out = torch.empty((w.n_layers, w.batch, w.n_q_heads, w.head_dim), dtype=torch.float32, device=R.DEV)
    for t, q in enumerate(W.query_stream(w, rig.q0, w.steps, R.DEV)):
        out.fill_(float("nan"))
        rig.kvd.step_layers(0, w.n_layers, t, q, out)
        for l in range(w.n_layers):
            one.step(l, t, q[l])
            chain.step(l, t, q[l])
            assert torch.equal(out[l], one.out) and torch.equal(one.sel_slots, chain.sel_slots), (t, l)
            assert float((one.out - chain.out).norm() / chain.out.norm()) < 1e-6
    assert torch.equal(rig.pool, chain.pool)
    one.kvd.set_profiling(2)
    one.step(0, w.steps, q[0])
    role = one.kvd.step_timeline()[:, 4] & 0xff
    passes, n_score, splits, groups = one.kvd.step_shape()
    assert int((role == 2).sum()) == splits * w.units and int((role == 0).sum()) == n_score * groups
    with pytest.raises(K.KvdError):
        rig.kvd.set_step_shape(passes=9)
    with pytest.raises(K.KvdError):                       # shapes are calibrated in form -1 only
        rig.kvd.calibrate_step_shape(0, w.steps, q[0], rig.out)
    for r in (rig, one, chain):
        r.close()


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("k", [1, 10, 11, 21, 22, 43, 70, 115])
def test_tiles_of_a_split_and_of_its_waves(k, dtype):
    """One split of k pages of 12 tokens: 1, 8, 9, 16, 17, 33, 53 and 87 tiles for 8 waves; sequences that fill the selection, end in
    its first tiles, and are a token long."""
    w = small("natural-tiles", page=12, ctx=12 * 120, topk_pages=k, capacity=k + 9, batch=4, n_kv_heads=2, n_q_heads=6, heavy_count=0, steps=3,
              dtype=dtype, rho=0.5)
    seq = [w.ctx, 12 * max(1, k - 2) - 5, 12 * (k // 3) + 1, 1]   # (waves that end before the split does)
    one, chain = (R.Rig(w, seq_lens=seq, micro_batches=mb, attn_splits=1) for mb in (0, 1))
    assert one.kvd.step_form() == 0 and one.kvd.step_shape()[2] == 1
    for t, q in enumerate(W.query_stream(w, one.q0, w.steps, R.DEV)):
        one.out.fill_(float("nan"))
        one.step(0, t, q[0])
        chain.step(0, t, q[0])
        assert torch.equal(one.sel_slots, chain.sel_slots)
        assert float((one.out - chain.out).norm() / chain.out.norm()) < 1e-6 and float((one.lse - chain.lse).abs().max()) < 1e-4
        # a selection that is all of its sequence: attention over it in fp64
        for b in range(w.batch):
            if -(-seq[b] // w.page) > k:
                continue
            kv = one.store[0, b].double()
            K_, V_ = (kv[:, :, i].reshape(w.n_kv_heads, -1, 128)[:, :seq[b]] for i in (0, 1))
            qb = q[0][b].double().cpu().view(w.n_kv_heads, w.group, 128)
            logits = qb @ K_.transpose(1, 2) / 128 ** 0.5
            want = (torch.softmax(logits, -1) @ V_).reshape(w.n_q_heads, 128)
            got = one.out[b].double().cpu()
            assert float((got - want).norm() / want.norm()) < 1e-5, (t, b)
    one.close()
    chain.close()
