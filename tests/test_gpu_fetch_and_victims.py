"""The copy of missed pages, piece by piece, and the choice of victims, at the edges of what a batch of a wave's pieces, a thread's slots and a
bucket of victims hold."""
import numpy as np
import pytest
import torch

from paper_2605_18071_amd import workloads as W
from tests import helpers as H
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests import gpu_rig as R


# Pieces of a page: half its tokens, rounded up, in natural order (1 KiB each), else a quarter.  A workgroup has 64 (natural) or 32
# of them on their way at a time; with 48 units and more 24 (in the chain 16) and 8 (16).
@pytest.mark.parametrize("batch", [1, 23, 24])
@pytest.mark.parametrize("mb", [0, 1], ids=["one-launch", "chain"])
@pytest.mark.parametrize("page,ks", [
    (1, [1, 7, 8, 9, 63, 64, 65, 129]),                   # a piece that is half there
    (2, [64, 65]),
    (3, [4, 31, 32, 33]),                                 # ... behind one that is
    (15, [1, 2, 3, 4]),                                   # 8 pieces a page
    (254, [1]), (255, [1, 2]),
    (4, [1, 7, 8, 9, 31, 32, 33, 65]),
    (8, [16, 17]),
    (16, [1, 7, 8, 9, 17]),
    (48, [2, 3]), (256, [1, 2]),
])
def test_pages_of_any_number_of_pieces(page, ks, mb, batch):
    for k in ks:
        if batch * 2 * (k + 3) * page > 60_000:
            continue
        w = small("pieces", page=page, ctx=page * (k + 3), topk_pages=k, capacity=k + 2, batch=batch, n_kv_heads=2, n_q_heads=4, heavy_count=0,
                  steps=1, seed=10 * page + k)
        rig = R.Rig(w, micro_batches=mb)
        rig.pool.view(torch.int16).fill_(0x2a55)
        q = next(iter(W.query_stream(w, rig.q0, 1, R.DEV)))[0]
        rig.step(0, 0, q)
        assert np.array_equal(rig.n_counts, [[0, k, 0]] * w.units), k
        for u in range(w.units):
            pages, slots = rig.n_sel_pages[u], rig.n_sel_slots[u]
            assert sorted(slots.tolist()) == list(range(k))
            pool, store = rig.pool[0].flatten(0, 1)[u].cpu(), rig.store[0].flatten(0, 1)[u]
            for s in range(w.capacity):
                got = pool[s].view(torch.int16).reshape(-1)
                if s in slots:
                    assert torch.equal(got, H.slot_image(store[int(pages[list(slots).index(s)])])), (k, u, s)
                else:                                     # a slot that no page went to
                    assert bool((got == 0x2a55).all()), (k, u, s)
        rig.close()


# A thread holds as few consecutive slots as make up the window: 1 up to 512 (or, in the chain, 1024) slots, then one more for each 512.
@pytest.mark.parametrize("mb", [0, 1], ids=["one-launch", "chain"])
@pytest.mark.parametrize("capacity,t0,kw", [
    (300, 0, dict()),                                     # the newest class alone; k is the window
    (511, 1, dict()),
    (512, 10, dict(policy="lookahead")),
    (513, 61, dict()),                                    # ages 62 and on: the oldest class that is split by pages, then the one of all older
    (1024, 62, dict(sink_pages=3)),
    (1025, 63, dict()),
    (1030, 5, dict(policy="lookahead", lookahead_pool=400)),
    (1536, 20, dict()),
    (1537, 2**31 - 200, dict()),                          # the last steps there are
    (2500, 0, dict(policy="lookahead", lookahead_pool=2600)),
    (3076, 3, dict()),                                    # slots in loads of four: in the chain from 3073 on, in the launch from 3585
    (3588, 8, dict(policy="lookahead")),
    (3590, 8, dict()),                                    # a number of slots that is no multiple of four
    (4095, 30, dict()),
    (4096, 0, dict()),                                    # more pages of one class than a list holds
    (4096, 100, dict(policy="lookahead")),
])
def test_windows_of_any_number_of_slots_and_victims_of_any_age(capacity, t0, kw, mb):
    w = small("windows", **{**dict(page=4, ctx=4 * (capacity + 800), topk_pages=300, capacity=capacity, batch=1, n_kv_heads=2, n_q_heads=4,
                                   heavy_count=0, steps=8, rho=0.2, seed=capacity + t0), **kw})
    rig = R.Rig(w, micro_batches=mb)
    assert rig.kvd.step_form() == (-1 if mb == 0 else 1)
    gen = np.random.default_rng(capacity)
    n = max(0, capacity - 3) if capacity > 300 else capacity          # (three free slots: misses beyond them evict)
    warm = [sorted(gen.choice(w.n_pages, n, replace=False).tolist()) for _ in range(w.units)]
    gen.shuffle(warm[0])                                  # pages in no order over the slots
    rig.kvd.cache_warm(0, [int(p) for lst in warm for p in lst], [n] * w.units)
    units = [R.OracleUnit(rig, 0, 0, h, lazy=True) for h in range(w.n_kv_heads)]
    for ou in units:
        ou.window.warm(warm[ou.u], stamp=-1)
    rep = R.StepReport()
    evicted = 0
    for t, q in zip([t0, t0 + 1, t0 + 2, t0 + 40, t0 + 63, t0 + 64, t0 + 65, t0 + 190], W.query_stream(w, rig.q0, w.steps, R.DEV)):
        rig.step(0, t, q[0])
        evicted += int(rig.n_counts[:, 2].sum())
        for ou in units:
            R.compare_unit(rig, ou, t, q[0], rep)
        R.check_directory(rig, 0, units, check_data=False)
    assert evicted > 200 and rep.tie_divergences <= 2 and rep.victim_tie_divergences <= 2
    R.check_directory(rig, 0, units)
    rig.close()


@pytest.mark.parametrize("pages,same,k,sink,recent", [(16385, 1, 1024, 0, 0), (32768, 1, 1025, 0, 0), (20001, 50, 400, 7, 9), (24576, 2500, 64, 0, 0),
                                                      (28672, 9000, 500, 2, 0), (30001, 30001, 90, 0, 5)])
def test_the_selection_alone_by_quads(pages, same, k, sink, recent, monkeypatch):
    """kvd_score_select of units of 16385 pages and more: what the size-agnostic kernels select."""
    w = small("select-alone", ctx=4 * pages, page=4, topk_pages=k, capacity=k + 4, batch=2, n_kv_heads=1, n_q_heads=4, heavy_count=0, steps=2,
              sink_pages=sink, recent_pages=recent)
    seq = [w.ctx - 1, w.ctx - w.ctx // 7]
    fused = R.Rig(w, seq_lens=seq, build_index=False)
    monkeypatch.setenv("KVD_GENERIC_SELECT", "1")
    plain = R.Rig(w, seq_lens=seq, build_index=False)
    gen = torch.Generator(device=R.DEV)
    gen.manual_seed(pages + k)
    rows = max(1, pages // same)
    base = torch.randn(w.units, rows, 128, device=R.DEV, generator=gen)
    summ = base[:, torch.randperm(pages, device=R.DEV, generator=gen) % rows].to(w.torch_dtype)
    for r in (fused, plain):
        r.summaries.copy_(summ.view(r.summaries.shape))
    for q in W.query_stream(w, fused.q0, w.steps, R.DEV):
        for r in (fused, plain):
            r.sel_pages.fill_(-7)
            r.kvd.score_select(0, q[0], r.sel_pages, r.scores)
        torch.cuda.synchronize()
        assert torch.equal(fused.scores, plain.scores) and torch.equal(fused.sel_pages, plain.sel_pages)
    fused.close()
    plain.close()
