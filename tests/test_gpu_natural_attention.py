"""Attention over pages kept in natural order (sizes that are neither 4, 8 nor a multiple of 16): tiles of 16
consecutive tokens of the selection, whichever pages they lie in, against the oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import kvd_oracle as orc
from tests import helpers as H
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests import gpu_rig as R


def attend(w, seq, splits, edit=None):
    """(GPU output, GPU lse, oracle output, oracle lse) of a made-up selection over cold-fetched pages."""
    rig = R.Rig(w, seq_lens=seq, attn_splits=splits, build_index=False)
    if edit is not None:
        edit(rig.store)
    rng = np.random.default_rng(5)
    sel = np.full((w.units, w.topk_pages), -1, dtype=np.int32)
    for u in range(w.units):
        n = -(-seq[u // w.n_kv_heads] // w.page)
        kk = min(w.topk_pages, n)
        sel[u, :kk] = np.sort(np.append(rng.choice(n - 1, size=kk - 1, replace=False), n - 1))   # the ragged last page included
    rig.sel_pages.copy_(torch.from_numpy(sel))
    q = next(R.W.query_stream(w, rig.q0, 1, R.DEV))[0]
    rig.kvd.cache_resolve(0, 0, rig.sel_pages, rig.sel_slots)
    rig.kvd.sparse_decode_attn(0, q, rig.sel_pages, rig.sel_slots, rig.out, rig.lse)
    torch.cuda.synchronize()
    out, lse = torch.zeros_like(rig.out, device="cpu", dtype=torch.float64), torch.zeros_like(rig.lse, device="cpu", dtype=torch.float64)
    for u in range(w.units):
        b, h = divmod(u, w.n_kv_heads)
        pages = torch.from_numpy(sel[u][sel[u] >= 0]).long()
        tok = (pages[:, None] * w.page + torch.arange(w.page)).reshape(-1)
        k, v = (rig.store[0, b, h, pages, i].reshape(-1, w.head_dim)[tok < seq[b]].double() for i in (0, 1))
        heads = slice(h * w.group, (h + 1) * w.group)
        logits = q[b, heads].double().cpu() @ k.T / math.sqrt(w.head_dim)
        out[b, heads], lse[b, heads] = torch.softmax(logits, -1) @ v, torch.logsumexp(logits, -1)
    got = rig.out.cpu().double(), rig.lse.cpu().double()
    rig.close()
    return got[0], got[1], out, lse


@pytest.mark.parametrize("page", [1, 2, 3, 5, 6, 7, 12, 15, 17, 20, 24, 33, 100, 255])
@pytest.mark.parametrize("dtype,group", [("f16", 7), ("bf16", 4), ("bf16", 1), ("f16", 8)])
def test_page_sizes(page, dtype, group):
    k = max(2, min(61, 1300 // page))
    w = small("natural", page=page, ctx=page * 90, topk_pages=k, capacity=k + 3, dtype=dtype, batch=2, n_kv_heads=2, n_q_heads=2 * group)
    got, got_lse, want, lse = attend(w, [w.ctx, max(1, w.ctx - w.page * 40 - page // 2)], 0)
    # P carries 22 bits or more, q.k and the sums are fp32: what the fp32 arithmetic of a few thousand terms leaves
    assert float((got - want).norm() / want.norm()) < 1e-6
    assert float((got_lse - lse).abs().max()) < 1e-4


@pytest.mark.parametrize("splits", [1, 3, 64])
def test_splits_and_budgets_beyond_the_staged_entries(splits):
    """2000 pages of 3 tokens: with one split its entries do not fit the staging area."""
    w = small("natural-splits", page=3, ctx=3 * 2500, topk_pages=2000, capacity=2000, batch=1, n_kv_heads=2, n_q_heads=8)
    got, _, want, _ = attend(w, [w.ctx - 1], splits)
    assert float((got - want).norm() / want.norm()) < 1e-6


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_infinities_and_rows_beyond_the_end(dtype):
    """An infinite V element makes its dim infinite and nothing else; what lies beyond the end does not matter."""
    w = small("natural-inf", page=20, ctx=20 * 40, topk_pages=30, capacity=40, dtype=dtype, batch=2, n_kv_heads=2, n_q_heads=8)
    seq = [w.ctx - 3, w.ctx - 25]

    def edit(store):
        for b in range(2):
            flat = store[0, b].permute(0, 2, 1, 3, 4).reshape(w.n_kv_heads, 2, -1, w.head_dim)   # (a copy: rows located, then written)
            page, row = divmod(seq[b], w.page)
            assert flat.shape[2] == w.ctx
            store[0, b, :, page, :, row:] = float("nan")
            store[0, b, :, page + 1:] = float("inf")
        last = (seq[0] - 1) // w.page                    # the last page is always selected
        store[0, 0, 0, last, 1, 0, 5] = float("inf")
        store[0, 0, 1, last, 1, 1, 77] = float("-inf")

    got, got_lse, want, lse = attend(w, seq, 2, edit)
    assert torch.isfinite(got_lse).all() and float((got_lse - lse).abs().max()) < 1e-4
    assert torch.equal(torch.isinf(got), torch.isinf(want)) and not torch.isnan(got).any()
    assert torch.equal(got[torch.isinf(got)], want[torch.isinf(want)])
    ok = torch.isfinite(want)
    assert float((got[ok] - want[ok]).norm() / want[ok].norm()) < 1e-6
