"""Selection of units of 16385 to 32768 pages, of which only the quads that can hold a selected page are looked at closely: the
result of the size-agnostic kernels at the edges of what the list of quads holds."""
import numpy as np
import pytest
import torch

from paper_2605_18071_amd import workloads as W
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
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
