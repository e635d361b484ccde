"""The index build over page sizes on both sides of what one block covers (64 tokens), bit for bit."""
import numpy as np
import pytest
import torch

from oracle import kvd_oracle as orc
from tests import helpers as H
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests import gpu_rig as R


@pytest.mark.parametrize("page,pages", [(1, 130), (4, 33), (6, 21), (24, 7), (33, 5), (63, 3), (64, 3), (65, 3), (128, 2), (200, 3), (256, 2)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_summaries_bits(page, pages, dtype):
    w = small("summaries", page=page, ctx=page * pages, topk_pages=2, capacity=2, dtype=dtype, batch=3)
    # a full sequence, a ragged one, and one that ends inside the first page: the pages beyond the end are zero
    lens = [page * pages, max(1, page * (pages // 2) + page // 3), max(1, page // 2)]
    rig = R.Rig(w, seq_lens=lens, build_index=False)
    rig.summaries.fill_(7.0)
    rig.kvd.build_summaries(0)
    torch.cuda.synchronize()
    for b in range(w.batch):
        for h in range(w.n_kv_heads):
            want = orc.page_summaries(H.f64(rig.store[0, b, h, :, 0]).reshape(-1, w.head_dim), page, lens[b], H.dtype_code(w.torch_dtype))
            got = rig.summaries[0, b, h].cpu()
            n = want.shape[0]
            assert np.array_equal(H.bits(got[:n]), orc.f64_to_bits(want, H.dtype_code(w.torch_dtype))), (b, h)
            assert not got[n:].any()
    rig.close()
