"""Attention over keys and values chosen for their arithmetic (probabilities far below one, logits of minus infinity),
against 64-bit sums of the same selection."""
import math

import pytest
import torch

from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests import gpu_rig as R

D = 128


def attend(page, dtype, heads, fill, splits=1):
    """(output, log-sum-exp) of the GPU and in 64 bits, [heads, ...], of one sequence and one KV head whose 30 selected
    pages hold what fill(q [heads, D], k [tokens, D], v [tokens, D]) writes into q, k and v (zeros before)."""
    w = small("values", page=page, ctx=page * 30, topk_pages=30, capacity=30, dtype=dtype, batch=1, n_kv_heads=1, n_q_heads=heads)
    rig = R.Rig(w, attn_splits=splits, build_index=False)
    q = torch.zeros(heads, D, dtype=torch.float64)
    k, v = (torch.zeros(30 * page, D, dtype=torch.float64) for _ in range(2))
    fill(q, k, v)
    q, k, v = (x.to(w.torch_dtype) for x in (q, k, v))
    rig.store[0, 0, 0, :, 0] = k.view(30, page, D)
    rig.store[0, 0, 0, :, 1] = v.view(30, page, D)
    rig.sel_pages.copy_(torch.arange(30, dtype=torch.int32).view(1, 30))
    rig.kvd.cache_resolve(0, 0, rig.sel_pages, rig.sel_slots)
    rig.kvd.sparse_decode_attn(0, q.to(R.DEV).view(1, heads, D), rig.sel_pages, rig.sel_slots, rig.out, rig.lse)
    torch.cuda.synchronize()
    got = rig.out[0].double().cpu(), rig.lse[0].double().cpu()
    rig.close()
    # (the products in the order of fp32, so that what overflows there does here; the sums in 64 bits)
    logits = (q.float() @ k.float().T).double() / math.sqrt(D)
    return got, (torch.softmax(logits, -1) @ v.double(), torch.logsumexp(logits, -1))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("page", [6, 20])
@pytest.mark.parametrize("log2p", [-20, -50, -90])
@pytest.mark.parametrize("at", [0, 15])
def test_vanishing_probabilities_over_natural_pages_keep_their_weight(page, dtype, log2p, at):
    """One token of a tile has all the weight and no value; the others' probabilities are 2^log2p, and the output is theirs."""
    gen = torch.Generator().manual_seed(7)
    few = [t for t in range(16) if t != at]

    def fill(q, k, v):
        q[:, 0] = torch.tensor([4.0, 5.0, 4.0])
        k[:, 0] = log2p * math.log(2.0) * math.sqrt(D) / 4.0
        k[at, 0] = 0.0
        v[few] = torch.randn(15, D, generator=gen, dtype=torch.float64)
        v[few[3], 5] = math.inf

    (out, lse), (want, want_lse) = attend(page, dtype, 3, fill)
    assert torch.equal(torch.isinf(out), torch.isinf(want)) and torch.isinf(want[:, 5]).all()
    ok = torch.isfinite(want)
    assert ok.sum() == 3 * (D - 1)
    # an exponent (1.25 log2p for the second head) has two roundings of 2^-24 of itself, exp2f and the sums a few of 2^-23
    assert float(((out - want)[ok] / want[ok].abs().max()).abs().max()) < 1.25 * abs(log2p) * 2 * 2 ** -24 + 1e-6
    assert float((lse - want_lse).abs().max()) < 1e-6


@pytest.mark.parametrize("dtype,heads", [("f16", 1), ("f16", 7), ("bf16", 4)])
@pytest.mark.parametrize("page,splits", [(5, 1), (24, 3)])
def test_logits_of_every_spread_over_natural_pages(page, splits, dtype, heads):
    """Tiles whose probabilities span few and many powers of two, mixed: the first head's logits differ by tenths, the
    last one's by up to a hundred."""
    gen = torch.Generator().manual_seed(11)

    def fill(q, k, v):
        q[:] = torch.randn(heads, D, generator=gen, dtype=torch.float64) * torch.linspace(0.1, 15.0, heads, dtype=torch.float64)[:, None]
        k[:] = torch.randn(k.shape, generator=gen, dtype=torch.float64)
        v[:] = torch.randn(k.shape, generator=gen, dtype=torch.float64)

    (out, lse), (want, want_lse) = attend(page, dtype, heads, fill, splits)
    # logits of up to 60 x log2(e), rounded once in q.k (a sum of 128 products) and once or twice in the exponent
    assert float(((out - want).norm(dim=1) / want.norm(dim=1)).max()) < 90 * 4 * 2 ** -24
    assert float((lse - want_lse).abs().max()) < 90 * 4 * 2 ** -24


@pytest.mark.parametrize("page", [16, 8, 20, 64])
@pytest.mark.parametrize("dtype,which", [("bf16", "one head"), ("bf16", "all heads"), ("f16", "all heads")])
@pytest.mark.parametrize("splits", [1, 3])
def test_logits_of_minus_infinity_have_no_weight(page, dtype, which, splits):
    """The first 150 tokens, and with them the first tile of every wave of the first split, have a logit of minus infinity
    in one head or in all of them: the output is that of the other tokens."""
    gen = torch.Generator().manual_seed(13)

    def fill(q, k, v):
        for x in (q, k, v):
            x[:] = torch.randn(x.shape, generator=gen, dtype=torch.float64)
        q[:, 0], k[:, 0] = 0.0, 0.0
        if which == "one head":
            q[1, 0], k[:150, 0] = -3e38, 3e38           # finite factors, the product beyond fp32
        else:
            q[:, 0], k[:150, 0] = 1.0, -math.inf

    (out, lse), (want, want_lse) = attend(page, dtype, 3, fill, splits)
    assert torch.isfinite(want).all() and torch.isfinite(out).all() and torch.isfinite(lse).all()
    # probabilities multiply V in 16 bits (two parts of them for bf16) over pages kept as tiles
    assert float(((out - want).norm(dim=1) / want.norm(dim=1)).max()) < (2 ** -11 if dtype == "f16" else 2 ** -16)
    assert float((lse - want_lse).abs().max()) < 1e-5


@pytest.mark.parametrize("page", [16, 20])
@pytest.mark.parametrize("dtype,size", [("f16", 3e2), ("f16", 3e4), ("bf16", 1e6), ("bf16", 1e15)])
def test_logits_beyond_the_integers_of_fp32(page, dtype, size):
    """Logits of 1e6 to 1e31: the largest token takes all, whatever the rounding of its logit."""
    gen = torch.Generator().manual_seed(17)

    def fill(q, k, v):
        for x in (q, k):
            x[:] = size * torch.rand(x.shape, generator=gen, dtype=torch.float64)
        v[:] = torch.randn(v.shape, generator=gen, dtype=torch.float64)
        k[3::7] *= torch.linspace(0.5, 0.9, k[3::7].shape[0], dtype=torch.float64)[:, None]

    (out, lse), (want, want_lse) = attend(page, dtype, 4, fill)
    assert torch.isfinite(out).all() and torch.isfinite(lse).all()
    assert float((lse / want_lse - 1).abs().max()) < 1e-6
    assert float(((out - want).norm(dim=1) / want.norm(dim=1)).max()) < 2 ** -16
