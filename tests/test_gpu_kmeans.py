"""The k-means build of the hierarchical index against the oracle, where its screening on the matrix
cores could go wrong: point and centroid counts around the sizes of its blocks and tiles, data whose
differences are small against its magnitude, fp16 subnormals, exact ties."""
import numpy as np
import pytest
import torch

from oracle import kvd_oracle as orc
from tests import helpers as H
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests import gpu_rig as R


def points(kind, units, pages, dtype, gen):
    x = torch.randn(units, pages, 128, device=R.DEV, generator=gen)
    if kind == "offset":                   # a common mean 200 times the spread
        x = 0.05 * x + 10.0 * torch.randn(units, 1, 128, device=R.DEV, generator=gen).sign()
    elif kind == "components":             # dims at and beyond the span that is shifted, of either sign, among ordinary ones
        lo, hi = 1.0, torch.tensor([1.0, 1.5, 3.0, 3.03125, 8.0], device=R.DEV)[torch.arange(128, device=R.DEV) % 5]
        z = lo + (hi - lo) * torch.rand(x.shape, device=R.DEV, generator=gen)
        z[:, 0], z[:, 1] = lo, hi
        size = torch.tensor([100.0, 2.0 ** -12, 2.0 ** -13, 8e3, -30.0, -2.0 ** -12, -1.0], device=R.DEV)[torch.arange(128, device=R.DEV) % 7]
        x = torch.where(torch.arange(128, device=R.DEV) % 3 == 0, x, z * size)
    elif kind == "tiny":                   # fp16: mostly subnormals
        x = 2e-5 * x
    elif kind == "drift":                  # neighbouring pages alike, so that distances fall slowly along the pages
        x = torch.cumsum(0.1 * x, dim=1)
    elif kind == "same":                   # every page the same vector
        x = x[:, :1].expand(-1, pages, -1)
    elif kind == "huge":                   # squared norms beyond fp32
        x = 3e19 * x
    elif kind == "few huge":               # ... of every 50th page only, so that some centroids stay in range
        x[:, 3::50] *= 1e25
    elif kind == "minute":                 # squared norms among the subnormals of fp32, or zero there
        x = 2e-22 * (x[:, :1] + 0.02 * x)
    elif kind == "pairs":                  # every vector 40 times: more equal centroids than are compared one by one
        x = x[:, torch.arange(pages, device=R.DEV) % max(1, pages // 40)]
    return x.to(dtype)


@pytest.mark.parametrize("pages,nc,kind,dtype,seq", [
    (255, 1, "normal", "bf16", (255 * 16, 1)),             # one centroid; a sequence of one page
    (256, 16, "normal", "f16", None),                      # exactly one block of points, one tile of centroids
    (257, 17, "normal", "bf16", None),                     # one point and one centroid more
    (600, 33, "drift", "f16", (600 * 16, 513 * 16 - 5)),   # three tiles: uneven halves
    (300, 300, "normal", "bf16", None),                    # a centroid per page
    (520, 200, "offset", "bf16", None),
    (520, 200, "offset", "f16", None),
    (520, 200, "components", "bf16", (520 * 16, 300 * 16 + 7)),
    (520, 200, "components", "f16", (520 * 16, 300 * 16 + 7)),
    (300, 64, "tiny", "f16", None),
    (300, 64, "tiny", "bf16", None),
    (300, 50, "same", "bf16", None),                       # all distances tie
    (700, 100, "pairs", "f16", None),
    (1100, 20, "same", "bf16", (1100 * 16, 1030 * 16)),    # more open pages than blocks of four
    (300, 5, "huge", "bf16", None),
    (300, 150, "huge", "bf16", None),
    (600, 9, "few huge", "bf16", None),
    (600, 200, "few huge", "bf16", None),
    (300, 5, "minute", "bf16", None),
    (600, 64, "minute", "bf16", None),
])
def test_build_matches_the_oracle_round_by_round(pages, nc, kind, dtype, seq):
    w = small("kmeans", ctx=16 * pages, topk_pages=min(24, pages), capacity=min(60, pages), heavy_count=0, dtype=dtype,
              index_centroids=nc, index_iterations=3)
    rig = R.Rig(w, seq_lens=list(seq) if seq else None, build_index=False)
    gen = torch.Generator(device=R.DEV)
    gen.manual_seed(31_000 + pages * 7 + nc)
    rig.summaries.copy_(points(kind, w.units, pages, w.torch_dtype, gen).view(rig.summaries.shape))
    rig.kvd.build_centroids(0, w.index_iterations, rig.assign_trace[0])
    torch.cuda.synchronize()
    trace = rig.assign_trace.cpu().numpy()[0]
    code, differ = H.dtype_code(w.torch_dtype), 0
    for u in range(w.units):
        b, h = divmod(u, w.n_kv_heads)
        n = -(-rig.seq_lens[b] // w.page)
        x = H.f64(rig.summaries[0, b, h])[:n]
        cent = orc.kmeans_init(x, nc)
        for it in range(w.index_iterations):
            # (the oracle's own distances come from the expanded square, which loses the small differences of
            # "offset" and "tiny": here the sum of squares itself)
            d = np.stack([np.square(x - c).sum(axis=1) for c in cent], axis=1)
            own, gpu = d.argmin(axis=1), trace[it, u, :n].astype(np.int32)
            rows = np.nonzero(own != gpu)[0]
            # both sum 128 squares in 64 bits, in whatever order: 128 x 2^-53 apart at most, with a wide margin
            assert np.all(d[rows, gpu[rows]] <= d[rows].min(axis=1) * (1 + 1e-12)), (u, it, rows[:5])
            differ += len(rows)
            cent = orc.kmeans_update(x, gpu, cent)
        got = rig.centroids[0, b, h].cpu()
        assert np.array_equal(H.bits(got), orc.f64_to_bits(cent, code)), f"centroids of unit {u}"
        start, listed = rig.cluster_start[0, u].cpu().numpy(), rig.cluster_pages[0, u].cpu().numpy()
        last = trace[-1, u, :n]
        assert start[0] == 0 and start[-1] == n and np.all(listed[n:] == -1)
        for c in range(nc):
            assert np.array_equal(listed[start[c]:start[c + 1]], np.nonzero(last == c)[0]), f"cluster {c} of unit {u}"
    assert differ <= 2
    rig.close()
