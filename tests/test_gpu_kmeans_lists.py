"""Rounds after the first collect a point's candidates in one sweep, in a list of 24 that is filtered afterwards: more equal
centroids than are compared one by one but fewer than the list holds, and more than it holds (the sweep is made again and
the page left to the comparison with every centroid), over more rounds than the lists need to settle."""
import numpy as np
import pytest
import torch

import tests.test_gpu_kmeans as K
from tests import helpers as H
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests import gpu_rig as R


@pytest.mark.parametrize("pages,nc,kind,dtype", [
    (700, 250, "pairs", "bf16"),            # 15 equal centroids each: filtered, then more than eight are left
    (700, 690, "pairs", "f16"),             # 41 each: the list is too short
    (1030, 400, "drift", "bf16"),           # neighbours alike: candidates come in rising order
])
def test_lists_of_one_sweep(pages, nc, kind, dtype):
    K.test_build_matches_the_oracle_round_by_round(pages, nc, kind, dtype, None)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_pages_of_a_cluster_that_is_no_number(dtype):
    """A page that is no number goes to the first cluster, whose centroid is none from then on: the pages that it had find
    the nearest of the others, wherever among the tiles of centroids that is."""
    pages, nc = 700, 100
    w = small("kmeans-nan", ctx=16 * pages, topk_pages=24, capacity=60, heavy_count=0, dtype=dtype, index_centroids=nc, index_iterations=3)
    rig = R.Rig(w, build_index=False)
    gen = torch.Generator(device=R.DEV)
    gen.manual_seed(37)
    x = K.points("normal", w.units, pages, w.torch_dtype, gen)
    x[:, 400, 5] = float("nan")
    rig.summaries.copy_(x.view(rig.summaries.shape))
    rig.kvd.build_centroids(0, w.index_iterations, rig.assign_trace[0])
    torch.cuda.synchronize()
    trace = rig.assign_trace.cpu().numpy()[0]
    for u in range(w.units):
        x = H.f64(rig.summaries[0].view(w.units, pages, 128)[u])
        numbers = np.arange(pages) != 400
        cent = x[((np.arange(nc) + 0.5) * pages / nc).astype(int)]
        for it in range(w.index_iterations):
            d = np.stack([np.square(x - c).sum(axis=1) for c in cent], axis=1)
            d[np.isnan(d)] = np.inf
            gpu = trace[it, u]
            assert gpu[400] == 0
            # (the two sums of 128 squares: as in the test of whole builds)
            far = np.nonzero(numbers & ~(d[np.arange(pages), gpu] <= d.min(axis=1) * (1 + 1e-12)))[0]
            assert far.size == 0, (u, it, far, gpu[far], d.argmin(axis=1)[far])
            cent = np.stack([x[gpu == c].mean(axis=0) if (gpu == c).any() else cent[c] for c in range(nc)])
    rig.close()
