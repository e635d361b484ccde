"""Rounds after the first collect a point's candidates in one sweep, in a list of 24 that is filtered afterwards: more equal
centroids than are compared one by one but fewer than the list holds, and more than it holds (the sweep is made again and
the page left to the comparison with every centroid), over more rounds than the lists need to settle."""
import pytest
import torch

import tests.test_gpu_kmeans as K

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pages,nc,kind,dtype", [
    (700, 250, "pairs", "bf16"),            # 15 equal centroids each: filtered, then more than eight are left
    (700, 690, "pairs", "f16"),             # 41 each: the list is too short
    (1030, 400, "drift", "bf16"),           # neighbours alike: candidates come in rising order
])
def test_lists_of_one_sweep(pages, nc, kind, dtype):
    K.test_build_matches_the_oracle_round_by_round(pages, nc, kind, dtype, None)
