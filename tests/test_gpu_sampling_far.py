"""The distance histogram of sets with a few points far from all others: their
box is too wide for the single-precision bin, and a coarse grid over it has most
points in one cell."""

import numpy as np
import pytest

from paper_1810_04758_amd import datagen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def knn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_04758_amd import api
    api.load()
    return api


@pytest.mark.parametrize("n", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("far", [150.0, 1e4, 1e6, 1e9])
def test_counts_with_far_points(knn, oracle_mod, n, far):
    """One and four points per thread, every bin by double precision."""
    import torch
    for N in (20_000, (1 << 18) + 9):
        D = datagen.uniform(N, n, seed=620 + n)
        D[:3] = far
        print(f"[sampling far] n={n} N={N} far={far}", flush=True)
        idx = knn.build_index(torch.from_numpy(D).cuda())
        s = idx.sampling()
        idx.close()
        ref = oracle_mod.dist_histogram(D, s["hist_sample"], 1.0 / s["bin_width"], 1000)
        assert np.array_equal(s["counts"], ref)
