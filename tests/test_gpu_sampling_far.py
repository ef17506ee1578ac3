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


def _two_groups(N, n, seed):
    D = datagen.uniform(N, n, seed=seed) * 1e-4
    D[N // 2:] += 3.0
    return D


@pytest.mark.parametrize("n", [2, 3, 4])
@pytest.mark.parametrize("name,gen", [
    # by cell; too wide for the cells; a cell that names half of the sample
    ("far100", lambda N, n: np.concatenate([datagen.uniform(N, n, seed=630), np.full((3, n), 1e4)])),
    ("far1e6", lambda N, n: np.concatenate([datagen.uniform(N, n, seed=631), np.full((3, n), 1e8)])),
    ("two_groups", lambda N, n: _two_groups(N, n, seed=632)),
], ids=["far100", "far1e6", "two_groups"])
def test_counts_by_cell_or_pair(knn, n, name, gen):
    """Large sets, by cell or by pair as the cells decide: the same counts as
    the pass over every pair (points given without their box)."""
    import torch
    D = torch.from_numpy(np.ascontiguousarray(gen((1 << 21) + 31, n))).cuda()
    print(f"[sampling far] {name} n={n}", flush=True)
    idx = knn.build_index(D)
    s = idx.sampling()
    idx.close()
    full = knn.dist_histogram(D, torch.from_numpy(s["hist_sample"]).cuda(), 1.0 / s["bin_width"],
                              1000)
    torch.cuda.synchronize()
    full = full.cpu().numpy().view(np.uint64)
    last = int(np.nonzero(s["counts"])[0][-1])
    assert np.array_equal(s["counts"][:last + 1], full[:last + 1])
    assert full[:last + 1].sum() >= 1024 * 500
