"""Columns of the run search that fill unevenly: stored order decides which half
of a column a neighbour goes to, so points of one curve cell (which keep their
stored order) can put all of them into one half."""

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


def _one_sided(n, N, seed):
    """Two tight groups far enough apart that a first radius around one does not
    reach the other, and one point so far out that both lie in one curve cell.
    Every other four points belong to the first group (places 0-3 and 8-11 of a
    leaf: one half of the columns); the first leaf of a run has one of them
    only, but for the first run of a parent (1024 points).  So a query's half
    column holds 25 entries after its own leaves and 33 after the next one."""
    rng = np.random.default_rng(seed)
    D = rng.random((N, n)) * 1e-3
    i = np.arange(N)
    first = (i % 8 < 4) & ((i % 64 >= 16) | (i % 64 == 0) | (i % 1024 < 64))
    D[~first] += 0.9
    D[0] = 0.0
    D[-1] = 2.0 ** (62 // n)  # as many cells of side 1 a dimension
    return D


@pytest.mark.parametrize("n", [3, 4, 5, 6])
@pytest.mark.parametrize("K", [7, 8, 9, 16, 31, 32, 33, 64])
def test_one_half_takes_all(knn, oracle_mod, n, K):
    import torch
    D = _one_sided(n, 40_001, seed=600 + n)
    rows = np.linspace(0, D.shape[0] - 1, 400).astype(np.int64)
    print(f"[run columns] n={n} K={K}", flush=True)
    idx = knn.build_index(torch.from_numpy(D).cuda())
    ids, dists, st = idx.self_join(K, with_stats=True)
    torch.cuda.synchronize()
    idx.close()
    assert st["levels"] == 1 and st["lanes_per_query"] == 1
    ref_i, ref_d = oracle_mod.knn(D, K, rows=rows)
    assert np.array_equal(ids.cpu().numpy()[rows], ref_i)
    assert np.array_equal(dists.cpu().numpy()[rows], ref_d)
