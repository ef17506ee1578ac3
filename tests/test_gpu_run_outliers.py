"""A few points far from all others: the runs that hold them are handed over
before they cut their columns back at every leaf, so the set takes about as long
as without them; every row stays the oracle's."""

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


def _search_ms(knn, D, K):
    import torch
    idx = knn.build_index(torch.from_numpy(D).cuda())
    ms = []
    for _ in range(4):
        ids, dists, st = idx.self_join(K, with_stats=True)
        ms.append(st["ms_search"][0])
    torch.cuda.synchronize()
    idx.close()
    assert st["levels"] == 1 and st["lanes_per_query"] == 1
    return min(ms), ids.cpu().numpy(), dists.cpu().numpy()


@pytest.mark.parametrize("n,N,K", [(4, 200_000, 32), (5, 50_000, 16), (6, 50_000, 16)])
def test_far_points_do_not_hold_the_join_up(knn, oracle_mod, n, N, K):
    """Without the limit on cuts the three points take 12 to 17 times the whole
    set's search time, with it the set takes 1.3 to 2 times as long."""
    D = datagen.uniform(N, n, seed=820 + n)
    print(f"[run outliers] n={n} N={N} K={K}", flush=True)
    plain, _, _ = _search_ms(knn, D, K)
    D[:3] = 1e4
    far, ids, dists = _search_ms(knn, D, K)
    rows = np.concatenate([np.arange(64), np.linspace(64, N - 1, 200).astype(np.int64)])
    ref_i, ref_d = oracle_mod.knn(D, K, rows=rows)
    assert np.array_equal(ids[rows], ref_i) and np.array_equal(dists[rows], ref_d)
    assert far <= 5 * plain, (plain, far)
