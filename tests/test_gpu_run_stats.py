"""Join statistics of the run search: the candidates of every query count, those
of queries searched one by one included."""

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


@pytest.mark.parametrize("n,N,K", [(2, 700, 64), (2, 12_000, 8), (3, 30_000, 16), (4, 3000, 1),
                                   (5, 3000, 40), (6, 30_000, 64)])
def test_candidates_of_small_sets(knn, n, N, K):
    """Every query evaluates its own leaf and at least its K neighbours."""
    import torch
    idx = knn.build_index(torch.from_numpy(datagen.uniform(N, n, seed=800 + n)).cuda())
    _, _, st = idx.self_join(K, with_stats=True)
    idx.close()
    print(f"[run stats] n={n} N={N} K={K} {st['cand_per_query'][0]}", flush=True)
    assert K + 1 <= st["cand_per_query"][0] <= 4 * N + 64


def test_candidates_of_far_queries(knn):
    """Queries far from the set evaluate at least the K they return."""
    import torch
    idx = knn.build_index(torch.from_numpy(datagen.uniform(20_000, 3, seed=810)).cuda())
    Q = torch.full((100, 3), 1e4, dtype=torch.float64, device="cuda")
    _, _, st = idx.join(Q, 33, with_stats=True)
    idx.close()
    assert 33 <= st["cand_per_query"][0] <= 4 * 20_000 + 64
