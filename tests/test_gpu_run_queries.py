"""The run search run by run (k_run_search: more runs than the sets searched
query by query): external query sets, and the rarer data."""

import numpy as np
import pytest

from paper_1810_04758_amd import datagen

pytestmark = pytest.mark.gpu

# queries above which a set is searched run by run
LINE = {2: 192 * 64, 3: 512 * 64, 4: 512 * 64, 5: 512 * 64, 6: 512 * 64}


@pytest.fixture(scope="module")
def knn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_04758_amd import api
    api.load()
    return api


def _queries(S, gen, NQ, n, seed):
    """Queries of another draw, copies of indexed points, and a few far ones on
    both sides of the box."""
    copies, far = NQ // 50, 61
    Q = np.concatenate([gen(NQ - copies - far, n, seed), S[:copies],
                        np.where(np.arange(far)[:, None] % 2, 5.0, -4.0) *
                        (1 + np.arange(far)[:, None]) * (S.max(0) - S.min(0))])
    rng = np.random.default_rng(seed)
    return np.ascontiguousarray(Q[rng.permutation(Q.shape[0])])


def _join_rows(knn, oracle_mod, S, Q, Ks, seed, rows=250):
    import torch
    idx = knn.build_index(torch.from_numpy(S).cuda())
    Qd = torch.from_numpy(Q).cuda()
    for K in Ks:
        print(f"[run queries] n={S.shape[1]} N={S.shape[0]} NQ={Q.shape[0]} K={K}", flush=True)
        ids, dists, st = idx.join(Qd, K, with_stats=True)
        torch.cuda.synchronize()
        assert st["levels"] == 1 and st["lanes_per_query"] == 1
        ids, dists = ids.cpu().numpy(), dists.cpu().numpy()
        rng = np.random.default_rng(seed)
        sel = np.unique(np.concatenate([rng.choice(Q.shape[0], rows, replace=False),
                                        np.argsort(dists[:, -1])[-100:],
                                        np.argsort(dists[:, -1])[:30],
                                        np.arange(Q.shape[0] - 5, Q.shape[0])]))
        ref_i, ref_d = oracle_mod.knn_rs(S, Q, K, rows=sel)
        assert np.array_equal(ids[sel], ref_i) and np.array_equal(dists[sel], ref_d)
    idx.close()


@pytest.mark.parametrize("n", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("kind", ["uniform", "exponential"])
def test_query_sets(knn, oracle_mod, n, kind):
    gen = getattr(datagen, kind)
    S = gen(30_000, n, 840 + n)
    for NQ in (LINE[n] + 1, LINE[n] + 2047):
        _join_rows(knn, oracle_mod, S, _queries(S, gen, NQ, n, 850 + n), (1, 8, 16, 32, 33, 64),
                   860 + n)


@pytest.mark.parametrize("n,NQ,N", [(5, 65_536, 4 * 65_536), (5, 65_537, 4 * 65_537),
                                    (6, 34_001, 4 * 34_001), (6, 34_001, 4 * 34_001 - 1),
                                    (6, 131_072, 4 * 131_072), (6, 131_073, 4 * 131_073)])
def test_queries_few_beside_the_points(knn, oracle_mod, n, NQ, N):
    """Both sides of the lines up to which they are searched one by one."""
    S = datagen.exponential(N, n, seed=895)
    Q = _queries(S, datagen.exponential, NQ, n, 896)
    assert Q.shape[0] == NQ
    _join_rows(knn, oracle_mod, S, Q, (8, 32, 33, 64), 897)


@pytest.mark.parametrize("n", [2, 4, 6])
def test_query_sets_of_few_points(knn, oracle_mod, n):
    """Fewer indexed points than a run, and K = N."""
    S = datagen.uniform(64, n, seed=870 + n)
    Q = _queries(S, lambda m, d, s: datagen.uniform(m, d, seed=s), LINE[n] + 130, n, 880)
    _join_rows(knn, oracle_mod, S[:40], Q, (1, 40), 881)
    _join_rows(knn, oracle_mod, S, Q, (17, 64), 882)


def test_clustered_query_set(knn, oracle_mod):
    S = datagen.clustered(200_000, seed=25)
    Q = np.concatenate([datagen.clustered(100_000, seed=26), [[1e4, 1e4], [-1e5, 3.0]]])
    _join_rows(knn, oracle_mod, S, Q, (4, 16, 50), 883, rows=1200)


RARE = [
    ("same2d", lambda: np.full((13_000, 2), 3.25)),
    ("line2d", lambda: np.stack([np.linspace(0, 1, 14_000) ** 4, np.zeros(14_000)], 1)),
    ("overflow2d", lambda: (datagen.uniform(13_000, 2, seed=884) - 50.0) * 1e158),
    ("two_scales2d", lambda: np.concatenate([datagen.uniform(9_000, 2, seed=885),
                                             datagen.uniform(9_000, 2, seed=886) * 1e-9 + 7.0])),
    ("offset3d", lambda: datagen.uniform(34_000, 3, seed=887) * 1e-3 + 3e6),
    ("underflow3d", lambda: datagen.uniform(34_000, 3, seed=888) * 1e-166),
    ("overflow4d", lambda: (datagen.uniform(34_000, 4, seed=889) - 50.0) * 1e158),
    ("offset5d", lambda: datagen.uniform(34_000, 5, seed=890) * 1e-2 + 1e5),
    ("far_pair5d", lambda: np.concatenate([datagen.uniform(20_000, 5, seed=891) * 1e-6,
                                           datagen.uniform(20_037, 5, seed=892) * 1e-6 + 9.0])),
    ("underflow6d", lambda: datagen.uniform(34_000, 6, seed=893) * 1e-166),
    ("overflow6d", lambda: (datagen.uniform(34_000, 6, seed=894) - 50.0) * 1e158),
]


@pytest.mark.parametrize("name,gen", RARE, ids=[r[0] for r in RARE])
def test_rare_data_run_by_run(knn, oracle_mod, name, gen):
    import torch
    D = np.ascontiguousarray(gen())
    assert D.shape[0] > LINE[D.shape[1]]
    idx = knn.build_index(torch.from_numpy(D).cuda())
    rows = np.unique(np.linspace(0, D.shape[0] - 1, 300).astype(np.int64))
    for K in (3, 8, 16, 24, 32, 64):
        print(f"[run rare] {name} K={K}", flush=True)
        ids, dists, st = idx.self_join(K, with_stats=True)
        torch.cuda.synchronize()
        assert st["levels"] == 1 and st["lanes_per_query"] == 1
        ref_i, ref_d = oracle_mod.knn(D, K, rows=rows)
        assert np.array_equal(ids.cpu().numpy()[rows], ref_i)
        assert np.array_equal(dists.cpu().numpy()[rows], ref_d)
    idx.close()
