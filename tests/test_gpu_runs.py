"""The run search (default options, K <= 64): ids identical
and distances bit-identical to the oracle on every row, at the sizes where its
leaves (16 points), runs (64 queries) and box levels (64 children) begin and
end, at the K where its register lists change size, and on data that takes its
rarer paths: exact ties and duplicates (order by id), runs that reach more
leaves than their list holds, radii that start too small or infinite, squared
distances that overflow or underflow, queries outside the points' box."""

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


def _self(knn, D, K, **opts):
    import torch
    idx = knn.build_index(torch.from_numpy(D).cuda())
    ids, dists, st = idx.self_join(K, with_stats=True, **opts)
    torch.cuda.synchronize()
    idx.close()
    # one level, no lanes shared by a query, no tail: the run search ran
    assert st["levels"] == 1 and st["lanes_per_query"] == 1 and st["tail_queries"] == 0
    return ids.cpu().numpy(), dists.cpu().numpy()


def _check(knn, oracle_mod, D, K):
    ids, dists = _self(knn, D, K)
    ref_i, ref_d = oracle_mod.knn(D, K)
    bad = np.nonzero((ids != ref_i).any(axis=1) | (dists != ref_d).any(axis=1))[0]
    assert bad.size == 0, (f"{bad.size} rows differ, first {bad[0]}: {ids[bad[0]]} {dists[bad[0]]} "
                           f"want {ref_i[bad[0]]} {ref_d[bad[0]]}")


@pytest.mark.parametrize("n", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("N", [2, 15, 16, 17, 63, 64, 65, 1023, 1024, 1025, 4097])
def test_sizes(knn, oracle_mod, n, N):
    print(f"[runs sizes] N={N} n={n}", flush=True)
    for K in sorted({1, min(N - 1, 7), min(N - 1, 64)}):
        _check(knn, oracle_mod, datagen.exponential(N, n, seed=100 + N), K)


@pytest.mark.parametrize("K", [1, 8, 9, 16, 17, 32, 33, 63, 64])
def test_register_lists(knn, oracle_mod, K):
    print(f"[runs lists] K={K}", flush=True)
    for n in (2, 3, 4, 5, 6):
        _check(knn, oracle_mod, datagen.uniform(3000 + K, n, seed=200 + K), K)


def test_third_box_level(knn):
    """65 groups of 64 leaves (a third level of boxes) and clustered data
    against the grid levels' result."""
    import torch
    D = datagen.clustered(64 * 64 * 16 + 1, seed=301)
    print(f"[runs levels] N={D.shape[0]}", flush=True)
    ids, dists = _self(knn, D, 12)
    idx = knn.build_index(torch.from_numpy(D).cuda())
    gi, gd = idx.self_join(12, zorder=-1)
    torch.cuda.synchronize()
    idx.close()
    assert np.array_equal(ids, gi.cpu().numpy()) and np.array_equal(dists, gd.cpu().numpy())


def _spread(n, seed):
    """A dense cluster of 2e4 points and 130 points far around it: their balls
    reach most of the cluster's leaves."""
    rng = np.random.default_rng(seed)
    far = rng.standard_normal((130, n))
    far = 50.0 * far / np.linalg.norm(far, axis=1, keepdims=True)
    return np.concatenate([rng.standard_normal((20000, n)), far])


RARE = [
    ("lattice2d", lambda: datagen.lattice(40, 2), 12),
    ("lattice3d", lambda: datagen.lattice(11, 3), 33),
    ("lattice4d", lambda: datagen.lattice(6, 4), 64),
    ("lattice6d", lambda: datagen.lattice(4, 6), 40),
    ("dyadic", lambda: datagen.dyadic(3000, 2, seed=302, bits=3, span=4), 20),
    ("copies", lambda: np.concatenate([datagen.uniform(300, 3, seed=303)] * 9), 16),
    ("same", lambda: np.full((700, 2), 3.25), 40),
    ("line", lambda: np.stack([np.linspace(0, 1, 2000) ** 4, np.zeros(2000)], 1), 8),
    ("offset", lambda: datagen.uniform(2500, 3, seed=304) * 1e-3 + 3e6, 10),
    ("same5d", lambda: np.full((500, 5), -7.5), 24),
    ("offset5d", lambda: datagen.uniform(2500, 5, seed=311) * 1e-2 + 1e5, 12),
    ("overflow", lambda: (datagen.uniform(400, 2, seed=305) - 50.0) * 1e158, 24),
    ("overflow4d", lambda: (datagen.uniform(400, 4, seed=312) - 50.0) * 1e158, 24),
    ("underflow", lambda: datagen.uniform(500, 3, seed=306) * 1e-166, 24),
    ("underflow6d", lambda: datagen.uniform(500, 6, seed=313) * 1e-166, 10),
    ("two_scales", lambda: np.concatenate([datagen.uniform(1500, 2, seed=307),
                                           datagen.uniform(1500, 2, seed=308) * 1e-9 + 7.0]), 16),
    ("spread2d", lambda: _spread(2, 309), 30),
    ("spread4d", lambda: _spread(4, 310), 64),
    ("spread6d", lambda: _spread(6, 314), 20),
    # two clusters far apart in one run: the matrix filter's rounding is
    # coarse against their spacing
    ("far_pair5d", lambda: np.concatenate([datagen.uniform(1000, 5, seed=315) * 1e-6,
                                           datagen.uniform(1037, 5, seed=316) * 1e-6 + 9.0]), 16),
]


@pytest.mark.parametrize("name,gen,K", RARE, ids=[r[0] for r in RARE])
def test_rare_paths(knn, oracle_mod, name, gen, K):
    D = np.ascontiguousarray(gen())
    print(f"[runs rare] {name} N={D.shape[0]} n={D.shape[1]} K={K}", flush=True)
    _check(knn, oracle_mod, D, K)


@pytest.mark.parametrize("n,NQ,K", [(2, 1, 5), (2, 64, 64), (3, 1501, 17), (4, 65, 8), (4, 700, 40),
                                    (5, 130, 12), (6, 900, 33)])
def test_query_set(knn, oracle_mod, n, NQ, K):
    import torch
    S = datagen.exponential(3000, n, seed=400 + n)
    Q = np.concatenate([datagen.exponential(NQ, n, seed=401 + n)[:NQ - NQ // 3],
                        S[:NQ // 6], np.full((NQ // 3 - NQ // 6, n), -2.0) * np.arange(1, NQ // 3 - NQ // 6 + 1)[:, None]])
    print(f"[runs query] NQ={Q.shape[0]} n={n} K={K}", flush=True)
    idx = knn.build_index(torch.from_numpy(S).cuda())
    ids, dists, st = idx.join(torch.from_numpy(Q).cuda(), K, with_stats=True)
    torch.cuda.synchronize()
    assert st["levels"] == 1 and st["lanes_per_query"] == 1
    ref_i, ref_d = oracle_mod.knn_rs(S, Q, K)
    assert np.array_equal(ids.cpu().numpy(), ref_i) and np.array_equal(dists.cpu().numpy(), ref_d)
    # K = N: every point
    s = datagen.uniform(40, n, seed=402)
    small = knn.build_index(torch.from_numpy(s).cuda())
    ids, dists = small.join(torch.from_numpy(Q).cuda(), 40)
    torch.cuda.synchronize()
    ref_i, ref_d = oracle_mod.knn_rs(s, Q, 40)
    assert np.array_equal(ids.cpu().numpy(), ref_i) and np.array_equal(dists.cpu().numpy(), ref_d)
    small.close()
    idx.close()


def test_options_keep_the_grid_levels(knn):
    """Any option of the grid levels runs on them, with the same result."""
    import torch
    D = datagen.exponential(5000, 3, seed=500)
    ids, dists = _self(knn, D, 10)
    idx = knn.build_index(torch.from_numpy(D).cuda())
    for o in (dict(w_factor=1.0), dict(lanes_per_query=8), dict(schedule=1), dict(tail_pairs=-1.0),
              dict(zorder=1), dict(predict_fail=-1)):
        gi, gd, st = idx.self_join(10, with_stats=True, **o)
        torch.cuda.synchronize()
        assert st["lanes_per_query"] > 1, o
        assert np.array_equal(ids, gi.cpu().numpy()) and np.array_equal(dists, gd.cpu().numpy()), o
    idx.close()


@pytest.mark.parametrize("n,K", [(2, 1), (2, 20), (2, 64), (3, 33), (4, 8), (6, 64)])
def test_far_queries_one_by_one(knn, oracle_mod, n, K):
    """Runs that reach across the whole set are searched query by query: all
    of a dense cluster at nearly one distance (cut back by bisection), the same
    at exactly one distance (more equal entries than the list holds, so by id),
    and an ordinary set searched from far away."""
    import torch
    rng = np.random.default_rng(700 + n)
    far = rng.standard_normal((150, n))
    far *= 100.0 / np.linalg.norm(far, axis=1, keepdims=True)
    near = rng.standard_normal((20_000, n)) * 1e-3
    for name, D in (("cluster", near), ("duplicates", np.zeros((3000, n))),
                    ("uniform", datagen.uniform(30_000, n, seed=701))):
        print(f"[runs far queries] {name} n={n} K={K}", flush=True)
        D = np.ascontiguousarray(np.concatenate([D, far]))
        _check(knn, oracle_mod, D, K)
        Q = np.ascontiguousarray(far[:131] * 3.0)
        idx = knn.build_index(torch.from_numpy(D).cuda())
        i, d = idx.join(torch.from_numpy(Q).cuda(), K)
        torch.cuda.synchronize()
        idx.close()
        ref_i, ref_d = oracle_mod.knn_rs(D, Q, K)
        assert np.array_equal(i.cpu().numpy(), ref_i) and np.array_equal(d.cpu().numpy(), ref_d)


def _check_rows(knn, oracle_mod, D, K, count=600):
    N = D.shape[0]
    rows = np.linspace(0, N - 1, count).astype(np.int64)
    ids, dists = _self(knn, D, K)
    ref_i, ref_d = oracle_mod.knn(D, K, rows=rows)
    assert np.array_equal(ids[rows], ref_i) and np.array_equal(dists[rows], ref_d)


@pytest.mark.parametrize("n,N", [(2, 192 * 64), (2, 192 * 64 + 1), (2, 20_001), (3, 512 * 64),
                                 (3, 512 * 64 + 1), (3, 40_000), (4, 512 * 64 + 1), (4, 40_001),
                                 (5, 512 * 64 + 1), (5, 45_000), (6, 512 * 64 + 1), (6, 45_000)])
def test_run_by_run(knn, oracle_mod, n, N):
    """Sets of few runs are searched query by query, larger ones run by run:
    both sides of that line, over the register lists."""
    for gen in (datagen.uniform, datagen.exponential):
        D = gen(N, n, seed=900 + n)
        for K in (1, 8, 9, 16, 17, 32, 33, 64):
            print(f"[runs run by run] {gen.__name__} n={n} N={N} K={K}", flush=True)
            _check_rows(knn, oracle_mod, D, K)


@pytest.mark.parametrize("name,gen", [
    ("lattice2d", lambda: datagen.lattice(150, 2)),
    ("lattice3d", lambda: datagen.lattice(33, 3)),
    ("lattice4d", lambda: datagen.lattice(14, 4)),
    ("lattice5d", lambda: datagen.lattice(9, 5)),
    ("lattice6d", lambda: datagen.lattice(6, 6)),
    ("rounded2d", lambda: np.round(datagen.uniform(30_000, 2, seed=910), 0) / 10),
    ("duplicates3d", lambda: np.concatenate([datagen.uniform(9_000, 3, seed=911)] * 4)),
    ("huge3d", lambda: datagen.exponential(40_000, 3, seed=912) * 1e153),
    ("tiny2d", lambda: datagen.exponential(20_000, 2, seed=913) * 1e-160),
    ("far_pair4d", lambda: np.concatenate([datagen.uniform(40_000, 4, seed=914),
                                           np.full((2, 4), 1e7)])),
], ids=lambda v: v if isinstance(v, str) else "")
def test_rare_paths_run_by_run(knn, oracle_mod, name, gen):
    D = np.ascontiguousarray(gen())
    for K in (4, 20, 64):
        print(f"[runs rare paths, run by run] {name} K={K}", flush=True)
        _check_rows(knn, oracle_mod, D, K)
