"""The grid levels where joins with no option set take the run search: an option
that keeps the defaults (queue_grain=-4, the default granularity) runs on them.
At full size their rows are those of the run search, which are compared with the
oracle elsewhere."""

import numpy as np
import pytest

from paper_1810_04758_amd import datagen

pytestmark = pytest.mark.gpu

GRID = dict(queue_grain=-4)
LEVELS = dict(w_factor=1.0, tail_pairs=-1.0)  # no brute-force tail: level after level


@pytest.fixture(scope="module")
def knn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_04758_amd import api
    api.load()
    return api


def _on_levels(st):
    return st["levels"] > 1 or st["lanes_per_query"] > 1


@pytest.mark.parametrize("name,Ks", [("unif2d_50k", [5]), ("expo2d_2m", [1, 32]),
                                     ("expo4d_2m", [8, 64]), ("unif6d_5m", [32]),
                                     ("clustered2d_20m", [16])])
def test_fullsize_both_ways(knn, name, Ks):
    import torch
    D, _, _ = datagen.config_points(name)
    print(f"[grid levels] {name} K={Ks}", flush=True)
    Dd = torch.from_numpy(D).cuda()
    idx = knn.build_index(Dd)
    for K in Ks:
        gi, gd, st = idx.self_join(K, with_stats=True, **GRID)
        assert _on_levels(st)
        ri, rd, st = idx.self_join(K, with_stats=True)
        assert not _on_levels(st)
        assert torch.equal(gi, ri) and torch.equal(gd, rd), K
        del gi, gd, ri, rd
    idx.close()
    del Dd
    torch.cuda.empty_cache()


@pytest.mark.parametrize("name,gen,K", [
    ("unif2d", lambda: datagen.uniform(3001, 2, seed=21), 5),
    ("unif3d", lambda: datagen.uniform(2999, 3, seed=22), 8),
    ("expo4d", lambda: datagen.exponential(4099, 4, seed=23), 16),
    ("unif5d", lambda: datagen.uniform(2050, 5, seed=24), 3),
    ("unif6d", lambda: datagen.uniform(3000, 6, seed=25), 32),
    ("clus2d", lambda: datagen.clustered(5003, seed=26), 16),
    ("expo2d_k64", lambda: datagen.exponential(4001, 2, seed=27), 64),
    ("expo3d_k100", lambda: datagen.exponential(4001, 3, seed=29), 100),
], ids=lambda v: v if isinstance(v, str) else "")
def test_parity_on_the_levels(knn, oracle_mod, name, gen, K):
    import torch
    D = gen()
    print(f"[grid levels] {name} K={K}", flush=True)
    idx = knn.build_index(torch.from_numpy(D).cuda())
    ids, dists, st = idx.self_join(K, with_stats=True, **(GRID if K <= 64 else {}))
    torch.cuda.synchronize()
    idx.close()
    assert _on_levels(st)
    ref_i, ref_d = oracle_mod.knn(D, K)
    assert np.array_equal(ids.cpu().numpy(), ref_i) and np.array_equal(dists.cpu().numpy(), ref_d)


@pytest.mark.parametrize("name,gen,K", [
    ("expo2d", lambda: datagen.exponential(20011, 2, seed=31), 8),
    ("unif6d", lambda: datagen.uniform(6007, 6, seed=32), 8),
], ids=["expo2d", "unif6d"])
def test_graph_replay_of_levels(knn, oracle_mod, name, gen, K):
    """Several levels and the range sizing of 5-6 dimensions replay."""
    import torch
    D = gen()
    N = D.shape[0]
    print(f"[grid levels] replay {name}", flush=True)
    idx = knn.build_index(torch.from_numpy(D).cuda())
    ref_i, ref_d, st_e = idx.self_join(K, with_stats=True, **LEVELS)
    assert st_e["levels"] > 1
    rows = np.arange(0, N, 11)
    oi, od = oracle_mod.knn(D, K, rows=rows)
    assert np.array_equal(ref_i.cpu().numpy()[rows], oi) and np.array_equal(ref_d.cpu().numpy()[rows], od)
    gi = torch.empty((N, K), dtype=torch.int32, device="cuda")
    gd = torch.empty((N, K), dtype=torch.float64, device="cuda")
    for rep in range(4):
        gi.fill_(-1)
        gd.fill_(float("nan"))
        if rep == 2:  # an eager join by the run search in between
            idx.self_join(K + 1)
        _, _, st = idx.self_join(K, ids=gi, dists=gd, with_stats=True, use_graph=1, **LEVELS)
        torch.cuda.synchronize()
        assert torch.equal(gi, ref_i) and torch.equal(gd, ref_d), rep
        assert st["levels"] == st_e["levels"] and st["attempted"] == st_e["attempted"]
    idx.close()
