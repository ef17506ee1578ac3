"""What a measured setting does to later joins: one with no option set takes the
grid levels with the cached setting where they were faster than the run search,
and the run search otherwise; joins on the grid levels take the cached setting
in any case."""

import numpy as np
import pytest

from paper_1810_04758_amd import datagen

pytestmark = pytest.mark.gpu

# a workload class that no other test uses: 5 dimensions, N in [4^5, 4^6), K in [32, 63]
N, DIMS, K = 3500, 5, 40
CLASS = (DIMS, 5, 5)


@pytest.fixture(scope="module")
def knn():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_04758_amd import api
    api.load()
    return api


def _load(knn, tmp_path, zorder, w_factor=1.75, fields=11):
    line = [*CLASS, w_factor, 1.5, 0, -1, 2.5e8, 0, zorder, 8][:fields]
    path = tmp_path / "tune.txt"
    path.write_text(" ".join(str(v) for v in line) + "\n")
    knn.autotune_load(str(path))


def _stats(idx, K, **o):
    import torch
    ids, dists, st = idx.self_join(K, with_stats=True, **o)
    torch.cuda.synchronize()
    return ids.cpu().numpy(), dists.cpu().numpy(), st


@pytest.mark.parametrize("zorder,fields,levels", [(-2, 11, True), (-3, 11, False), (-1, 11, False),
                                                  (-1, 10, False)])
def test_default_joins_take_the_faster_way(knn, oracle_mod, tmp_path, zorder, fields, levels):
    import torch
    print(f"[autotune] zorder field {zorder} of {fields}", flush=True)
    D = datagen.exponential(N, DIMS, seed=830)
    idx = knn.build_index(torch.from_numpy(D).cuda())
    try:
        _load(knn, tmp_path, zorder, fields=fields)
        ids, dists, st = _stats(idx, K)
        side = 1.75 * idx.eps_min(K)
        assert (st["lanes_per_query"] > 1 or st["levels"] > 1) == levels
        assert (st["cell_width"][0] == side) == levels
        ref_i, ref_d = oracle_mod.knn(D, K)
        assert np.array_equal(ids, ref_i) and np.array_equal(dists, ref_d)
        # on the grid levels the cached side holds in any case
        ids, dists, st = _stats(idx, K, queue_grain=-4)
        assert st["cell_width"][0] == side
        assert np.array_equal(ids, ref_i) and np.array_equal(dists, ref_d)
        # a query set goes the same way
        Q = torch.from_numpy(D[:200].copy()).cuda()
        qi, qd, st = idx.join(Q, K, with_stats=True)
        torch.cuda.synchronize()
        assert (st["cell_width"][0] == side) == levels
        ref_i, ref_d = oracle_mod.knn_rs(D, D[:200], K)
        assert np.array_equal(qi.cpu().numpy(), ref_i) and np.array_equal(qd.cpu().numpy(), ref_d)
        # the graph's replay too
        gi, gd = torch.empty((N, K), dtype=torch.int32, device="cuda"), \
            torch.empty((N, K), dtype=torch.float64, device="cuda")
        for _ in range(3):
            gi.zero_(), gd.zero_()
            idx.self_join(K, ids=gi, dists=gd, use_graph=1)
            torch.cuda.synchronize()
            assert np.array_equal(gi.cpu().numpy(), ids) and np.array_equal(gd.cpu().numpy(), dists)
        # what was loaded is saved again
        path = str(tmp_path / "saved.txt")
        knn.autotune_save(path)
        lines = [l.split() for l in open(path)]
        mine = [l for l in lines if tuple(map(int, l[:3])) == CLASS]
        assert len(mine) == 1 and int(mine[0][9]) == zorder and float(mine[0][3]) == 1.75
    finally:
        idx.close()
        _load(knn, tmp_path, -1, w_factor=1.0)


def test_large_K_takes_the_cached_setting(knn, tmp_path):
    import torch
    idx = knn.build_index(torch.from_numpy(datagen.exponential(N, DIMS, seed=831)).cuda())
    path = tmp_path / "tune.txt"
    path.write_text("5 6 5 1.75 1.5 0 -1 2.5e8 0 -3 8\n")
    knn.autotune_load(str(path))
    _, _, st = _stats(idx, 100)
    assert st["cell_width"][0] == 1.75 * idx.eps_min(100)
    path.write_text("5 6 5 1.0 1.5 0 -1 2.5e8 0 -1 8\n")
    knn.autotune_load(str(path))
    idx.close()


def test_measured_choice(knn, tmp_path):
    """The tuner's answer is what the next join with no option set does."""
    import torch
    print("[autotune] measured", flush=True)
    idx = knn.build_index(torch.from_numpy(datagen.uniform(N, DIMS, seed=832)).cuda())
    try:
        assert idx.autotune(100)["run_search"] == 0
        r = idx.autotune(K)
        assert r["run_search"] in (1, -1)
        _, _, st = _stats(idx, K)
        if r["run_search"] == 1:
            assert st["levels"] == 1 and st["lanes_per_query"] == 1
        else:
            assert st["cell_width"][0] == r["w_factor"] * idx.eps_min(K)
    finally:
        idx.close()
        _load(knn, tmp_path, -1, w_factor=1.0)
