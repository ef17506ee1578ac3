"""The benchmark's roofline of the run search: figures of a uniform 6-D join
(5e6 points, K=32, 24 thousand candidates a query, 36 ms), whose candidates the
matrix cores reject, stay below the peaks they are set against."""

import importlib.util
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _bench():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def _stats(N, cand, ms, lanes=1):
    zero = [0]
    return dict(levels=1, lanes_per_query=lanes, attempted=[N], failed=zero, deferred=zero,
                heavy_queries=zero, heavy_failed=zero, heavy_cand=zero, cand_per_query=[cand],
                ms_search=[ms])


def test_filtered_candidates_are_matrix_work():
    b = _bench()
    roof = b.roofline_of([(6, 32, _stats(5_000_000, 24_000, 36.0))])
    fracs = [roof["frac"], roof["other_roof"]["frac"], roof["third_roof"]["frac"]]
    assert roof["kernel"] == "k_run_search" and all(0 < f <= 1 for f in fracs)
    assert roof["alg_fp64_ops_per_launch"] == 5_000_000 * 32 * 18
    assert roof["alg_f16_matrix_ops_per_launch"] == 5_000_000 * 24_000 * 32


def test_two_dimensions_and_the_grid_are_fp64_work():
    b = _bench()
    for lanes, K in ((1, 16), (8, 16)):
        roof = b.roofline_of([(2, K, _stats(20_000_000, 400, 8.0, lanes))])
        assert roof["bound"] == "alu" and roof["alg_fp64_ops_per_launch"] == 20_000_000 * 400 * 6
        assert "third_roof" not in roof and roof["frac"] <= 1
    roof = b.roofline_of([(6, 32, _stats(100_000, 1000, 5.0, lanes=8))])
    assert roof["kernel"] == "k_search" and roof["alg_fp64_ops_per_launch"] == 100_000 * 1000 * 18
