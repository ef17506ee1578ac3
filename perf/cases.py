"""What is timed of this framework: its public joins, over the range of sizes,
dimensions, K and distributions that its own benchmark, serving pool and tests
use (2-6 dimensions, 1e4 to 2e7 points, K from 1 to 64; uniform, exponential
and clustered coordinates).

A case names a path:
  join   knn_self_join_device on an index that the program keeps
  step   knn_build_index_device and knn_self_join_device on new points (the
         benchmark's step)
  query  knn_join_device: the neighbours of a query set in a kept index
  host   knn_build_index and knn_self_join: numpy in, numpy out
  eps    the distance similarity self-join (level, counts, every pair) on a
         kept index
"""

import math

import torch

from paper_1810_04758_amd import api


def _case(name, path, kind, n, N, K=0, NQ=0, pairs=0.0, **opts):
    c = {"path": path, "kind": kind, "n": n, "N": N, "K": K, "NQ": NQ, "pairs": pairs}
    c.update({"opt_" + k: v for k, v in opts.items()})
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest configuration of the benchmark, many times over on one
        # index: latency, launches and read-backs
        _case("join_unif2d_50k_k5", "join", "uniform", 2, 50_000, K=5),
        # a small data set seen once: index build and join
        _case("step_expo3d_10k_k4", "step", "exponential", 3, 10_007, K=4),
        # the benchmark's skewed sets, at a small and at a larger K
        _case("join_expo2d_2m_k8", "join", "exponential", 2, 2_000_000, K=8),
        _case("join_expo4d_2m_k32", "join", "exponential", 4, 2_000_000, K=32),
        # the serving pool's three-dimensional sets and its largest K
        _case("join_unif3d_1m_k16", "join", "uniform", 3, 1_000_003, K=16),
        _case("join_expo4d_150k_k64", "join", "exponential", 4, 150_001, K=64),
        # the highest dimension
        _case("join_unif6d_5m_k32", "join", "uniform", 6, 5_000_000, K=32),
        # the benchmark's headline: the largest set, build and join
        _case("step_clus2d_20m_k16", "step", "clustered", 2, 20_000_000, K=16),
        # a program that gives the level structure and cell side itself, as the
        # autotuner answered for this kind of set
        _case("join_clus2d_3m_k16_opts", "join", "clustered", 2, 3_000_001, K=16,
              zorder=1, w_factor=0.14, queue_grain=-16),
        # queries of another draw against a resident set
        _case("query_clus2d_2m_100k_k16", "query", "clustered", 2, 2_000_000, K=16, NQ=100_003),
        # results in host memory, as the serving loop returns them
        _case("host_unif2d_300k_k4", "host", "uniform", 2, 300_007, K=4),
        # every pair within eps, about 32 a point
        _case("eps_expo2d_2m_32", "eps", "exponential", 2, 2_000_000, pairs=32.0),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))) | rng.randint(0, 1)

    path = rng.choice(["join", "join", "join", "step", "step", "query", "host", "eps"])
    kind = rng.choice(["uniform", "exponential", "clustered"])
    n = 2 if kind == "clustered" else rng.choice([2, 2, 3, 3, 4, 4, 5, 6])
    K = size(1, 64)
    top = {2: 8e6, 3: 4e6, 4: 2e6, 5: 6e5, 6: 4e5}[n]
    if path == "query":
        return _case("", path, kind, n, size(2e4, top), K=K, NQ=size(500, 3e5))
    if path == "host":
        return _case("", path, kind, n, size(1e4, 3e5), K=K)
    if path == "eps":
        return _case("", path, kind, n, size(1e4, min(top, 2e6)), pairs=float(size(4, 64)))
    return _case("", path, kind, n, size(1e4, top), K=K)


def _points(kind, n, N, gen):
    """The shapes of the package's generators, drawn on the GPU."""
    dev = "cuda"
    if kind == "uniform":
        return torch.rand((N, n), dtype=torch.float64, device=dev, generator=gen) * 100.0
    if kind == "exponential":  # rate 40
        return torch.rand((N, n), dtype=torch.float64, device=dev, generator=gen).neg_().log1p_().mul_(-1.0 / 40.0)
    # 70 % in 500 Gaussian clusters on [0,360) x [-90,90), the rest uniform
    rand = lambda *s: torch.rand(s, dtype=torch.float64, device=dev, generator=gen)  # noqa: E731
    m = int(round(0.7 * N))
    span = torch.tensor([360.0, 180.0], dtype=torch.float64, device=dev)
    low = torch.tensor([0.0, -90.0], dtype=torch.float64, device=dev)
    centre = rand(500, 2) * span + low
    sigma = 0.05 * torch.exp(rand(500) * math.log(2.0 / 0.05))
    which = torch.randint(0, 500, (m,), device=dev, generator=gen)
    pts = torch.empty((N, 2), dtype=torch.float64, device=dev)
    pts[:m] = centre[which] + sigma[which, None] * torch.randn((m, 2), dtype=torch.float64,
                                                               device=dev, generator=gen)
    pts[m:] = rand(N - m, 2) * span + low
    return pts[torch.randperm(N, device=dev, generator=gen)].contiguous()


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    D = _points(case["kind"], case["n"], case["N"], gen)
    Q = _points(case["kind"], case["n"], case["NQ"], gen) if case["NQ"] else None
    return D, Q


def _eps(case):
    """The search distance at which a point has about case["pairs"] neighbours
    on average (the mean density over the points; the clustered set's is taken
    of its mean cluster and its background)."""
    n, N, pairs = case["n"], case["N"], case["pairs"]
    ball = math.pi ** (n / 2) / math.gamma(n / 2 + 1)
    if case["kind"] == "uniform":
        density = N / 100.0 ** n
    elif case["kind"] == "exponential":
        density = N * 20.0 ** n  # the density over the points averages to half the peak a dimension
    else:
        s1, s2 = 0.05, 2.0
        inv = (s1 ** -2 - s2 ** -2) / (2 * math.log(s2 / s1))  # mean of 1 / sigma^2
        density = N * (0.49 * inv / (500 * 4 * math.pi) + 1.0 / (360 * 180))
    return (pairs / (density * ball)) ** (1.0 / n)


def prepare(case, seed):
    D, Q = _inputs(case, seed)
    state = {"case": case, "opts": {k[4:]: v for k, v in case.items() if k.startswith("opt_")}}
    if case["path"] == "host":
        state["D"] = D.cpu().numpy()
    elif case["path"] == "step":
        state["D"] = D
    else:
        state["index"] = api.build_index(D)
        state["Q"] = Q
    if case["path"] == "eps":
        state["eps"] = _eps(case)
        # the result buffers of a program that takes the pairs batch by batch
        # (one batch, unless the draw is far denser than its mean)
        cap = int(1.3 * case["N"] * case["pairs"])
        state["pairs"] = [torch.zeros(cap, dtype=t, device="cuda")
                          for t in (torch.int32, torch.int32, torch.float64)]
    torch.cuda.synchronize()
    return state


def run(state):
    case, K, opts = state["case"], state["case"]["K"], state["opts"]
    if case["path"] == "join":
        return state["index"].self_join(K, **opts)
    if case["path"] == "query":
        return state["index"].join(state["Q"], K, **opts)
    if case["path"] == "eps":
        # the level and the counts belong to the pass: a new eps has to build them
        index, eps, cursor = state["index"], state["eps"], 0
        index.eps_join_release()
        total, counts = index.eps_join_size(eps, counts=True)
        while cursor < case["N"]:
            _, cursor = index.eps_join_batch(eps, cursor, *state["pairs"])
        return [total, counts] + state["pairs"]
    index = api.build_index(state["D"])
    out = index.self_join_host(K, **opts) if case["path"] == "host" else index.self_join(K, **opts)
    index.close()
    return out


def work(case):
    """Points read once, results written once; per neighbour in the result one
    distance (n differences, n products, n - 1 sums) and one comparison."""
    n, N, K = case["n"], case["N"], case["K"]
    if case["path"] == "eps":
        found = N * case["pairs"]
        return {"bytes": 8.0 * N * n + 16.0 * found, "flops": 3.0 * n * found}
    rows = case["NQ"] or N
    return {"bytes": 8.0 * n * (N + case["NQ"]) + 12.0 * rows * K, "flops": 3.0 * n * rows * K}


def exact(case, seed):
    """The distances by brute force in 64 bits, where that is quick; the ids are
    whole numbers and have to be equal anyway."""
    rows = case["NQ"] or case["N"]
    if case["path"] == "eps" or rows * case["N"] > 2.5e10:
        return None
    D, Q = _inputs(case, seed)
    own = Q is None
    Q = D if own else Q
    K, step = case["K"], max(1, int(1e8) // case["N"])
    dists = torch.empty((rows, K), dtype=torch.float64, device=D.device)
    for a in range(0, rows, step):
        q = Q[a:a + step]
        d2 = torch.zeros((q.shape[0], case["N"]), dtype=torch.float64, device=D.device)
        for j in range(case["n"]):
            d2 += (q[:, j, None] - D[None, :, j]) ** 2
        if own:
            i = torch.arange(q.shape[0], device=D.device)
            d2[i, a + i] = math.inf
        dists[a:a + step] = torch.topk(d2, K, largest=False, sorted=True).values.sqrt()
    return None, (dists.cpu().numpy() if case["path"] == "host" else dists)
