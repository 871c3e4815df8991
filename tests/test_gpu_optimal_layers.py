"""rm_place_optimal over shapes whose layers hold several popcounts, against a
subset dynamic program over all 2^n unions in numpy (fp64, the same sums in
another order: a sum of at most n costs of at most 4 members, 1e-12
relative)."""
import itertools

import numpy as np
import pytest
import torch

import oracle
from paper_2607_16784_amd import api
from paper_2607_16784_amd import workloads as W

pytestmark = pytest.mark.gpu
REL = 1e-12


def library():
    L = W.config_library("cnn_64")
    r = oracle.pair_matrix(W.A100, L)
    N = len(r["iso_time"])
    return np.asarray(r["delay"]).reshape(N, N), r["iso_time"], r["kernel_count"]


def set_cost(delay, T, q, members):
    total = 0.0
    for p, i in enumerate(members):
        t = T[i]
        for r, j in enumerate(members):
            if r != p:
                t += max(q[i] / q[j], 1.0) * delay[i, j]
        total += (t - T[i]) / T[i]
    return total


def best_mean(delay, T, q, models, G, C):
    """min over at most G sets: a set is split off with the lowest model left."""
    n = len(models)
    full = np.arange(1 << n)
    f = np.full(1 << n, np.inf)
    f[0] = 0.0
    best = np.inf
    sets = [s for k in range(1, C + 1) for s in itertools.combinations(range(n), k)]
    cost = [set_cost(delay, T, q, [models[b] for b in s]) for s in sets]
    for _ in range(min(G, n)):
        g = np.full(1 << n, np.inf)
        for s, c in zip(sets, cost):
            bits = sum(1 << b for b in s)
            below = (1 << s[0]) - 1
            m = full[((full & bits) == bits) & ((full & below) == 0)]
            np.minimum.at(g, m, f[m ^ bits] + c)
        f = g
        best = min(best, f[-1])
    return best / n


@pytest.mark.parametrize("n,G,C", [(1, 3, 4), (4, 2, 4), (12, 3, 4), (13, 6, 4), (14, 5, 4),
                                   (12, 12, 2), (13, 8, 2), (11, 5, 3), (13, 9, 3), (9, 9, 1)])
def test_optimum_matches_subset_program(n, G, C):
    delay, T, q = library()
    rng = np.random.default_rng(100 * n + 10 * G + C)
    for models in (rng.choice(len(T), n, replace=False), rng.integers(0, 3, n)):
        print("optimal placement", n, G, C, models.tolist(), flush=True)
        st = api.new_status()
        out = api.rm_place_optimal(torch.as_tensor(delay.reshape(-1)).cuda(),
                                   torch.as_tensor(T).cuda(), torch.as_tensor(q).cuda(),
                                   torch.as_tensor(models.astype(np.int32)).cuda(), G, C,
                                   status=st)
        torch.cuda.synchronize()
        want = best_mean(delay, T, q, models, G, C)
        assert float(out["best_mean"].item()) == pytest.approx(want, rel=REL, abs=0.0)
        dev = out["best_device"].cpu().numpy()
        assert dev.min() == 0 and dev.max() < G and np.bincount(dev).max() <= C
        got = sum(set_cost(delay, T, q, models[dev == g]) for g in range(G)) / n
        assert got == pytest.approx(want, rel=REL, abs=0.0)
        assert int(st.item()) == 0


def best_of_kinds(delay, T, q, kinds, counts, G, C):
    """The same for replicas of a few kinds, over the counts left of each kind."""
    sets = [c for c in itertools.product(*(range(min(C, x) + 1) for x in counts))
            if 0 < sum(c) <= C]
    cost = {c: set_cost(delay, T, q, [m for m, x in zip(kinds, c) for _ in range(x)]) for c in sets}
    f = {(0,) * len(counts): 0.0}
    best = np.inf
    for _ in range(G):
        g = {}
        for left, v in f.items():
            for c, w in cost.items():
                to = tuple(a + b for a, b in zip(left, c))
                if all(a <= b for a, b in zip(to, counts)) and v + w < g.get(to, np.inf):
                    g[to] = v + w
        f = g
        best = min(best, f.get(tuple(counts), np.inf))
    return best / sum(counts)


@pytest.mark.parametrize("n,G,C", [(22, 9, 3), (24, 12, 3), (19, 7, 4), (20, 8, 4), (24, 6, 4),
                                   (24, 24, 2)])
def test_large_layers(n, G, C):
    # layers of more masks than lanes a launch aims at
    delay, T, q = library()
    rng = np.random.default_rng(n + G + C)
    kinds = rng.choice(len(T), 3, replace=False)
    counts = [n // 3, n // 3, n - 2 * (n // 3)]
    replicas = rng.permutation(np.repeat(kinds, counts))
    for models in (replicas, rng.choice(len(T), n, replace=False)):
        print("optimal placement", n, G, C, models.tolist(), flush=True)
        st = api.new_status()
        out = api.rm_place_optimal(torch.as_tensor(delay.reshape(-1)).cuda(),
                                   torch.as_tensor(T).cuda(), torch.as_tensor(q).cuda(),
                                   torch.as_tensor(models.astype(np.int32)).cuda(), G, C, status=st)
        torch.cuda.synchronize()
        got = float(out["best_mean"].item())
        if models is replicas:
            assert got == pytest.approx(best_of_kinds(delay, T, q, kinds, counts, G, C), rel=REL, abs=0.0)
        dev = out["best_device"].cpu().numpy()
        assert dev.min() == 0 and dev.max() < G and np.bincount(dev).max() <= C
        score = sum(set_cost(delay, T, q, models[dev == g]) for g in range(G)) / n
        assert score == pytest.approx(got, rel=REL, abs=0.0)
        for _ in range(200):     # no random placement is better
            d = rng.permutation(np.repeat(np.arange(G), C))[:n]
            assert sum(set_cost(delay, T, q, models[d == g]) for g in range(G)) / n >= got * (1 - REL)
        assert int(st.item()) == 0
