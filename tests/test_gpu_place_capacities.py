"""rm_place at capacities that are no power of two, where a device's lanes
hold empty slots past its capacity: bit for bit the oracle's decisions, means
and final state, on either side of the limit of 64 lanes, with departures,
both drops and an initial state."""
import numpy as np
import pytest

import oracle
from paper_2607_16784_amd import api
from paper_2607_16784_amd import workloads as W
from test_gpu_place import gpu_place, same

pytestmark = pytest.mark.gpu


def matrix(N, seed):
    rng = np.random.default_rng(seed)
    q = rng.integers(1, 400, N).astype(np.int32)
    T = q * rng.uniform(20.0, 80.0, N)
    return np.minimum(T[:, None], T[None, :]) * rng.uniform(0.0, 0.5, (N, N)), T, q


@pytest.mark.parametrize("drop", [0, 1])
@pytest.mark.parametrize("G,C", [(1, 3), (16, 3), (17, 3), (21, 3), (8, 5), (9, 5), (8, 6), (8, 7),
                                 (1, 7), (9, 7), (64, 1), (32, 2)])
def test_capacities(G, C, drop):
    N = 40
    D, T, q = matrix(N, 10 * G + C)
    for lam, departures in ((np.inf, False), (1.5, True), (0.4, True)):
        print("place", G, C, drop, lam, departures, flush=True)
        ev = W.arrival_stream(300, N, seed=G + C, departures=departures, dwell=(8, 48))
        want = oracle.place(D, T, q, G, C, ev, lam, drop)
        same(gpu_place(D, T, q, G, C, ev, lam, drop), want)


def test_initial_state_and_bad_events():
    N, G, C = 20, 5, 3
    D, T, q = matrix(N, 3)
    rng = np.random.default_rng(4)
    count = np.array([3, 0, 1, 2, 3], np.int32)
    resident = rng.integers(0, N, (G, C)).astype(np.int32)
    ev = np.array([4, 7, N + 2, -1, 5, -1 - 9, 6, -2, 8, 9, -9, 3, 1, 0, 2, -5], np.int32)
    want = oracle.place(D, T, q, G, C, ev, 1.0, 0, resident=resident.copy(), resident_count=count.copy())
    same(gpu_place(D, T, q, G, C, ev, 1.0, 0, resident=resident, count=count), want)
    for bad in (4, -1):      # a count beyond the capacity
        c = count.copy()
        c[1] = bad
        got = gpu_place(D, T, q, G, C, ev, 1.0, 0, resident=resident, count=c)
        assert got["status"] & api.ST_BAD_MODEL_ID
        assert np.all(got["placed_device"] == -1) and np.isnan(got["placed_mu_mean"]).all()
