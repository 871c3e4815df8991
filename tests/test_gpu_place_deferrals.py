"""rm_place on long runs of arrivals that lambda defers (evaluated 15 to 256 at a time):
bit for bit the oracle's decisions, means and final state, at the lengths where
a run starts or fills a batch, with models that end a run at every distance,
with departures and unknown models inside a run, and for every lane count of a
device."""
import numpy as np
import pytest

import oracle
from paper_2607_16784_amd import workloads as W
from test_gpu_place import gpu_place, same

pytestmark = pytest.mark.gpu


def matrix(N, light, seed):
    """Models that slow each other beyond any use, but for the first `light`."""
    rng = np.random.default_rng(seed)
    q = rng.integers(1, 400, N).astype(np.int32)
    T = q * rng.uniform(20.0, 80.0, N)
    D = np.minimum(T[:, None], T[None, :]) * rng.uniform(0.8, 2.0, (N, N))
    D[:light] *= 0.01
    D[:, :light] *= 0.01
    return D, T, q


@pytest.mark.parametrize("drop", [0, 1])
@pytest.mark.parametrize("G,C", [(16, 3), (16, 4), (4, 4), (7, 3), (12, 2), (20, 2),
                                 (64, 1), (8, 5), (6, 8), (2, 6)])
def test_runs(G, C, drop):
    N, light = 30, 3
    D, T, q = matrix(N, light, 7 * G + C)
    rng = np.random.default_rng(G + C)
    for n in (15, 16, 17, 33, 80, 81, 145, 600):
        for gap in (0, 20, 64, 270):
            print("deferrals", G, C, drop, n, gap, flush=True)
            ev = rng.integers(light, N, G + n).astype(np.int32)
            if gap:
                ev[G + gap::gap] = rng.integers(0, light, len(ev[G + gap::gap]))   # placed
            if n == 600:
                ev[G + 40] = N + 1           # unknown
                ev[G + 200] = -1 - 2         # departure of the model placed by event 2
                ev[G + 210] = -1 - (G + 5)   # of a deferred arrival
            same(gpu_place(D, T, q, G, C, ev, 0.3, drop), oracle.place(D, T, q, G, C, ev, 0.3, drop))


def test_departing_stream():
    N = 40
    D, T, q = matrix(N, 8, 5)
    ev = W.arrival_stream(600, N, seed=9, departures=True, dwell=(60, 200))
    same(gpu_place(D, T, q, 12, 4, ev, 0.3, 0), oracle.place(D, T, q, 12, 4, ev, 0.3, 0))


@pytest.mark.parametrize("G,chunk", [(1, 256), (3, 240), (5, 120), (9, 60), (16, 60), (17, 30),
                                     (33, 15), (64, 15)])
def test_chunks(G, chunk):
    # runs that end just before, at and after a scan's start and its chunks,
    # one placement between them; capacities of one lane a device and of as
    # many as fit 64 lanes
    N, light = 30, 3
    D, T, q = matrix(N, light, G)
    rng = np.random.default_rng(G)
    for C in sorted({1, 64 // G if 64 // G < 8 else 8}):
        ev = [light + g % 3 for g in range(G)]
        for n in (7, 8, 9, 9, 8, 8 + chunk - 1, 8 + chunk, 9 + chunk, 2 * chunk + 1):
            ev += [0] + list(rng.integers(light + 3, N, n))
        ev = np.array(ev, np.int32)
        print("chunks", G, C, len(ev), flush=True)
        for lam in (0.3, 0.9):
            same(gpu_place(D, T, q, G, C, ev, lam, 0), oracle.place(D, T, q, G, C, ev, lam, 0))


def test_scan_while_the_delays_are_checked():
    # a matrix so large that the first runs of deferrals come before the
    # other waves have checked it
    N, light = 2000, 40
    D, T, q = matrix(N, light, 1)
    rng = np.random.default_rng(2)
    ev = rng.integers(light, N, 1200).astype(np.int32)
    ev[16::150] = rng.integers(0, light, len(ev[16::150]))
    for G, C in ((16, 3), (1, 8)):
        print("unchecked", G, C, flush=True)
        same(gpu_place(D, T, q, G, C, ev, 0.3, 0), oracle.place(D, T, q, G, C, ev, 0.3, 0))
