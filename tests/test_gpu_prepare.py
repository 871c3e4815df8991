"""The isolated timelines at the edges of the prepare kernel's blocks, spans,
sub-chunks and chunks: iso_time (the last prefix sum) bit for bit against the
sequential sum, and the boundaries through the delays of the adjusted
simulation's OFFSETS: the kernel of model i that runs when j joins at tau has
P_i[k + 1] - tau of work left, so the delay depends on that boundary's last
bit."""
import numpy as np
import pytest

import oracle
from gpu_common import gpu_pair
from paper_2607_16784_amd import api
from paper_2607_16784_amd import workloads as W
from test_gpu_adjusted import same

pytestmark = pytest.mark.gpu

EDGES = [1, 15, 16, 17, 31, 32, 33, 127, 128, 129, 511, 512, 513, 640, 2047, 2048, 2049, 2560,
         4096, 4097, 4609]


def library(lengths, seed):
    parts = [W.make_library(1, n, "uniform", W.A100, seed=seed + m) for m, n in enumerate(lengths)]
    L = {k: np.concatenate([p[k] for p in parts]) for k in parts[0] if k != "offsets"}
    L["offsets"] = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    return L


def test_iso_time_is_the_sequential_sum():
    L = library(EDGES, seed=5)
    got = gpu_pair(W.A100, L, max_kernels_per_model=max(EDGES))
    off = L["offsets"]
    for m, n in enumerate(EDGES):
        want = np.cumsum(L["duration"][off[m]:off[m + 1]])[-1]   # in order, fp64
        assert got["iso_time"][m] == want, n
    assert np.array_equal(got["kernel_count"], EDGES)


@pytest.mark.parametrize("pair", [(17, 130), (513, 40), (2049, 33), (4097, 20)])
def test_boundaries(pair):
    # 64 boundaries of either model, each ordered pair
    L = library(list(pair), seed=11)
    K = 64
    kw = dict(align_mode=api.ALIGN_OFFSETS, reduce_mode="max", num_offsets=K,
              sweep_mode=api.SWEEP_ADJUSTED, per_alignment=True)
    got = gpu_pair(W.A100, L, **kw)
    kw["reduce_mode"] = oracle.REDUCE_MAX
    want = oracle.pair_matrix(W.A100, L, **kw)
    same(got["per_alignment"], want["per_alignment"], f"{pair}")


def test_every_boundary():
    # kernels of nearly one length, each longer than the step between two
    # offsets: every boundary of the long model ends the kernel that some
    # offset falls into
    L = library([2600, 3], seed=13)
    rng = np.random.default_rng(13)
    L["duration"][:2600] = rng.uniform(0.8, 1.2, 2600)
    K = 4096
    end = np.cumsum(L["duration"][:2600])
    running = np.searchsorted(end, end[-1] * np.arange(K) / K, side="right")
    assert np.array_equal(np.unique(running), np.arange(2600))
    kw = dict(align_mode=api.ALIGN_OFFSETS, reduce_mode="max", num_offsets=K,
              sweep_mode=api.SWEEP_ADJUSTED, per_alignment=True)
    got = gpu_pair(W.A100, L, **kw)
    kw["reduce_mode"] = oracle.REDUCE_MAX
    same(got["per_alignment"], oracle.pair_matrix(W.A100, L, **kw)["per_alignment"], "2600")


def test_bad_durations_are_flagged_wherever_they_are():
    for at in (0, 15, 16, 511, 512, 2047, 2048, 2200):
        L = library([2300, 3], seed=2)
        L["duration"][at] = -1.0
        got = gpu_pair(W.A100, L)
        assert got["status"] & api.ST_BAD_DURATION, at
