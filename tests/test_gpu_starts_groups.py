"""CONFLICT_STARTS at the edges of its lane groups, chunks and selection: every
alignment's delay against the CPU oracle (sums of at most some hundred fp64
terms of one sign in another order: 1e-12 relative), and the reduction exactly
-- the median and maximum of the GPU's own per-alignment values."""
import numpy as np
import pytest

import oracle
from gpu_common import assert_rel, gpu_pair
from paper_2607_16784_amd import api
from paper_2607_16784_amd import workloads as W

pytestmark = pytest.mark.gpu


def library(lengths, seed, same=False, kernels="uniform"):
    parts = [W.make_library(1, n, kernels, W.A100, seed=seed + m) if n else
             W.make_library(1, 0, kernels, W.A100, seed=1) for m, n in enumerate(lengths)]
    L = {k: np.concatenate([p[k] for p in parts]) for k in parts[0] if k != "offsets"}
    L["offsets"] = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    if same:   # every kernel alike: thousands of equal delays
        for k in L:
            if k != "offsets":
                L[k][:] = L[k][0]
        L["grid"][:], L["threads"][:], L["regs"][:], L["smem"][:] = 4000, 1024, 40, 0
    return L


CASES = {
    "short": ([1, 2, 7, 8, 9, 0, 63, 64, 65], 65),
    "eight-lanes-most": ([128, 100, 127], 128),        # pair cap 256
    "sixteen-lanes": ([129, 126, 5], 129),             # pair cap 258
    "sixteen-lanes-most": ([320, 51, 40], 320),        # pair cap 640, 320 x 51 start pairs
    "whole-wave": ([1000, 16, 15], 1000),
    "no-hint": ([60, 61, 3], 0),
    # the reduction's lanes: 64 up to 512 start pairs a pair, 256 up to 1024 and for
    # many pairs, 1024 beyond; 64 and 65 members are ranked and counted
    "reduce-64": ([1, 8, 22, 0, 9, 16], 22),
    "reduce-256": ([23, 32, 2, 13, 5], 32),
    "reduce-256-many": ([33, 50, 1, 0, 13] + [3, 8, 5] * 9, 80),
    "reduce-1024-few": ([33, 50, 1, 13], 80),
}


@pytest.mark.parametrize("red", ["median", "max"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_groups(name, red):
    lengths, hint = CASES[name]
    L = library(lengths, seed=17)
    N, nk = len(lengths), int(sum(lengths))
    print("starts", name, red, flush=True)
    mode = oracle.REDUCE_MAX if red == "max" else oracle.REDUCE_MEDIAN
    got = gpu_pair(W.A100, L, align_mode=api.ALIGN_CONFLICT_STARTS, reduce_mode=red,
                   max_kernels_per_model=hint, per_alignment=True)
    want = oracle.pair_matrix(W.A100, L, align_mode=oracle.ALIGN_CONFLICT_STARTS, reduce_mode=mode,
                              per_alignment=True)
    pa = got["per_alignment"].reshape(nk, nk)
    ref = np.asarray(want["per_alignment"]).reshape(nk, nk)
    off = L["offsets"]
    for i in range(N):
        for j in range(N):
            block = np.s_[off[i]:off[i + 1], off[j]:off[j + 1]]
            if lengths[i] * lengths[j] > api_limit():
                assert np.isnan(pa[block]).all() and np.isnan(got["delay"][i, j])
                continue
            assert_rel(pa[block], ref[block], 1e-12, f"{name} ({i}, {j})")
            v = pa[block][~np.isnan(pa[block])]
            mid = 0.0 if v.size == 0 else (np.max(v) if red == "max" else np.median(v))
            assert got["delay"][i, j] == mid


def api_limit():
    return 16384      # RM_MAX_STARTS_PER_PAIR


def test_ties():
    # thousands of equal delays, and a few distinct values among them
    for lengths in ([60, 60], [64, 3]):
        L = library(lengths, seed=1, same=True)
        for red in ("median", "max"):
            got = gpu_pair(W.A100, L, align_mode=api.ALIGN_CONFLICT_STARTS, reduce_mode=red,
                           max_kernels_per_model=64, per_alignment=True)
            nk = sum(lengths)
            pa = got["per_alignment"].reshape(nk, nk)
            off = L["offsets"]
            for i in range(2):
                for j in range(2):
                    v = pa[off[i]:off[i + 1], off[j]:off[j + 1]].reshape(-1)
                    assert not np.isnan(v).any()
                    assert got["delay"][i, j] == (np.max(v) if red == "max" else np.median(v))


@pytest.mark.parametrize("count", [1, 2, 63, 64, 65, 66, 127, 128, 300])
def test_members_ranked_or_counted(count):
    # one model of one kernel against `count` kernels that all interfere with it
    L = library([1, count], seed=3)
    L["grid"][:], L["threads"][:], L["regs"][:], L["smem"][:] = 4000, 1024, 40, 0
    for hint in (count, 0):
        for red in ("median", "max"):
            got = gpu_pair(W.A100, L, align_mode=api.ALIGN_CONFLICT_STARTS, reduce_mode=red,
                           max_kernels_per_model=hint, per_alignment=True)
            v = got["per_alignment"].reshape(count + 1, count + 1)[0, 1:]
            assert not np.isnan(v).any()
            assert got["delay"][0, 1] == (np.max(v) if red == "max" else np.median(v))


@pytest.mark.parametrize("sweep", ["temporal", "adjusted"])
def test_many_models(sweep):
    # 2,050^2 ordered pairs: more of them than workgroups of one dispatch
    N = 2050
    lengths = np.random.default_rng(8).integers(1, 3, N)
    L = W.make_library(N, 2, "uniform", W.A100, seed=12)
    take = np.concatenate([np.arange(n) + 2 * m for m, n in enumerate(lengths)])
    for k in ("grid", "threads", "regs", "smem", "duration"):
        L[k] = L[k][take]
    L["offsets"] = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    mode = api.SWEEP_NAMES[sweep]
    print("many models", sweep, flush=True)
    want = oracle.pair_matrix(W.A100, L, align_mode=oracle.ALIGN_CONFLICT_STARTS, sweep_mode=mode)
    for hint in (2, 0, 40):     # 64, 1024 and 256 lanes
        got = gpu_pair(W.A100, L, align_mode=api.ALIGN_CONFLICT_STARTS, sweep_mode=mode,
                       max_kernels_per_model=hint)
        assert_rel(got["delay"], want["delay"], 1e-12, f"{sweep} {hint}")
        assert_rel(got["slowdown"], want["slowdown"], 1e-12, f"{sweep} {hint}")
