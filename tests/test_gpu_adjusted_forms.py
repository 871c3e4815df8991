"""The adjusted-occupancy simulation's two record forms and two ways of
reading ahead against the CPU oracle, bit for bit, under every policy: float
block counts at their largest capacities, the general form just beyond them
(capacity, blocks per SM), block demands on and beside divisors of what a
kernel leaves, kernels that fit no SM or are invalid, and runs few and many
enough for either event loop."""
import numpy as np
import pytest

import oracle
from gpu_common import gpu_pair
from paper_2607_16784_amd import api
from paper_2607_16784_amd import workloads as W
from test_gpu_adjusted import same

pytestmark = pytest.mark.gpu
ADJ = api.SWEEP_ADJUSTED
TOP = (1 << 22) - 2     # largest capacity of the float form

DEVICES = {
    # warps, slots, registers, shared memory
    "float-top": dict(num_sm=2, max_threads_per_sm=1024, max_blocks_per_sm=15, regs_per_sm=TOP,
                      smem_per_sm=8000, warp_size=32),
    "float-top-smem": dict(num_sm=2, max_threads_per_sm=1024, max_blocks_per_sm=15,
                           regs_per_sm=8000, smem_per_sm=TOP, warp_size=32),
    "general-capacity": dict(num_sm=2, max_threads_per_sm=1024, max_blocks_per_sm=15,
                             regs_per_sm=TOP + 1, smem_per_sm=8000, warp_size=32),
    "float-blocks": dict(num_sm=1, max_threads_per_sm=127 * 32, max_blocks_per_sm=58,
                         regs_per_sm=65535, smem_per_sm=65535, warp_size=32),
    "general-blocks": dict(num_sm=1, max_threads_per_sm=127 * 32, max_blocks_per_sm=255,
                           regs_per_sm=65535, smem_per_sm=65535, warp_size=32),
    "one-block": dict(num_sm=4, max_threads_per_sm=1024, max_blocks_per_sm=1, regs_per_sm=65536,
                      smem_per_sm=65536, warp_size=64),
}


def library(device, models, q, seed):
    """Kernels whose register and shared-memory demands sit on and beside
    divisors of the capacities, with invalid and infeasible ones among them."""
    rng = np.random.default_rng(seed)
    n = models * q
    threads = rng.choice([1, 32, 33, 64, 96, 256, 512], n)
    threads = np.minimum(threads, device["max_threads_per_sm"])
    parts = rng.integers(1, 80, n)
    regs = device["regs_per_sm"] // (parts * threads) + rng.integers(-1, 2, n)
    smem = device["smem_per_sm"] // rng.integers(1, 80, n) + rng.integers(-1, 2, n)
    regs = np.where(rng.random(n) < 0.15, 0, np.maximum(regs, 0))
    smem = np.where(rng.random(n) < 0.15, 0, np.maximum(smem, 0))
    grid = rng.integers(1, 200, n)
    odd = rng.random(n)
    grid[odd < 0.01] = 0                                        # invalid
    threads[(odd > 0.01) & (odd < 0.02)] = 2 * device["max_threads_per_sm"]   # fits no SM
    smem[(odd > 0.02) & (odd < 0.03)] = 2 * device["smem_per_sm"]
    # repeated durations, so that kernels of two models end together
    dur = rng.choice([1.0, 2.0, 3.0, 0.5], n) * rng.choice([1.0, 1.0, 1.25, 0.7], n)
    i32 = lambda x: x.astype(np.int32)  # noqa: E731
    return dict(offsets=np.arange(models + 1, dtype=np.int64) * q, grid=i32(grid),
                threads=i32(threads), regs=i32(regs), smem=i32(smem), duration=dur)


@pytest.mark.parametrize("name", sorted(DEVICES))
@pytest.mark.parametrize("policy", ["equal", "priority", "fcfs"])
def test_forms(name, policy):
    device = DEVICES[name]
    L = library(device, 7, 90, seed=len(name))
    pol = api.POLICY_NAMES[policy]
    draws = W.start_draws(7, 9, seed=3)
    for align, K in (("first", 1), ("offsets", 5), ("sampled_starts", 9)):
        print("forms", name, policy, align, flush=True)
        am = api.ALIGN_NAMES[align]
        kw = dict(start_draws=draws) if align == "sampled_starts" else {}
        want = oracle.pair_matrix(device, L, align_mode=am, num_offsets=K, sweep_mode=ADJ,
                                  policy=pol, **kw)
        if kw:
            import torch
            kw = dict(start_draws=torch.as_tensor(draws.reshape(-1)).cuda())
        got = gpu_pair(device, L, align_mode=am, num_offsets=K, sweep_mode=ADJ, policy=pol, **kw)
        same(got["delay"], want["delay"], f"{align} delay")
        same(got["slowdown"], want["slowdown"], f"{align} slowdown")
        assert got["status"] == want["status"]


@pytest.mark.parametrize("policy", ["equal", "priority", "fcfs"])
@pytest.mark.parametrize("models", [1, 285, 286])
def test_few_and_many_runs(models, policy):
    # two lanes a run: the 40,755 unordered pairs of 285 models fit 1280 waves,
    # the 41,041 of 286 do not; lengths so short that runs end within the
    # events read ahead
    device = W.A100
    L = library(device, models, 6, seed=models)
    rng = np.random.default_rng(1)
    lens = rng.integers(1, 7, models)
    take = np.concatenate([np.arange(n) + 6 * m for m, n in enumerate(lens)])
    for k in ("grid", "threads", "regs", "smem", "duration"):
        L[k] = L[k][take]
    L["offsets"] = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    pol = api.POLICY_NAMES[policy]
    print("runs", models, policy, flush=True)
    want = oracle.pair_matrix(device, L, sweep_mode=ADJ, policy=pol)
    got = gpu_pair(device, L, sweep_mode=ADJ, policy=pol, per_alignment=True)
    same(got["delay"], want["delay"], "delay")
    same(got["per_alignment"], want["delay"], "per alignment")
    same(got["slowdown"], want["slowdown"], "slowdown")


@pytest.mark.parametrize("name", ["a100", "general-blocks"])
def test_priority_one_lane(name):
    # more than 250,000 runs under PRIORITY take one lane each, in tiles of 8 x 8
    # ordered pairs: model counts on and beside a multiple of 8, a bound on the
    # number of offsets or draws at which the rule turns, invalid and empty models
    device = W.A100 if name == "a100" else DEVICES[name]
    pol = api.POLICY_NAMES["priority"]
    for models, align, K in ((500, "first", 1), (501, "first", 1), (504, "first", 1),
                             (62, "offsets", 66), (63, "offsets", 63), (64, "offsets", 62),
                             (63, "sampled_starts", 64), (1, "offsets", 4096)):
        L = library(device, models, 6, seed=models + K)
        lens = np.random.default_rng(2).integers(0, 7, models)
        take = np.concatenate([np.arange(n) + 6 * m for m, n in enumerate(lens)])
        for k in ("grid", "threads", "regs", "smem", "duration"):
            L[k] = L[k][take]
        L["offsets"] = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
        am = api.ALIGN_NAMES[align]
        print("one lane", name, models, align, K, flush=True)
        kw, gk = {}, {}
        if align == "sampled_starts":
            import torch
            draws = W.start_draws(models, K, seed=3)
            kw, gk = dict(start_draws=draws), dict(start_draws=torch.as_tensor(draws.reshape(-1)).cuda())
        want = oracle.pair_matrix(device, L, align_mode=am, num_offsets=K, sweep_mode=ADJ,
                                  policy=pol, **kw)
        got = gpu_pair(device, L, align_mode=am, num_offsets=K, sweep_mode=ADJ, policy=pol, **gk)
        same(got["delay"], want["delay"], f"{align} delay")
        same(got["slowdown"], want["slowdown"], f"{align} slowdown")
        assert got["status"] == want["status"]


def test_more_runs_than_lanes_of_a_dispatch():
    # 520^2 ordered pairs of 4096 offsets are 1.1e9 runs of two lanes: more lanes
    # than one dispatch takes.  Two kinds of models, so four kinds of pairs.
    import torch
    N, K = 520, 4096
    two = library(W.A100, 2, 3, seed=21)
    print("many runs", flush=True)
    want = oracle.pair_matrix(W.A100, two, align_mode=api.ALIGN_OFFSETS, reduce_mode=oracle.REDUCE_MAX,
                              num_offsets=K, sweep_mode=ADJ)
    L = {k: np.tile(two[k], N // 2) for k in two if k != "offsets"}
    L["offsets"] = np.arange(N + 1, dtype=np.int64) * 3
    D = api.library_to_device(L)
    out = dict(delay=torch.full((N * N,), -1.0, dtype=torch.float64, device="cuda"),
               iso_time=torch.empty(N, dtype=torch.float64, device="cuda"),
               kernel_count=torch.empty(N, dtype=torch.int32, device="cuda"))
    got = api.rm_pair_slowdown_matrix(W.A100, D["offsets"], D["grid"], D["threads"], D["regs"],
                                      D["smem"], D["duration"], align_mode="offsets",
                                      reduce_mode="max", num_offsets=K, sweep_mode=ADJ, out=out)
    torch.cuda.synchronize()
    ref = torch.as_tensor(np.tile(np.asarray(want["delay"]).reshape(2, 2), (N // 2, N // 2))).cuda()
    assert torch.equal(got["delay"].view(N, N), ref)
