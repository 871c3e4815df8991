"""SAMPLED_STARTS around the largest number of interfering draws that are
ordered by window length before they are swept (128), with every draw
interfering and with window lengths that are all distinct or all alike:
against the CPU oracle, whose fp64 sums of at most some hundred terms of one
sign run in another order (1e-12 relative)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import assert_rel, gpu_pair
from paper_2607_16784_amd import api
from paper_2607_16784_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alike", [False, True])
@pytest.mark.parametrize("K", [64, 127, 128, 129, 200])
def test_members_around_the_limit(K, alike):
    L = W.make_library(3, (150, 170), "uniform", W.A100, seed=K)
    L["grid"][:], L["threads"][:], L["regs"][:], L["smem"][:] = 4000, 1024, 40, 0   # all interfere
    draws = W.start_draws(3, K, seed=5)
    if alike:
        draws[:] = draws.reshape(-1)[0]
    print("sampled order", K, alike, flush=True)
    ref = oracle.pair_matrix(W.A100, L, align_mode=oracle.ALIGN_SAMPLED_STARTS, num_offsets=K,
                             start_draws=draws, per_alignment=True)
    got = gpu_pair(W.A100, L, align_mode=api.ALIGN_SAMPLED_STARTS, num_offsets=K,
                   start_draws=torch.as_tensor(draws.reshape(-1)).cuda(), per_alignment=True)
    want = np.asarray(ref["per_alignment"])
    assert not np.isnan(want).any()
    assert_rel(got["per_alignment"].reshape(want.shape), want, 1e-12, "per alignment")
    assert_rel(got["delay"], ref["delay"], 1e-12, "delay")
