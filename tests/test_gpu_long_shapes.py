"""FIRST on libraries longer than two models per staging half, one for each way
the tile shape is chosen there (one pair per item, two rows by one column, the
usual shape with some pairs swept from memory, the same for few long models
among more than 64, no bound given, a model longer than the whole LDS), against the CPU oracle: sums of some thousand fp64 terms
of one sign in another order, 1e-12 relative."""
import numpy as np
import pytest

import oracle
from gpu_common import assert_rel, gpu_pair
from paper_2607_16784_amd import workloads as W
from test_gpu_parity_limits import sized_library

pytestmark = pytest.mark.gpu

CASES = {
    # lengths, bound given
    "one-pair": ([4000, 3900, 1000, 2600, 1, 3000, 0, 2500], 4000),
    "three-fit": ([2600] * 5, 2600),
    "three-fit-ragged": ([100, 3000, 2900, 1500, 1700, 3343], 3343),
    "mostly-short": ([300, 200, 4000, 500, 300, 250, 400, 300, 350, 10], 4000),
    "few-long-of-65": ([1200, 4000] + [60, 90, 1100] * 21, 4000),
    "no-bound": ([2600, 2700, 5200, 3000, 1], 0),
    "longer-than-lds": ([10100, 60, 5100, 4000], 10100),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_first(name):
    lengths, bound = CASES[name]
    L = sized_library(lengths, seed=600, kernels="decode")
    print("long shapes", name, flush=True)
    want = oracle.pair_matrix(W.A100, L)
    got = gpu_pair(W.A100, L, max_kernels_per_model=bound, per_alignment=True)
    assert got["status"] == want["status"]
    assert_rel(got["delay"], want["delay"], 1e-12, "delay")
    assert_rel(got["slowdown"], want["slowdown"], 1e-12, "slowdown")
    assert np.array_equal(got["per_alignment"].reshape(-1), got["delay"].reshape(-1))
