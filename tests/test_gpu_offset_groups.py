"""OFFSETS at the edges of its lane groups: offset counts on either side of 16
and 32 and beside multiples of a workgroup's groups, models of one kernel up
to some hundred and a pair swept from memory, every alignment against the CPU
oracle (sums of one sign in another order, 1e-12 relative) and both reductions
of the GPU's own values."""
import numpy as np
import pytest

import oracle
from gpu_common import assert_rel, gpu_pair
from paper_2607_16784_amd import api
from paper_2607_16784_amd import workloads as W
from test_gpu_parity_limits import sized_library

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 100])
@pytest.mark.parametrize("red", ["median", "max"])
def test_groups(K, red):
    lengths = [1, 2, 9, 130, 0, 517, 64]
    L = sized_library(lengths, seed=90 + K, kernels="uniform")
    N = len(lengths)
    print("offsets", K, red, flush=True)
    mode = oracle.REDUCE_MAX if red == "max" else oracle.REDUCE_MEDIAN
    want = oracle.pair_matrix(W.EDGE, L, align_mode=oracle.ALIGN_OFFSETS, reduce_mode=mode,
                              num_offsets=K, per_alignment=True)
    for hint in (517, 100):      # 100: the longest pairs are read from memory
        got = gpu_pair(W.EDGE, L, align_mode=api.ALIGN_OFFSETS, reduce_mode=red, num_offsets=K,
                       max_kernels_per_model=hint, per_alignment=True)
        assert_rel(got["per_alignment"], want["per_alignment"], 1e-12, "per offset")
        pa = got["per_alignment"].reshape(N, N, K)
        mid = pa.max(2) if red == "max" else np.median(pa, 2)
        assert np.array_equal(got["delay"], mid)
        assert_rel(got["slowdown"], want["slowdown"], 1e-12, "slowdown")
