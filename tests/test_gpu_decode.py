"""The general-k decode (k > 64) against the oracle, bit for bit, where its
buffer, cell list and passes change course: buffers that fit every candidate
and buffers that overflow and are cut many times, cell lists that fit and that
are taken in pieces, filtered passes and completions with zero counts, R = 1
(nothing to filter by), 256- and 1024-thread workgroups, 16- and 32-bit cells."""
import numpy as np
import pytest

import oracle
from gpu_common import log
from workloads import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_2106_11565_amd as flinng
    flinng.lib()
    return flinng


@pytest.mark.parametrize("N,R,B,K,L", [
    (6000, 1, 40, 6, 6),        # no filter; cells of 150 members
    (20011, 3, 50, 5, 12),      # most cells positive, every pass large
    (20000, 4, 1021, 10, 20),   # more positive cells than one list
    (30000, 8, 8192, 8, 16),    # 1024 threads, 16-bit cells
    (30001, 8, 16384, 10, 5),   # 1024 threads, 32-bit cells, little LDS left
    (300, 2, 300, 12, 4),       # one member per cell, mostly zero counts
])
def test_general_k_equals_oracle(fl, N, R, B, K, L):
    X, Q, _ = synth.dense_gmm(N=N, d=24, n_centres=max(3, N // 300), sigma=0.2, nq=24)
    gi = fl.Index(X, 0, K, L, R, B, seed=77)
    oi = oracle.OracleIndex(oracle.SRP_F32, X, K, L, R, B, 77)
    for k in (65, 100, 257, 1000, 2049, 4096):
        if B == 16384 and k > 1000:
            continue  # its counters and the k keys pass the LDS limit
        want = oi.query(Q, k)
        for pers in (False, True):
            log("general k", N, R, B, "k", k, "persistent", pers)
            got = gi.query(Q, k, persistent=pers)
            assert np.array_equal(got[0], want[0]), (k, pers)
            assert np.array_equal(got[1], want[1]), (k, pers)
