"""SRP codes of large batches against the oracle, bit for bit: enough rows that
the projection takes its 96-row tiles, with a remainder of rows, a last chunk of
k that is not full, groups of hyperplanes that do and do not fill the tile, rows
in place and padded; and the same rows in a small batch."""
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


@pytest.mark.parametrize("n,d,K,L", [
    (24_575, 1024, 24, 12),   # 288 hyperplanes, whole chunks
    (24_481, 1032, 16, 17),   # 272 hyperplanes, padded rows, a chunk of 32
    (24_576, 1120, 13, 40),   # two groups of 20 tables
])
def test_large_batch_codes_equal_oracle(fl, n, d, K, L):
    X, _, _ = synth.dense_relu(N=n, d=d, n_centres=40, nq=1)
    gi = fl.Index(X[:300], fl.SRP_BF16, K, L, 2, 8, seed=80)
    oi = oracle.OracleIndex(oracle.SRP_BF16, X[:300], K, L, 2, 8, 80)
    log("large srp batch", n, d, K, L)
    want = oi.hash(X)
    got = gi.debug_hash(X)
    assert np.array_equal(got, want)
    assert np.array_equal(gi.debug_hash(X[:100]), want[:100])


@pytest.mark.parametrize("n,d,K,L", [
    (65536, 33, 6, 5),    # 1,024 tiles: two sets of fragments
    (65537, 33, 6, 5),    # one more: one set, an odd count of 32-wide steps
    (65537, 288, 3, 5),   # two sets again, an odd count of steps
    (33000, 100, 13, 5),  # 1,032 tiles of two columns of workgroups, one set
    (33000, 640, 13, 5),  # two sets
])
def test_fp32_fragment_sets_equal_oracle(fl, n, d, K, L):
    """fp32 rows on both sides of the rule that picks one or two sets of operand
    fragments."""
    rng = np.random.default_rng(n + d)
    log("fp32 fragments", n, d, K * L)
    x = rng.standard_normal((n, d)).astype(np.float32)
    gi = fl.Index(x[:500], 0, K, L, 2, 50, seed=99)
    w = oracle.hyperplanes(99, K * L, d)
    assert np.array_equal(gi.debug_hash(x), oracle.srp_codes(x.astype(np.float64), 99, K, L, w=w))
