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


@pytest.mark.parametrize("nq,k", [(64, 10), (65, 10), (1024, 65), (1025, 65)])
@pytest.mark.parametrize("K", [4, 14])  # many and few list entries per query
def test_batch_sizes_around_the_workgroup_rule(fl, nq, k, K):
    X, Q, _ = synth.dense_gmm(N=8000, d=16, n_centres=30, sigma=0.2, nq=nq)
    gi = fl.Index(X, 0, K, 10, 3, 64, seed=79)
    oi = oracle.OracleIndex(oracle.SRP_F32, X, K, 10, 3, 64, 79)
    want = oi.query(Q, k)
    for pers in (False, True):
        log("batch size", nq, "k", k, "K", K, "persistent", pers)
        got = gi.query(Q, k, persistent=pers)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), pers


@pytest.mark.parametrize("R,K,L,nq", [
    (3, 14, 10, 256), (3, 14, 10, 257),  # any number of list entries
    (3, 4, 10, 512), (3, 4, 10, 513),    # some 1,900 per query
    (8, 2, 64, 1024), (8, 2, 64, 1025),  # all 32,768
])
@pytest.mark.parametrize("k", [65, 700])  # buffers of the smallest and of a larger size
def test_general_k_around_the_workgroup_rule(fl, R, K, L, nq, k):
    X, Q, _ = synth.dense_gmm(N=8000, d=16, n_centres=30, sigma=0.2, nq=nq)
    gi = fl.Index(X, 0, K, L, R, 64, seed=81)
    oi = oracle.OracleIndex(oracle.SRP_F32, X, K, L, R, 64, 81)
    want = oi.query(Q, k)
    log("general k, batch size", nq, "k", k, "R", R, "K", K, "L", L)
    got = gi.query(Q, k)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


def _sets(vals):
    return np.asarray(vals, dtype=np.uint32), np.arange(len(vals) + 1, dtype=np.uint64)


@pytest.mark.parametrize("R,B,L", [
    (4, 1000, 8),    # 128 threads; Bp is no multiple of 32
    (2, 37, 70),     # L > 64; cells of 160 members
    (16, 33, 8),     # a word and a bit per repetition
    (1, 500, 40),    # nothing to filter by
    (8, 5000, 60),   # 1024-thread grid, 16-bit cells
    (5, 14000, 30),  # 1024-thread grid, 32-bit cells, one member in most cells
])
def test_sparse_and_deferred_queries_equal_oracle(fl, R, B, L):
    """Sets of one item each, so that a query meets exactly its copies' cells
    in every table: most have a few copies, some so many that their entries
    pass the sparse kernel's limit and the general kernel takes over, and some
    queries have none (zero-count completion). Also after an insert, whose
    cells differ in size."""
    rng = np.random.default_rng(R * 77 + B)
    n = 20000 if B > 2000 else 6000
    vals = rng.integers(0, n // 3, n).astype(np.uint64)
    for j in range(3):
        vals[rng.permutation(n)[:1500 // (L // 8 + R) + 40]] = 10**6 + j
    vals = vals * 2654435761 % 2**32
    n0 = n - 57
    gi = fl.Index(_sets(vals[:n0]), fl.MINHASH_U32, 1, L, R, B, seed=3, bucket_bits=20)
    oi = oracle.OracleIndex(oracle.MINHASH_U32, _sets(vals[:n0]), 1, L, R, B, 3, bucket_bits=20)
    q = np.concatenate([rng.choice(vals, 150), (10**6 + np.arange(3)) * 2654435761 % 2**32,
                        rng.integers(2**31, 2**32, 20).astype(np.uint64)])
    reps = 4200 // len(q) + 1  # a batch that fills the chip
    log("sparse", R, B, L, "entries", gi.info.list_entries)
    for step in range(2):
        for k in (1, 10, 64):
            want = oi.query(_sets(q), k)
            for pers in (False, True):
                got = gi.query(_sets(np.tile(q, reps)), k, persistent=pers)
                assert np.array_equal(got[0], np.tile(want[0], (reps, 1))), (step, k, pers)
                assert np.array_equal(got[1], np.tile(want[1], (reps, 1))), (step, k, pers)
        if step == 0:
            gi.insert(_sets(vals[n0:]))
            oi.insert(_sets(vals[n0:]))
