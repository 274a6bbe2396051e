"""The sparse query kernel, variant by variant, and the queries it defers,
against the oracle, bit for bit.  The tables below are made so that a variant
serves them; that they are is checked from the exported lists."""
import numpy as np
import pytest

import oracle
from gpu_common import log

pytestmark = pytest.mark.gpu

# a variant's threads: mean list entries per query that it takes, entries of one
# query that it takes, queries in a batch from which it does (general kernel of
# 256 or of 1024 threads)
RULES = {128: (0, 409, 1024), 256: (410, 1638, 4096), 512: (1639, 4915, 8192)}


@pytest.fixture(scope="module")
def fl():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_2106_11565_amd as flinng
    flinng.lib()
    return flinng


def _sets(vals):
    return np.asarray(vals, dtype=np.uint32), np.arange(len(vals) + 1, dtype=np.uint64)


def _entries(gi, vals):
    """List entries that each of these one-item sets meets as a query."""
    offs, _, _ = gi.export()
    codes = gi.debug_hash(_sets(vals))
    t = np.arange(codes.shape[1])[None, :]
    return (offs[t, codes + np.uint32(1)] - offs[t, codes]).sum(1)


def _value(i):
    return np.asarray(i, dtype=np.uint64) * 2654435761 % 2**32


@pytest.mark.parametrize("T,R,B,L,copies,heavy", [
    (128, 4, 1000, 8, 1, 80),     # Bp is no multiple of 32
    (128, 2, 37, 70, 1, 30),      # L > 64; cells of 160 members
    (128, 16, 33, 8, 1, 30),      # a word and a bit per repetition
    (128, 1, 500, 40, 2, 90),     # nothing to filter by
    (128, 8, 5000, 20, 1, 25),    # 1024-thread grid
    (256, 8, 5000, 60, 1, 25),    # 16-bit cells
    (256, 4, 16384, 200, 1, 40),  # L > 128
    (256, 5, 14000, 30, 5, 90),   # 32-bit cells, one member in most cells
    (512, 8, 8190, 60, 5, 60),    # Bp is no multiple of 32
    (512, 2, 38000, 100, 15, 90),  # 32-bit cells
])
def test_every_variant_equals_oracle(fl, T, R, B, L, copies, heavy):
    """Sets of one item: a query meets its copies' cells in every table.  Most
    points have `copies` copies, two have `heavy` (their queries are deferred),
    some queries none (zero-count completion).  Also after an insert, whose
    cells differ in size, and with every query deferred."""
    rng = np.random.default_rng(R * 77 + B)
    wide = B > 2000  # the general kernel takes 1024 threads
    n = 40000 if B > 8192 else 20000 if wide else 6000
    vals = np.arange(n, dtype=np.uint64) // copies
    at = rng.permutation(n)[:2 * heavy]
    vals[at[:heavy]], vals[at[heavy:]] = 10**6, 10**6 + 1
    vals = rng.permutation(_value(vals))
    n0 = n - 57
    gi = fl.Index(_sets(vals[:n0]), fl.MINHASH_U32, 1, L, R, B, seed=3, bucket_bits=20)
    oi = oracle.OracleIndex(oracle.MINHASH_U32, _sets(vals[:n0]), 1, L, R, B, 3, bucket_bits=20)
    lo, hi, most = RULES[T]
    mean = _entries(gi, rng.choice(vals[:n0], 2000)).mean()
    two = _entries(gi, _value([10**6, 10**6 + 1]))
    log("sparse", T, R, B, L, "mean entries", mean, "heavy", two)
    assert 1.1 * lo <= mean <= 0.9 * hi and two.min() > most
    q = np.concatenate([rng.choice(vals, 150), _value([10**6, 10**6 + 1] * 3),
                        rng.integers(2**31, 2**32, 20).astype(np.uint64)])
    nq = 400 if wide else 4200
    pick = np.arange(nq) % len(q)
    for step in range(2):
        for k in (1, 10, 64):
            want = oi.query(_sets(q), k)
            for pers in (False, True):
                got = gi.query(_sets(q[pick]), k, persistent=pers)
                assert np.array_equal(got[0], want[0][pick]), (step, k, pers)
                assert np.array_equal(got[1], want[1][pick]), (step, k, pers)
            w = oi.query(_sets(_value([10**6, 10**6 + 1])), k)
            got = gi.query(_sets(_value(10**6 + np.arange(nq) % 2)), k)
            assert np.array_equal(got[0], w[0][np.arange(nq) % 2]), (step, k)
            assert np.array_equal(got[1], w[1][np.arange(nq) % 2]), (step, k)
        if step == 0:
            gi.insert(_sets(vals[n0:]))
            oi.insert(_sets(vals[n0:]))


@pytest.mark.parametrize("T,R,B,L,copies,heavy", [
    (128, 2, 601, 70, 1, 30),   # L > 64; nearly an eighth of the cells touched
    (128, 16, 97, 8, 1, 30),    # three words and a bit per repetition
])
def test_every_variant_of_small_grids_equals_oracle(fl, T, R, B, L, copies, heavy):
    test_every_variant_equals_oracle(fl, T, R, B, L, copies, heavy)


@pytest.mark.parametrize("R,B,L", [(4, 1000, 8), (8, 5000, 20)])
@pytest.mark.parametrize("nq", [4097, 66001])  # one, and several chunks of 64 per workgroup
@pytest.mark.parametrize("every", [1, 7, 64, 1001])
def test_deferred_queries_of_large_batches(fl, R, B, L, nq, every):
    """One query in `every` is deferred: runs of them, one in each chunk that
    the workgroups share, and few."""
    rng = np.random.default_rng(nq + every)
    n = 10000
    vals = np.arange(n, dtype=np.uint64)
    vals[rng.permutation(n)[:80]] = 10**6
    vals = _value(vals)
    gi = fl.Index(_sets(vals), fl.MINHASH_U32, 1, L, R, B, seed=4, bucket_bits=20)
    assert _entries(gi, _value([10**6]))[0] > 1024 and _entries(gi, vals[:2000]).mean() < 370
    q = np.concatenate([vals[:200], _value([10**6])])
    small = gi.query(_sets(q), 10)  # too few for the sparse kernel
    pick = np.where(np.arange(nq) % every == every // 2, 200, np.arange(nq) % 200)
    got = gi.query(_sets(q[pick]), 10)
    assert np.array_equal(got[0], small[0][pick]) and np.array_equal(got[1], small[1][pick])


@pytest.mark.parametrize("T,copies,R,B,L", [(128, 2, 2, 64, 4), (256, 10, 8, 8192, 10),
                                            (512, 30, 8, 8192, 10)])
def test_persistent_batches_at_the_grid_limit(fl, T, copies, R, B, L):
    """A batch whose sparse launch, a workgroup per query, would reach 2^32
    threads is answered by the persistent grid; one query fewer by the sparse
    kernel.  The answers are those of the same queries in a small batch."""
    import ctypes
    import torch
    n = max(300 * copies, B)
    vals = (np.arange(n, dtype=np.uint64) % (n // copies)) * 2654435761 % 2**32
    ix = fl.Index(_sets(vals), fl.MINHASH_U32, 1, L, R, B, seed=13, bucket_bits=20)
    met = _entries(ix, vals[:300]).mean()
    assert 1.1 * RULES[T][0] <= met <= 0.9 * RULES[T][1]
    base = torch.from_numpy(ix.debug_hash(_sets(vals[:300])).view(np.int32)).cuda()

    def run(codes):
        nq = codes.shape[0]
        ids = torch.full((nq, 1), -7, dtype=torch.int32, device="cuda")
        sc = torch.full((nq, 1), -7, dtype=torch.int32, device="cuda")
        s = torch.cuda.current_stream().cuda_stream
        fl.check(fl.lib().flinng_query_codes(
            ix.handle, ctypes.c_void_p(codes.data_ptr()), nq, 1, ctypes.c_void_p(ids.data_ptr()),
            ctypes.c_void_p(sc.data_ptr()), 1, None, ctypes.c_void_p(s)))
        torch.cuda.synchronize()
        return ids, sc

    want = run(base)
    assert int(want[1].min()) == L
    for nq in (2**32 // T - 1, 2**32 // T):
        log("grid limit", T, "queries", nq, "entries", met)
        rows = torch.arange(nq, device="cuda", dtype=torch.int32) % 300
        got = run(base[rows.long()])
        for g, w in zip(got, want):
            assert torch.equal(g, w[rows.long()])
