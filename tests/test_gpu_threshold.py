"""The fixed-threshold query against the oracle where its kernel changes
course: lists counted as one sequence and a table at a time, few positive cells
(whose members are filtered and ranked) and many (walked in order), answers and
cells that pass the lists in LDS, R = 1 (nothing to filter by), 256 and 1024
threads, 16- and 32-bit cells.  The ids come in order of the cell in the
repetition with the fewest positive cells, then of the id."""
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
    (20011, 1, 40, 8, 8),       # no filter; cells of 500 members: answers pass the list
    (20011, 2, 40, 6, 12),      # long lists
    (20003, 3, 200, 10, 20),    # few to most cells positive, by t
    (20000, 5, 1021, 12, 24),   # short lists; rows checked behind the filter
    (30000, 8, 8192, 8, 16),    # 1024 threads, 16-bit cells
    (30001, 8, 16384, 10, 5),   # 1024 threads, 32-bit cells
    (300, 2, 300, 6, 4),        # one member per cell
])
def test_threshold_equals_oracle_in_order(fl, N, R, B, K, L):
    X, Q, _ = synth.dense_gmm(N=N, d=24, n_centres=max(3, N // 300), sigma=0.2, nq=24)
    gi = fl.Index(X, 0, K, L, R, B, seed=78)
    oi = oracle.OracleIndex(oracle.SRP_F32, X, K, L, R, B, 78)
    cnt = oi.counts(oi.hash(Q))
    npos = set()
    for t in (0, 1, 2, L // 2, L - 1, L):
        want = []
        for c in cnt:
            ids = np.nonzero(oracle.query_fixed_t(c, oi.g, B, t))[0]
            n = (np.asarray(c).reshape(R, B) >= t).sum(axis=1)
            rep = int(np.argmin(n))
            npos.add(int(n[rep]))
            want.append(ids[np.lexsort((ids, oi.g[rep][ids]))])
        full = max(1, max(len(w) for w in want))
        for m in (full, max(1, full // 2), 0):
            log("threshold", N, R, B, "t", t, "slots", m)
            ids, counts = gi.query_threshold(Q, t, m)
            assert np.array_equal(counts, [len(w) for w in want])
            for i, w in enumerate(want):
                n = min(m, len(w))
                assert np.array_equal(ids[i][:n], w[:n]), (t, i)
                assert np.all(ids[i][n:] == 0xFFFFFFFF), (t, i)
    log("positive cells", sorted(npos)[:6], "to", max(npos))


@pytest.mark.parametrize("N,R,B,K,L", [
    (900, 1, 4, 8, 8), (1000, 1, 4, 8, 8), (1100, 1, 4, 8, 8),  # one cell about fills the answer's list
    (8000, 1, 400, 8, 8),      # few cells, whose members pass it together
    (5000, 4, 100, 3, 8),      # every cell positive: one group left behind the filter
    (3000, 16, 24, 4, 10),     # thirteen left
])
def test_threshold_where_members_pass_by_the_dozen(fl, N, R, B, K, L):
    test_threshold_equals_oracle_in_order(fl, N, R, B, K, L)
