"""The index build's kernels at the sizes where they change path, bit for bit
against the oracle: bucket runs just below, at and above the length a thread
per point handles, across the tiles of the run and sort kernels, in grids of
every row width and both cell widths, built in one pass and grown by inserts;
and a build whose tables do not fit one batch, against the definition."""
import numpy as np
import pytest

import oracle
from gpu_common import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_2106_11565_amd as flinng
    flinng.lib()
    return flinng


def _sets(vals):
    return np.asarray(vals, dtype=np.uint32), np.arange(len(vals) + 1, dtype=np.uint64)


def _same(gi, oi):
    offs, cells, groups = gi.export()
    assert np.array_equal(groups, oi.g)
    assert np.array_equal(offs, oi.offsets)
    assert np.array_equal(cells, oi.cells)


@pytest.mark.parametrize("R,B,bits", [(1, 7, 1), (2, 64, 8), (3, 100, 9), (4, 4093, 16),
                                      (8, 300, 17), (16, 4100, 24), (5, 1, 12)])
def test_lists_of_runs_of_every_length(fl, R, B, bits):
    rng = np.random.default_rng(R * 1000 + B)
    lens = [1] * 700 + [2] * 150 + [3, 5, 7, 8, 15, 16, 17] * 12
    lens += [31, 32, 33, 34, 63, 64, 65, 127, 128, 129, 255, 256, 257, 1000, 1024, 1025, 4097]
    lens += [32] * 40 + [33] * 40
    vals = np.repeat(rng.permutation(len(lens)).astype(np.uint64) * 2654435761 % 2**32,
                     lens)
    vals = rng.permutation(vals)
    n0 = len(vals) - 3001
    log("runs", R, B, bits, "points", len(vals))
    gi = fl.Index(_sets(vals[:n0]), fl.MINHASH_U32, 1, 3, R, B, seed=5, bucket_bits=bits)
    oi = oracle.OracleIndex(oracle.MINHASH_U32, _sets(vals[:n0]), 1, 3, R, B, 5, bucket_bits=bits)
    _same(gi, oi)
    for a, b in ((n0, n0 + 1), (n0 + 1, n0 + 34), (n0 + 34, len(vals))):
        gi.insert(_sets(vals[a:b]))
        oi.insert(_sets(vals[a:b]))
        _same(gi, oi)


def test_lists_in_batches_of_tables(fl):
    """2.1 million points in 255 tables: the sorted points of all tables pass
    the scratch limit, so the lists are made in two batches and joined."""
    n, L, B, bits = 2_100_000, 255, 50, 7
    vals = np.arange(n, dtype=np.uint64) * 2654435761 % 2**32
    gi = fl.Index(_sets(vals), fl.MINHASH_U32, 1, L, 1, B, seed=9, bucket_bits=bits)
    offs, cells, groups = gi.export()
    codes = np.concatenate([gi.debug_hash(_sets(vals[a:a + 300_000])) for a in range(0, n, 300_000)])
    key = groups[0].astype(np.uint32)
    assert offs[0, 0] == 0 and offs[-1, -1] == len(cells)
    assert np.array_equal(offs[1:, 0], offs[:-1, -1])
    for t in (0, 1, 100, 248, 249, 250, 251, 254):
        want = np.unique(codes[:, t] * np.uint32(64) + key)
        lo, hi = int(offs[t, 0]), int(offs[t, -1])
        assert np.array_equal(cells[lo:hi], want % 64), t
        assert np.array_equal(offs[t] - offs[t, 0],
                              np.searchsorted(want // 64, np.arange(2**bits + 1))), t
