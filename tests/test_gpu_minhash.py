"""MinHash codes at the edges of the kernel's split, against the oracle: function
counts around multiples of 64 (whole passes, and a last pass whose functions
share the lanes), set sizes around the 128 items staged at a time, tiny sets
whose values may all have the top bit, items of both widths, and the same sets
given as text with the longest and the shortest n-grams."""
import numpy as np
import pytest

import oracle
from gpu_common import log

pytestmark = pytest.mark.gpu

SIZES = [0, 1, 1, 2, 3, 5, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 700]


@pytest.fixture(scope="module")
def fl():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_2106_11565_amd as flinng
    flinng.lib()
    return flinng


@pytest.mark.parametrize("family", [2, 3])
@pytest.mark.parametrize("K,L", [(1, 2), (3, 11), (1, 63), (2, 32), (5, 13), (1, 128), (3, 43), (32, 255)])
def test_codes_at_the_splits(fl, family, K, L):
    rng = np.random.default_rng(K * 300 + L)
    sizes = np.array(SIZES * 2)
    offs = np.zeros(len(sizes) + 1, dtype=np.uint64)
    offs[1:] = np.cumsum(sizes)
    dt = np.uint64 if family == 3 else np.uint32
    items = rng.integers(0, 2**64 if family == 3 else 2**32, int(offs[-1]), dtype=np.uint64).astype(dt)
    log("minhash splits", family, K, L)
    gi = fl.Index((items, offs), family, K, L, 2, 5, seed=K + L, bucket_bits=19)
    want = oracle.minhash_codes(items.astype(np.uint64), offs, K + L, K, L, 19)
    assert np.array_equal(gi.debug_hash((items, offs)), want)


@pytest.mark.parametrize("family", [2, 3])
@pytest.mark.parametrize("gram,radix", [(1, 256), (3, 40), (20, 4), (32, 4), (64, 2), (8, 256)])
def test_text_codes_at_the_splits(fl, family, gram, radix):
    rng = np.random.default_rng(gram)
    sizes = np.array([0, 1, gram - 1, gram, gram + 1] + [gram + s for s in SIZES])
    offs = np.zeros(len(sizes) + 1, dtype=np.uint64)
    offs[1:] = np.cumsum(sizes)
    sym = rng.integers(0, radix, int(offs[-1])).astype(np.uint8)
    key = 0x9E3779B97F4A7C15
    K, L = 3, 23
    log("minhash text", family, gram, radix)
    it, of = oracle.text_items(sym, offs, gram, radix, key, 64 if family == 3 else 32)
    ga = fl.Index((sym, offs), family, K, L, 2, 5, seed=8, bucket_bits=18, text=(gram, radix, key))
    oi = oracle.OracleIndex(oracle.MINHASH_U64 if family == 3 else oracle.MINHASH_U32, (it, of), K, L, 2,
                            5, 8, bucket_bits=18)
    a, b = ga.export(), (oi.offsets, oi.cells, oi.g)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    want = oi.query((it, of), 7)
    got = ga.query_text((sym, offs), (gram, radix, key), 7)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.parametrize("family", [2, 3])
@pytest.mark.parametrize("K,L", [(1, 1), (2, 4), (1, 9), (1, 12), (1, 21), (1, 22), (1, 23), (1, 32), (1, 33),
                                 (1, 40), (1, 48), (5, 12), (8, 8), (5, 21), (8, 13)])
def test_codes_where_sets_are_not_staged(fl, family, K, L):
    """Function counts whose sets are read by the lanes themselves up to a size, or
    whose functions are taken in several passes above one; sets around the sizes."""
    rng = np.random.default_rng(K * 70 + L)
    LK = K * L
    near = [8, 12, 32, 16 * (64 // LK if LK < 64 else 1)]
    sizes = np.array([0, 1, 2] + [s + d for s in near for d in (-1, 0, 1, 2)] + [130, 300])
    offs = np.zeros(len(sizes) + 1, dtype=np.uint64)
    offs[1:] = np.cumsum(sizes)
    dt = np.uint64 if family == 3 else np.uint32
    items = rng.integers(0, 2**64 if family == 3 else 2**32, int(offs[-1]), dtype=np.uint64).astype(dt)
    log("minhash not staged", family, K, L)
    gi = fl.Index((items, offs), family, K, L, 2, 5, seed=K + L, bucket_bits=19)
    want = oracle.minhash_codes(items.astype(np.uint64), offs, K + L, K, L, 19)
    assert np.array_equal(gi.debug_hash((items, offs)), want)
    # the same as text: sets of one-symbol windows
    sym = rng.integers(0, 256, int(offs[-1])).astype(np.uint8)
    it, of = oracle.text_items(sym, offs, 1, 256, 77, 64 if family == 3 else 32)
    got = gi.query_text((sym, offs), (1, 256, 77), 3)
    want = gi.query((it, of), 3)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
