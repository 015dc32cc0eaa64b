"""Scans at the sizes where their form changes: one block, tiles that sum
the tiles before their own, and scanned tile sums.  A trie over (a, b) with
n0 distinct a scans one entry per level-1 set (its bitset words), one per
tile of 256 rows (its level sizes) and the radix histograms; its levels and
bitset words must be numpy's.  All integers: compared exactly."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lh():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1708_07859_amd import lh as binding
    return binding


# entries: one block takes 16384 of them, a tile 2048, self-summing tiles 1024 x 2048
SIZES = [1, 2, 255, 257, 16383, 16384, 16385, 16384 + 2048, 1024 * 2048 - 1, 1024 * 2048, 1024 * 2048 + 1]


@pytest.mark.parametrize("n0", SIZES)
def test_levels_at_scan_edges(lh, n0):
    print("sets", n0, file=sys.stderr, flush=True)
    a = np.arange(n0, dtype=np.uint32)
    a = np.concatenate([a, a[::3]])                      # every third set has two elements
    b = ((a.astype(np.uint64) * 7) % 1000).astype(np.uint32)
    b[n0:] += 1 + 40 * (a[n0:] & 3)                      # one word, or a word and the next
    t = lh.trie_build([a, b])
    try:
        order = np.lexsort((b, a))
        k0, o0 = t.read_level(0)
        k1, _ = t.read_level(1)
        assert np.array_equal(k0, np.arange(n0, dtype=np.uint32))
        assert np.array_equal(k1, b[order])
        assert np.array_equal(np.diff(o0.astype(np.int64)), 1 + (np.arange(n0) % 3 == 0))
        lo = (b[:n0] >> 6).astype(np.int64)
        hi = lo.copy()
        hi[::3] = b[n0:] >> 6
        pair = np.arange(n0) % 3 == 0
        span = np.zeros(n0, np.int64)
        span[pair] = b[n0:].astype(np.int64) - b[:n0][pair] + 1
        bits = ~pair | (span <= 64)                       # the plain rule: span <= 32 x card
        assert t.info()["level_bitsets"][1] == bits.sum()
        assert t.info()["level_words"][1] == ((hi - lo + 1) * bits).sum()
    finally:
        t.free()
