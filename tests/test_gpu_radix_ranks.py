"""The radix sort's ranking inside a wave, where its lanes share digits from one
item to the next: every pass has to keep the order that the passes before it
made.  Keys are read back as a trie's level and checked against numpy."""
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


# the digit of the second pass, by position; the first pass's digits are random
PATTERNS = {
    "one": lambda i: 0 * i,                   # all lanes, all items
    "per item": lambda i: i // 64 % 7,        # all lanes of an item
    "two": lambda i: i % 2,
    "neighbours": lambda i: i // 2 % 32,
    "by lane": lambda i: i % 64,              # a lane's own, the same in every item
    "rotating": lambda i: (i + i // 64) % 64, # another lane's of the item before
    "descending": lambda i: 255 - i // 16 % 256,
}


@pytest.mark.parametrize("n", [64, 513, 4096, 4097, 150_001])
@pytest.mark.parametrize("pattern", list(PATTERNS))
def test_ranks(lh, pattern, n):
    print(pattern, n, file=sys.stderr, flush=True)
    rng = np.random.default_rng(n)
    i = np.arange(n)
    for top in (8, 24):     # two passes, and four with the digits below the last two random
        key = (PATTERNS[pattern](i) << top | rng.integers(0, 1 << top, n)).astype(np.uint32)
        t = lh.trie_build([key], bag=True)
        keys, offs = t.read_level(0)
        want, count = np.unique(key, return_counts=True)
        assert np.array_equal(keys, want)
        assert np.array_equal(np.diff(offs), count)
        t.free()
