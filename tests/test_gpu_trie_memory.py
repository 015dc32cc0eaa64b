"""What a trie holds on the device: a relation of a set's keys as bitsets has
eight bytes a word and, where nothing lies below the level, no more."""
import sys

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lh():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1708_07859_amd import lh as binding
    return binding


@pytest.mark.parametrize("bag", [False, True])
@pytest.mark.parametrize("levels", [1, 2])
def test_wide_bitsets(lh, levels, bag):
    """300,000 keys over 1.2e9 values: 18.75 M words, 150 MB."""
    import torch
    print(levels, bag, file=sys.stderr, flush=True)
    rng = synth.rng_for(68)
    n, spread = 300_000, 4000
    keys = np.arange(n, dtype=np.uint32) * spread + rng.integers(0, spread, n).astype(np.uint32)
    cols = [torch.from_numpy(c.view(np.int32)).cuda() for c in [np.full(n, 3, np.uint32)] * (levels - 1) + [keys]]
    probe = np.sort(np.unique(np.concatenate([keys[::7], rng.integers(0, n * spread, 20_000).astype(np.uint32)])))
    tp = lh.trie_build([probe])
    warm = lh.trie_build(cols, bag=bag, layout="uint")
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    t = lh.trie_build(cols, bag=bag, layout="bitset")
    held = free - torch.cuda.mem_get_info()[0]
    words = t.info()["level_words"][-1]
    print("words", words, "held", held, file=sys.stderr, flush=True)
    assert words > 18_000_000
    # (a set's words alone; a bag's with their ranks; 32 MiB for the level's keys and offsets and for roundings)
    assert held <= words * (12 if bag else 8) + (32 << 20)
    # the ranks give positions: rows of a bag, and the children of a level
    k = levels
    p = lh.plan(k, [(t, list(range(k)), -1), (tp, [k - 1], -1)], out=[k - 1], agg="count",
                attr_order=[k - 1] + list(range(k - 1)), policy="fixed")
    got = lh.join_aggregate([p])[0].to_host()
    want = np.intersect1d(keys, probe)
    assert np.array_equal(got["keys"][:, 0], want)
    assert (got["counts"] == 1).all()
    del warm
