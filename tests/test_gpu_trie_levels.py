"""Tries of one to eight levels under every layout, from empty to several
tiles: levels against numpy, presorted and shuffled input alike, bitset
counts consistent with the layout, and a self-join that reaches every level
through positions inside its sets (the rank of a bitset word).  Integers:
compared exactly."""
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


@pytest.mark.parametrize("layout", ["plain", "uint", "bitset"])
@pytest.mark.parametrize("levels", [1, 2, 3, 8])
@pytest.mark.parametrize("bag", [False, True])
def test_levels(lh, levels, layout, bag):
    rng = synth.rng_for(levels)
    for n in (0, 1, 2, 64, 255, 257, 5000, 20_000):
        for order in ("shuffled", "sorted"):
            print(levels, layout, bag, n, order, file=sys.stderr, flush=True)
            # dense first level, runs of dense and of sparse sets below
            cols = [rng.integers(0, 300 if l % 2 == 0 else 7, n).astype(np.uint32) * (1 if l % 3 else 3)
                    for l in range(levels)]
            if order == "sorted" and n:
                at = np.lexsort(cols[::-1])
                cols = [c[at] for c in cols]
            t = lh.trie_build(cols, bag=bag, layout=layout)
            try:
                info = t.info()
                rows = np.unique(np.stack(cols, 1), axis=0) if n else np.zeros((0, levels), np.uint32)
                for l in range(levels):
                    nodes, first = np.unique(rows[:, :l + 1], axis=0, return_index=True)
                    k, o = t.read_level(l)
                    assert np.array_equal(k, nodes[:, l] if n else k[:0])
                    assert info["level_size"][l] == len(nodes)
                    if l + 1 < levels and n:
                        below = np.unique(rows[:, :l + 2], axis=0)
                        assert np.array_equal(np.diff(o.astype(np.int64)), np.unique(below[:, :l + 1], axis=0, return_counts=True)[1])
                    if layout == "uint":
                        assert info["level_bitsets"][l] == 0 and info["level_words"][l] == 0
                if bag and n:
                    runs = np.diff(t.read_level(levels - 1)[1].astype(np.int64))
                    assert np.array_equal(runs, np.unique(np.stack(cols, 1), axis=0, return_counts=True)[1])
                p = lh.plan(levels, [(t, list(range(levels)), -1)] * 2, out=list(range(levels)), agg="count")
                got = lh.join_aggregate([p])[0].to_host()
                p.free()
                assert np.array_equal(got["keys"], rows)
                want = np.unique(np.stack(cols, 1), axis=0, return_counts=True)[1] if n else np.zeros(0, np.int64)
                assert np.array_equal(got["counts"], (want ** 2 if bag else np.ones(len(rows))).astype(np.uint64))
            finally:
                t.free()
