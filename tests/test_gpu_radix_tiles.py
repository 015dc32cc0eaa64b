"""The radix sort at the edges of its tiles (4096 keys) and of its look-back
groups (32 tiles), for keys of one word, of two (65 to 96 bits) and wider,
and for each thing that can travel with them: nothing (a set), one
annotation, one meta column, both (the row permutation).  Checked against
numpy: levels by sorting, sums of multiples of 1/8 (exact in a double, so
equality is the tolerance), meta columns through GROUP BY."""
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


SIZES = [1, 4095, 4096, 4097, 131071, 131072, 131073, 300_001]
KEYS = {"7 bits": [7], "one word": [13, 12], "64 bits": [32, 32], "65 bits": [32, 33 - 1, 1], "96 bits": [32, 32, 32],
        "97 bits": [32, 32, 32, 1], "tail": [10, 20]}


@pytest.mark.parametrize("carry", ["set", "anno", "meta", "both"])
@pytest.mark.parametrize("keys", list(KEYS))
def test_sorted_rows(lh, keys, carry):
    rng = synth.rng_for(77)
    bits = KEYS[keys]
    for n in SIZES:
        print(keys, carry, n, file=sys.stderr, flush=True)
        # few distinct values per column (runs), the largest of each width among them
        cols = []
        for b in bits:
            pool = rng.integers(0, 1 << b, 40, dtype=np.uint64)
            pool[0] = (1 << b) - 1
            c = pool[rng.integers(0, 40, n)].astype(np.uint32)
            c[0] = (1 << b) - 1
            cols.append(c)
        if keys == "tail":
            cols[1].sort()
        v = rng.integers(-80, 81, n) / 8.0
        m = rng.integers(0, 5, n).astype(np.uint32)
        k = len(cols)
        bag = carry != "set"
        t = lh.trie_build(cols, [v] if carry in ("anno", "both") else [], [m] if carry in ("meta", "both") else [],
                          bag=bag)
        group = [(0, 0)] if carry in ("meta", "both") else []
        p = lh.plan(k, [(t, list(range(k)), 0 if carry in ("anno", "both") else -1)], out=list(range(k)), group=group,
                    agg="sum" if carry in ("anno", "both") else "count")
        got = lh.join_aggregate([p])[0].to_host()
        p.free()
        t.free()
        rows = np.stack(cols + ([m] if group else []), 1)
        want, at, cnt = np.unique(rows, axis=0, return_inverse=True, return_counts=True)
        assert np.array_equal(got["keys"], want)
        assert np.array_equal(got["counts"], np.ones(len(want), np.uint64) if not bag else cnt.astype(np.uint64))
        if carry in ("anno", "both"):
            assert np.array_equal(got["sums"], np.bincount(at.ravel(), weights=v, minlength=len(want)))
