"""Every order of a four-level relation against every other: a plan that
fixes the attribute order re-sorts the relation's trie (sorting only the
levels that the trie's own order leaves unsorted), with and without a
selection, as a set, as a bag with one annotation (which travels with the
keys) and as a bag with two columns (which follow by permutation).  Results
must not depend on the order; numpy gives them (sums of multiples of 1/8 are
exact in a double)."""
import itertools
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


@pytest.mark.parametrize("kind", ["set", "anno", "both"])
@pytest.mark.parametrize("build", [[0, 1, 2, 3], [3, 1, 0, 2]])
def test_every_order(lh, kind, build):
    rng = synth.rng_for(12)
    n = 9000
    cols = [rng.integers(0, d, n).astype(np.uint32) for d in (5, 300, 17, 40)]
    v = rng.integers(-80, 81, n) / 8.0
    m = rng.integers(0, 3, n).astype(np.uint32)
    bag = kind != "set"
    t = lh.trie_build(cols, [v] if bag else [], [m] if kind == "both" else [], level_order=build, bag=bag)
    other = lh.trie_build([np.arange(0, 300, 2, dtype=np.uint32)])
    rows = np.stack(cols, 1)
    if not bag:
        rows = np.unique(rows, axis=0)
    for eq in (None, 3):
        keep = rows[:, 1] % 2 == 0
        if eq is not None:
            keep &= rows[:, 0] == eq
        want, at, cnt = np.unique(rows[keep][:, [1, 3]], axis=0, return_inverse=True, return_counts=True)
        for order in itertools.permutations(range(4)):
            print(kind, build, eq, order, file=sys.stderr, flush=True)
            p = lh.plan(4, [(t, [0, 1, 2, 3], 0 if bag else -1), (other, [1], -1)], out=[1, 3],
                        agg="sum" if bag else "count", attr_order=list(order), policy="fixed",
                        filters=[] if eq is None else [{"atom": 0, "kind": "eq_key", "col": 0, "eq": eq}])
            got = lh.join_aggregate([p])[0].to_host()
            p.free()
            assert np.array_equal(got["keys"], want)
            assert np.array_equal(got["counts"], cnt.astype(np.uint64))
            if bag:
                assert np.array_equal(got["sums"], np.bincount(at.ravel(), weights=v[keep], minlength=len(want)))
