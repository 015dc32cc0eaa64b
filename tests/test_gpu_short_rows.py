"""Leaf and frontier units of eight lanes (sets of at most 24 elements on
average) and of a whole wave, at row lengths around their edges, with hub
rows among short ones: sums that one unit stores, that several units add,
and groups of several frontier rows; two and three atoms.  Values are
multiples of 1/8, so every sum is exact in a double and numpy's must be
equal."""
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


EDGES = [1, 2, 7, 8, 9, 31, 32, 33, 63, 64, 65, 255, 256, 257, 1023, 1025, 5000, 70_000]


def matrix(rng, short_rows):
    """Rows of the edge lengths among short_rows rows of one element."""
    deg = np.concatenate([EDGES, np.ones(short_rows, np.int64)])
    deg = deg[rng.permutation(len(deg))]
    n = 100_000
    rows = np.repeat(np.arange(len(deg)), deg).astype(np.uint32)
    cols = np.concatenate([rng.choice(n, d, replace=False) for d in deg]).astype(np.uint32)
    return len(deg), n, rows, cols, rng.integers(-80, 81, len(rows)) / 8.0


@pytest.mark.parametrize("short_rows", [0, 40, 20_000])
@pytest.mark.parametrize("atoms", [2, 3])
def test_row_sums(lh, short_rows, atoms):
    print("rows", short_rows, "atoms", atoms, file=sys.stderr, flush=True)
    rng = synth.rng_for(90 + atoms)
    m, n, rows, cols, vals = matrix(rng, short_rows)
    keep = np.sort(rng.choice(n, n - n // 3, replace=False)).astype(np.uint32)   # a third of the columns miss
    x = rng.integers(-8, 9, len(keep)) / 8.0
    full = np.full(n, np.nan)
    full[keep] = x
    ta = lh.trie_build([rows, cols], [vals], bag=True)
    tx = lh.trie_build([keep], [x], bag=True)
    at = [(ta, [0, 1], 0), (tx, [1], 0)]
    if atoms == 3:
        at.append((lh.trie_build([keep]), [1], -1))
    p = lh.plan(2, at, out=[0], agg="sum", attr_order=[0, 1], policy="fixed")
    got = lh.join_aggregate([p])[0].to_host()
    hit = ~np.isnan(full[cols])
    want = np.unique(rows[hit])
    assert np.array_equal(got["keys"][:, 0], want)
    assert np.array_equal(got["counts"], np.bincount(rows[hit], minlength=m)[want].astype(np.uint64))
    assert np.array_equal(got["sums"], np.bincount(rows[hit], weights=vals[hit] * full[cols[hit]], minlength=m)[want])
    assert got["n_join"] == hit.sum()
    p.free()


@pytest.mark.parametrize("short_rows", [0, 20_000])
def test_groups_of_many_rows(lh, short_rows):
    """GROUP BY i over A(i,j) B(j,k): a group's frontier rows are its j."""
    rng = synth.rng_for(95)
    m, n, rows, cols, vals = matrix(rng, short_rows)
    deg = rng.integers(0, 4, n)
    deg[:len(EDGES)] = np.minimum(EDGES, 300)
    bj = np.repeat(np.arange(n), deg).astype(np.uint32)
    bk = (np.arange(len(bj)) - np.repeat(np.cumsum(deg) - deg, deg)).astype(np.uint32)
    bv = rng.integers(-8, 9, len(bj)) / 8.0
    ta = lh.trie_build([rows, cols], [vals], bag=True)
    tb = lh.trie_build([bj, bk], [bv], bag=True)
    p = lh.plan(3, [(ta, [0, 1], 0), (tb, [1, 2], 0)], out=[0], agg="sum", attr_order=[0, 1, 2], policy="fixed")
    got = lh.join_aggregate([p])[0].to_host()
    s = np.bincount(bj, weights=bv, minlength=n)
    cnt = np.bincount(rows, weights=deg[cols], minlength=m)
    want = np.nonzero(cnt)[0]
    assert np.array_equal(got["keys"][:, 0], want)
    assert np.array_equal(got["counts"], cnt[want].astype(np.uint64))
    assert np.array_equal(got["sums"], np.bincount(rows, weights=vals * s[cols], minlength=m)[want])
    p.free()
