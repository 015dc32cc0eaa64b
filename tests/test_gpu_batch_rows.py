"""Batched instances with rows at the edges of the batch's row classes
(eight-lane vector rows, block rows, light, heavy and inner-product matrix
rows), thousands of rows without output between them (the packing walks
over those) and hub rows, on the first call (launched as it is) and on the
next ones (replayed as a graph).  Every instance must equal its own plan run
alone, bit for bit: both sums are exact."""
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


EDGES = [1, 2, 7, 8, 9, 15, 16, 17, 63, 64, 65, 127, 128, 129, 2047, 2048, 2049, 4000]


def matrix(rng, n, empty):
    """EDGES rows at random places among rows of one entry; `empty` of those
    point at columns at or above n (no row of B there)."""
    deg = np.concatenate([EDGES, np.ones(n - len(EDGES), np.int64)])
    deg = deg[rng.permutation(n)]
    rows = np.repeat(np.arange(n), deg)
    cols = np.concatenate([rng.choice(n, d, replace=False) for d in deg])
    one = np.flatnonzero(np.repeat(deg == 1, deg))
    lost = rng.choice(one, empty, replace=False)
    cols[lost] += n
    v = rng.integers(-80, 81, len(rows)) / 8.0
    v[rng.integers(0, len(v), 100)] = synth.uniform_pm1(rng, 100)
    return rows.astype(np.uint32), cols.astype(np.uint32), v


@pytest.mark.parametrize("kinds", ["spmv", "spgemm", "both"])
def test_rows_of_every_class(lh, kinds, tmp_path, monkeypatch):
    monkeypatch.setenv("LH_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
    rng = synth.rng_for(60)
    keep, plans = [], []
    for n, empty in ((5000, 0), (5000, 4500), (9001, 3000), (4097, 1)):
        print(kinds, n, empty, file=sys.stderr, flush=True)
        r, c, v = matrix(rng, n, empty)
        ta = lh.trie_build([r, c], [v], bag=True)
        keep.append(ta)
        if kinds != "spgemm":
            tx = lh.trie_build([np.arange(n, dtype=np.uint32)], [synth.uniform_pm1(rng, n)], bag=True)
            keep.append(tx)
            plans.append(lh.plan(2, [(ta, [0, 1], 0), (tx, [1], 0)], out=[0], agg="sum"))
        if kinds != "spmv":
            plans.append(lh.plan(3, [(ta, [0, 1], 0), (ta, [1, 2], 0)], out=[0, 2], agg="sum", attr_order=[0, 1, 2],
                                 policy="fixed"))
    want = [lh.join_aggregate([p])[0].to_host() for p in plans]
    for call in range(3):
        got = [x.to_host() for x in lh.join_aggregate(plans)]
        for g, w in zip(got, want):
            assert np.array_equal(g["keys"], w["keys"])
            assert np.array_equal(g["counts"], w["counts"])
            assert np.array_equal(g["sums"].view(np.uint64), w["sums"].view(np.uint64))
            assert g["n_join"] == w["n_join"]
    # a tuned signature: the first call of other plans launches without a graph
    again = lh.join_aggregate(plans[1:] + plans[:1])
    g = again[-1].to_host()
    assert np.array_equal(g["sums"].view(np.uint64), want[0]["sums"].view(np.uint64))
