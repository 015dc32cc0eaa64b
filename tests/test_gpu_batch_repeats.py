"""Batched products of bags that repeat key pairs: a row's products are pairs
of rows, whatever number of distinct keys they fall on.  Every instance must
equal its own plan run alone: join tuples, counts and (exact) sums."""
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


def repeated(rng, n, degree, most):
    """n rows of `degree` distinct columns, hub rows of many, each pair there 1..most times."""
    deg = np.full(n, degree)
    deg[rng.integers(0, n, 3)] = [min(n, 40), min(n, 300), n]
    rows = np.repeat(np.arange(n), deg)
    cols = np.concatenate([rng.choice(n, d, replace=False) for d in deg])
    times = rng.integers(1, most + 1, len(rows))
    rows, cols = np.repeat(rows, times), np.repeat(cols, times)
    return rows.astype(np.uint32), cols.astype(np.uint32), synth.uniform_pm1(rng, len(rows))


@pytest.mark.parametrize("most", [(1, 4), (4, 1), (3, 60)])
def test_repeated_pairs(lh, most, tmp_path, monkeypatch):
    monkeypatch.setenv("LH_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
    rng = synth.rng_for(61)
    keep, plans = [], []
    for n, degree in ((50, 2), (400, 3), (700, 20)):
        print(most, n, degree, file=sys.stderr, flush=True)
        ta, te = (lh.trie_build(list(m[:2]), [m[2]], bag=True) for m in (repeated(rng, n, degree, k) for k in most))
        xk = np.repeat(np.arange(n), rng.integers(1, most[1] + 1, n)).astype(np.uint32)
        tx = lh.trie_build([xk], [synth.uniform_pm1(rng, len(xk))], bag=True)
        keep += [ta, te, tx]
        for agg in ("sum", "count"):
            plans.append(lh.plan(3, [(ta, [0, 1], 0), (te, [1, 2], 0)], out=[0, 2], agg=agg, attr_order=[0, 1, 2],
                                 policy="fixed"))
        plans.append(lh.plan(2, [(ta, [0, 1], 0), (tx, [1], 0)], out=[0], agg="sum", attr_order=[0, 1],
                             policy="fixed"))
    want = [lh.join_aggregate([p])[0].to_host() for p in plans]
    for call in range(2):
        for g, w in zip([x.to_host() for x in lh.join_aggregate(plans)], want):
            assert np.array_equal(g["keys"], w["keys"])
            assert np.array_equal(g["counts"], w["counts"])
            if w["sums"] is not None:
                assert np.array_equal(g["sums"].view(np.uint64), w["sums"].view(np.uint64))
            assert g["n_join"] == w["n_join"] == w["counts"].sum()
