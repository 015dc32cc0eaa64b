"""Batched products with few outputs far apart: the packing must find them
past any number of rows without one, and not by walking over those."""
import sys
import time

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


def batch(lh, rng, n, rows):
    """Two matrix-vector plans over n rows of one entry each, whose vectors
    meet the given rows."""
    col = rng.permutation(n).astype(np.uint32)
    v = synth.uniform_pm1(rng, n)
    ta = lh.trie_build([np.arange(n, dtype=np.uint32), col], [v], bag=True)
    tx = [lh.trie_build([np.sort(col[r])], [np.full(len(r), 0.5)], bag=True) for r in rows]
    plans = [lh.plan(2, [(ta, [0, 1], 0), (t, [1], 0)], out=[0], agg="sum", attr_order=[0, 1], policy="fixed")
             for t in tx]
    return plans, v, (ta, tx)


GAPS = [1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 319, 320, 321, 5000, 64, 1, 20_000]


@pytest.mark.parametrize("first", [0, 1, 255, 4096])
@pytest.mark.parametrize("last", [0, 1, 64, 300])
def test_outputs_far_apart(lh, first, last, tmp_path, monkeypatch):
    monkeypatch.setenv("LH_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
    print(first, last, file=sys.stderr, flush=True)
    rng = synth.rng_for(62)
    a = first + np.concatenate([[0], np.cumsum(GAPS + GAPS[::-1])])
    n = int(a[-1]) + 1 + last
    b = np.unique(np.concatenate([a, np.arange(n // 2, n // 2 + 200), rng.integers(0, n, 3000)]))
    plans, v, keep = batch(lh, rng, n, [a, b])
    for r, g in zip([a, b], lh.join_aggregate(plans)):
        g = g.to_host()
        assert np.array_equal(g["keys"][:, 0], r)
        assert np.array_equal(g["sums"], 0.5 * v[r])


def test_sparse_outputs_cost_no_more_than_dense(lh, tmp_path, monkeypatch):
    monkeypatch.setenv("LH_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
    import torch
    rng = synth.rng_for(63)
    n = 2_000_000
    some = np.sort(rng.choice(n, 60, replace=False))
    took = []
    for rows in ([np.arange(n), np.arange(n)], [some, some]):
        plans, _, keep = batch(lh, rng, n, rows)
        best = np.inf
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            out = lh.join_aggregate(plans)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        took.append(best)
    assert took[1] <= 2 * took[0], took
