"""Sums over bags whose long runs of repeated key pairs lie next to each other:
the blocks' shares must not leave them to a few.  Values are multiples of
1/8, so every sum is exact in a double and numpy's must be equal."""
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


def relation(rng, rows, hot, cols, run, place):
    """`rows` rows of two columns each; the `hot` rows at place[0..hot) also hold
    `cols` columns `run` times each."""
    a = np.concatenate([np.repeat(place[:hot], cols * run), np.repeat(place, 2)])
    b = np.concatenate([np.tile(np.repeat(np.arange(cols), run), hot), rng.integers(0, 1000, 2 * rows)])
    return a.astype(np.uint32), b.astype(np.uint32), rng.integers(-80, 81, len(a)) / 8.0


def sum_plan(lh, a, b, v, x, out):
    ta = lh.trie_build([a, b], [v], bag=True)
    tx = lh.trie_build([np.arange(len(x), dtype=np.uint32)], [x], bag=True)
    return lh.plan(2, [(ta, [0, 1], 0), (tx, [1], 0)], out=out, agg="sum", attr_order=[0, 1], policy="fixed")


# (units of 32 elements: below, at and above one, two and four virtual blocks a run; past the largest grid)
@pytest.mark.parametrize("rows", [31, 65_000, 66_000, 132_000, 262_145, 1_100_000])
def test_sums_of_clustered_runs(lh, rows):
    print(rows, file=sys.stderr, flush=True)
    rng = synth.rng_for(64)
    x = rng.integers(-8, 9, 1000) / 8.0
    a, b, v = relation(rng, rows, min(rows, 400), 20, 50, np.arange(rows))
    got = lh.join_aggregate([sum_plan(lh, a, b, v, x, [0])])[0].to_host()
    assert np.array_equal(got["keys"][:, 0], np.arange(rows))
    assert np.array_equal(got["counts"], np.bincount(a).astype(np.uint64))
    assert np.array_equal(got["sums"], np.bincount(a, weights=v * x[b]))
    got = lh.join_aggregate([sum_plan(lh, a, b, v, x, [])])[0].to_host()
    assert got["counts"].tolist() == [len(a)]
    assert got["sums"].tolist() == [(v * x[b]).sum()]


@pytest.mark.parametrize("out", [[0], []])
def test_clustered_runs_are_shared_out(lh, out):
    import torch
    rng = synth.rng_for(65)
    x = synth.uniform_pm1(rng, 1000)
    took = []
    for place in (rng.permutation(2_000_000), np.arange(2_000_000)):
        p = sum_plan(lh, *relation(rng, 2_000_000, 4000, 20, 300, place), x, out)
        best = np.inf
        for _ in range(4):
            torch.cuda.synchronize()
            t = time.perf_counter()
            r = lh.join_aggregate([p])[0]
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        took.append(best)
        p.free()
    print(took, file=sys.stderr, flush=True)
    assert took[1] <= 2 * took[0], took
