"""Joins at the edges where the host's part changes: results sized before or
after the groups in use are counted (262,144 possible groups), few rows of
many work units and many rows of few, and a first attribute in one relation
or in two.  Values are multiples of 1/8, so every sum is exact in a double
and numpy's must be equal."""
import sys

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

CAP = 1 << 18


@pytest.fixture(scope="module")
def lh():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1708_07859_amd import lh as binding
    return binding


def check(got, group, hit, product, n):
    cnt = np.bincount(group[hit], minlength=n)
    want = np.nonzero(cnt)[0]
    assert np.array_equal(got["keys"][:, 0], want)
    assert np.array_equal(got["counts"], cnt[want].astype(np.uint64))
    assert np.array_equal(got["sums"], np.bincount(group[hit], weights=product[hit], minlength=n)[want])
    assert got["n_join"] == hit.sum()


@pytest.mark.parametrize("groups", [1, 3, CAP - 1, CAP, CAP + 1])
@pytest.mark.parametrize("by", ["prefix", "dense"])
@pytest.mark.parametrize("first", ["one", "two"])
def test_groups(lh, groups, by, first):
    """GROUP BY g over A(g, j) B(j) [C(g)]: half of the j have no partner."""
    print(groups, by, first, file=sys.stderr, flush=True)
    rng = synth.rng_for(400)
    per = 60_000 if groups <= 3 else 2
    g = np.repeat(np.arange(groups), per).astype(np.uint32)
    j = rng.integers(0, 100_000, len(g)).astype(np.uint32)
    keep = np.unique(np.stack([g, j], 1), axis=0)
    g, j = keep[:, 0].copy(), keep[:, 1].copy()
    v = rng.integers(-80, 81, len(g)) / 8.0
    bj = np.arange(0, 100_000, 2).astype(np.uint32)
    bv = rng.integers(-8, 9, len(bj)) / 8.0
    hit = j % 2 == 0
    product = v * bv[j // 2]
    order = [0, 1] if by == "prefix" else [1, 0]
    at = [(lh.trie_build([g, j] if by == "prefix" else [j, g], [v], bag=True), order, 0),
          (lh.trie_build([bj], [bv], bag=True), [1], 0)]
    if first == "two":
        cg = np.unique(np.concatenate([np.arange(0, groups, 3), [groups - 1]])).astype(np.uint32)
        at.append((lh.trie_build([cg]), [0], -1))
        hit &= np.isin(g, cg)
    kw = dict(group_impl="dense") if by == "dense" else {}
    p = lh.plan(2, at, out=[0], agg="sum", attr_order=order, policy="fixed", **kw)
    for _ in range(2):
        check(lh.join_aggregate([p])[0].to_host(), g, hit, product, groups)
    p.free()


@pytest.mark.parametrize("rows", [1, 2, 40])
@pytest.mark.parametrize("units", [16, 17, 400])
def test_units_of_long_rows(lh, rows, units):
    """Rows of the given number of wave units (and empty partners)."""
    print(rows, units, file=sys.stderr, flush=True)
    rng = synth.rng_for(401)
    n = units * 1024
    g = np.repeat(np.arange(rows), n).astype(np.uint32)
    j = np.tile(np.arange(n), rows).astype(np.uint32)
    v = rng.integers(-80, 81, len(g)) / 8.0
    bj = np.arange(0, n + 500, 1).astype(np.uint32)
    bv = rng.integers(-8, 9, len(bj)) / 8.0
    at = [(lh.trie_build([g, j], [v], bag=True), [0, 1], 0), (lh.trie_build([bj], [bv], bag=True), [1], 0)]
    p = lh.plan(2, at, out=[0], agg="sum", attr_order=[0, 1], policy="fixed")
    check(lh.join_aggregate([p])[0].to_host(), g, np.ones(len(g), bool), v * bv[j], rows)
    p.free()
