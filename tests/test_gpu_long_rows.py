"""Frontier rows far longer than their level's average: hub keys with many
children below a level of short sets.  Their cut into units may not cost what
a cut by the average would: memory, the number of units, or time."""
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


def hubs(lh, n_hubs, long, short):
    """S(y, z): n_hubs keys y of `long` children 0..long, and `short` keys of one."""
    import torch
    y = torch.cat([torch.arange(n_hubs).repeat_interleave(long), n_hubs + torch.arange(short)])
    z = torch.cat([torch.arange(long).repeat(n_hubs), torch.zeros(short, dtype=torch.int64)])
    t = lh.trie_build([y.to(torch.int32).cuda(), z.to(torch.int32).cuda()])
    n = t.info()["level_size"]
    assert n[1] <= 24 * n[0]
    return t


@pytest.mark.parametrize("long", [254, 255, 256, 257, 300, 5000])
@pytest.mark.parametrize("leaf", [False, True])
def test_rows_longer_than_a_wave(lh, long, leaf):
    """As a middle attribute (the frontier is filled) and as the last."""
    print(long, leaf, file=sys.stderr, flush=True)
    rng = synth.rng_for(66)
    ts = hubs(lh, 7, long, 7 * long)
    x, y = np.arange(40, dtype=np.uint32), rng.integers(0, 7, 40).astype(np.uint32)
    keep = np.sort(rng.choice(long, long - long // 3, replace=False)).astype(np.uint32)
    tr, tk = lh.trie_build([x, y], bag=leaf), lh.trie_build([keep])
    atoms = [(tr, [0, 1], -1), (ts, [1, 2], -1), (tk, [2], -1)]
    p = lh.plan(3, atoms, out=[0] if leaf else [0, 1, 2], agg="count", attr_order=[0, 1, 2], policy="fixed")
    got = lh.join_aggregate([p])[0].to_host()
    if leaf:
        assert np.array_equal(got["keys"][:, 0], x)
        assert (got["counts"] == len(keep)).all()
    else:
        want = np.stack([np.repeat(x, len(keep)), np.repeat(y, len(keep)), np.tile(keep, 40)], 1)
        assert np.array_equal(got["keys"], want)
        assert (got["counts"] == 1).all()


def test_units_of_long_rows_fit_the_static_scratch(lh):
    """100 rows of six million keys: their units by the level's average alone would fill the scratch."""
    import torch
    ts = hubs(lh, 1, 6_000_000, 300_000)
    tr = lh.trie_build([np.arange(100, dtype=np.uint32), np.zeros(100, np.uint32)])
    p = lh.plan(3, [(tr, [0, 1], -1), (ts, [1, 2], -1)], out=[0], agg="count", attr_order=[0, 1, 2], policy="fixed")
    keys = [torch.zeros(100, dtype=torch.int32, device="cuda")]
    counts = torch.zeros(100, dtype=torch.int64, device="cuda")
    assert lh.join_aggregate_noalloc(p, keys, counts) == 100
    assert keys[0].cpu().tolist() == list(range(100))
    assert (counts == 6_000_000).all()


def test_more_short_units_than_32_bits(lh):
    """1.5e11 driver elements are fewer than 2^32 units of a wave's 256."""
    n, long = 100_000, 1_500_000
    ts = hubs(lh, 1, long, 100_000)
    tr = lh.trie_build([np.arange(n, dtype=np.uint32), np.zeros(n, np.uint32)])
    p = lh.plan(3, [(tr, [0, 1], -1), (ts, [1, 2], -1)], out=[0], agg="count", attr_order=[0, 1, 2], policy="fixed")
    got = lh.join_aggregate([p])[0].to_host()
    assert np.array_equal(got["keys"][:, 0], np.arange(n))
    assert (got["counts"] == long).all()
