"""The two-set COUNT leaf's probes of sorted sets at the edges of their forms:
one to five driver keys a lane, probed ranges that are staged whole, searched
through staged samples or through samples in memory, lines cut by a range's
ends, values at both ends of the key range, and bitsets that are probed as
bitsets or, sparse and hardly larger than the driver, by their sorted keys.
Counts must equal numpy's."""
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


DRIVER = [1, 2, 63, 64, 65, 128, 129, 192, 193, 255, 256, 257, 300, 513]
PROBED = [1, 3, 8, 9, 31, 32, 33, 64, 500, 1023, 1024, 1025, 2600, 9000, 40_000]


@pytest.mark.parametrize("space", [60_000, 1 << 32])
@pytest.mark.parametrize("grouped", [False, True])
@pytest.mark.parametrize("layout", ["uint", "plain", "bitset"])
def test_probes(lh, space, grouped, layout):
    print(space, grouped, layout, file=sys.stderr, flush=True)
    rng = synth.rng_for(500)
    a, b, want = [], [], []
    for d in DRIVER:
        for m in PROBED:
            x = np.unique(rng.integers(0, space, d, dtype=np.uint64))
            y = np.unique(rng.integers(0, space, m, dtype=np.uint64))
            take = rng.choice(x, (len(x) + 1) // 2, replace=False)
            y = np.unique(np.concatenate([y, take, [0, space - 1] if (d + m) % 3 else []]).astype(np.uint64))
            x = np.unique(np.concatenate([x, [0] if d % 2 else [space - 1]]).astype(np.uint64))
            a.append(x)
            b.append(y)
            want.append(len(np.intersect1d(x, y)))
    # one large balanced pair: the top bucket, in units of 512 keys
    for d, m in [(9000, 9000), (9000, 17_500), (12_000, 90_000)]:
        x = np.unique(rng.integers(0, 1 << 32, d, dtype=np.uint64))
        y = np.unique(np.concatenate([rng.integers(0, 1 << 32, m, dtype=np.uint64), x[::3]]))
        a.append(x)
        b.append(y)
        want.append(len(np.intersect1d(x, y)))
    want = np.array(want, np.uint64)

    def trie(sets):
        i = np.repeat(np.arange(len(sets)), [len(v) for v in sets]).astype(np.uint32)
        return lh.trie_build([i, np.concatenate(sets).astype(np.uint32)], layout=layout)

    ta, tb = trie(a), trie(b)
    for first, second in ((ta, tb), (tb, ta)):
        p = lh.plan(2, [(first, [0, 1], -1), (second, [0, 1], -1)], out=[0] if grouped else [], agg="count",
                    attr_order=[0, 1], policy="fixed")
        got = lh.join_aggregate([p])[0].to_host()
        if grouped:
            use = np.nonzero(want)[0]
            assert np.array_equal(got["keys"][:, 0], use)
            assert np.array_equal(got["counts"], want[use])
        else:
            assert got["counts"][0] == want.sum()
        p.free()
