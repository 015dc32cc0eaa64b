"""Results whose buffers were sized before their rows were counted: kept ones
may not hold device memory for groups that turned out empty."""
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


@pytest.mark.parametrize("agg", ["sum", "count"])
@pytest.mark.parametrize("where", ["prefix", "dense"])
@pytest.mark.parametrize("used", [0, 1, 700, 49_999, 50_000, 200_000])
def test_rows_of_many_possible_groups(lh, where, agg, used):
    """200,000 possible groups (an attribute of the order's prefix, or outside it), `used` with a tuple."""
    import torch
    print(where, agg, used, file=sys.stderr, flush=True)
    rng = synth.rng_for(67)
    n = 200_000
    i, j = np.arange(n, dtype=np.uint32), rng.permutation(n).astype(np.uint32)
    v = synth.uniform_pm1(rng, n)
    hit = np.sort(rng.choice(n, used, replace=False)) if used < n else np.arange(n)
    on = np.sort(j[hit]) if used else np.array([n + 5], np.uint32)
    tx = lh.trie_build([on], [np.full(len(on), 0.5)], bag=True)
    if where == "prefix":
        ta = lh.trie_build([i, j], [v], bag=True)
        p = lh.plan(2, [(ta, [0, 1], 0), (tx, [1], 0)], out=[0], agg=agg, attr_order=[0, 1], policy="fixed")
    else:
        ta = lh.trie_build([j, i], [v], bag=True)
        p = lh.plan(2, [(ta, [1, 0], 0), (tx, [1], 0)], out=[0], agg=agg, attr_order=[1, 0], policy="fixed",
                    group_impl="dense")
    lh.join_aggregate([p])
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    kept = [lh.join_aggregate([p])[0] for _ in range(40)]
    held = free - torch.cuda.mem_get_info()[0]
    row = 4 + 8 + (8 if agg == "sum" else 0)
    print("held", held, file=sys.stderr, flush=True)
    # (what the rows take four times over, and 1 MiB a result and 32 MiB in all for roundings)
    assert held <= 40 * (4 * used * row + (1 << 20)) + (32 << 20)
    for r in (kept[0], kept[-1]):
        got = r.to_host()
        assert np.array_equal(got["keys"][:, 0], hit) if used else len(got["keys"]) == 0
        assert (got["counts"] == 1).all()
        if agg == "sum":
            assert np.array_equal(got["sums"], 0.5 * v[hit])
        assert got["n_join"] == used
