"""GROUP BY arrays and tables near their byte limits: padding a slot to a power
of two words may not take them past those."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lh():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1708_07859_amd import lh as binding
    return binding


@pytest.mark.parametrize("space", [1000, 60_000_000, 80_000_000])
def test_dense_array(lh, space):
    """A count and two digits a slot: 24 bytes, 32 when padded; the limit is 2 GiB."""
    import torch
    print(space, file=sys.stderr, flush=True)
    n = 500
    rng = np.random.default_rng(5)
    b = np.sort(rng.choice(space, n, replace=False)).astype(np.uint32)
    b[-1] = space - 1
    v = rng.integers(1, 1 << 20, n).astype(np.float64)
    ta = lh.trie_build([np.zeros(1, np.uint32)], [np.array([1048575.0])], bag=True)
    tb = lh.trie_build([np.zeros(n, np.uint32), b], [v], bag=True)
    p = lh.plan(2, [(ta, [0], 0), (tb, [0, 1], 0)], out=[1], agg="sum", attr_order=[0, 1], policy="fixed",
                group_impl="dense")
    assert p.info()["exact_digits"] == 2
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    got = lh.join_aggregate([p])[0].to_host()
    took = free - torch.cuda.mem_get_info()[0]
    print("took", took, file=sys.stderr, flush=True)
    assert took <= (2 << 30) + (64 << 20)
    assert np.array_equal(got["keys"][:, 0], b)
    assert np.array_equal(got["sums"], v * 1048575.0)
