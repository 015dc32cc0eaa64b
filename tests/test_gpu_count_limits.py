"""Tuple counts of many lanes and units that only together come near 2^64: any
count that fits 64 bits is returned, one that does not is refused.  Expected
values are products of run lengths."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RUN = 1 << 14


@pytest.fixture(scope="module")
def lh():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1708_07859_amd import lh as binding
    return binding


def counted(lh, cols, out, ys, others=3):
    """COUNT over R(cols.., y) and `others` relations of RUN equal rows for each y below ys
    (and one row for y = ys)."""
    err = lh.LHError
    r = lh.trie_build(cols, bag=True)
    y = np.concatenate([np.repeat(np.arange(ys), RUN), [ys]]).astype(np.uint32)
    u = lh.trie_build([y], bag=True)
    k = len(cols)
    p = lh.plan(k, [(r, list(range(k)), -1)] + [(u, [k - 1], -1)] * others, out=out, agg="count",
                attr_order=list(range(k)), policy="fixed")
    try:
        return lh.join_aggregate([p])[0].to_host(), err
    except err as e:
        return e, err


# 2^15 rows of R a tuple: 2^57 a key
@pytest.mark.parametrize("out", [[0], []])
@pytest.mark.parametrize("keys", [1, 9, 16, 64, 100, 127, 128, 300])
def test_keys_of_one_row(lh, out, keys):
    print(out, keys, file=sys.stderr, flush=True)
    y = np.repeat(np.arange(keys), 1 << 15).astype(np.uint32)
    got, err = counted(lh, [np.full(len(y), 5, np.uint32), y], out, keys)
    if keys << 57 < 1 << 64:
        assert got["counts"].tolist() == [keys << 57]
        assert got["n_join"] == keys << 57
    else:
        assert isinstance(got, err) and "2^64" in str(got)


# a group of many frontier rows, in front of enough others that a wave takes several of its rows
@pytest.mark.parametrize("out", [[0], []])
@pytest.mark.parametrize("rows", [40, 100, 127, 128])
def test_rows_of_one_group(lh, out, rows):
    print(out, rows, file=sys.stderr, flush=True)
    short = 300_000
    x = np.concatenate([np.zeros(rows << 15), np.arange(1, short + 1)]).astype(np.uint32)
    z = np.concatenate([np.repeat(np.arange(rows), 1 << 15), np.zeros(short)]).astype(np.uint32)
    y = np.concatenate([np.zeros(rows << 15), np.ones(short)]).astype(np.uint32)
    got, err = counted(lh, [x, z, y], out, 1)
    if (rows << 57) + (0 if out else short) < 1 << 64:
        want = [rows << 57] + [1] * short
        assert got["counts"].tolist() == (want if out else [sum(want)])
    else:
        assert isinstance(got, err) and "2^64" in str(got)
