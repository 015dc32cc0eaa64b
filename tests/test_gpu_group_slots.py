"""GROUP BY accumulators outside the order's prefix in every slot form:
padded slots of 2, 4 and 8 words (one request per tuple), nine words, slots
that carry wraps (so many tuples might meet that signed digits could leave
int64), counts only, repeated rows, and few groups (LDS).  Each must equal
the sort-based GROUP BY bit for bit: both sums are exact and rounded once,
so no tolerance applies."""
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


def relations(rng, n, groups, spread, repeat):
    """R(x, y), S(y, z): values spread over 2^spread, rows repeated; with
    repeat "long", runs that never meet but could."""
    rx, ry = rng.integers(0, 500, n // 10), rng.integers(1, 60, n // 10)
    sy, sz = rng.integers(1, 60, n), rng.integers(0, groups, n)
    if repeat == "some":
        rx, ry = np.concatenate([rx, rx[::7]]), np.concatenate([ry, ry[::7]])
        sy, sz = np.concatenate([sy, sy[::5], sy[::50]]), np.concatenate([sz, sz[::5], sz[::50]])
    elif repeat == "long":
        rx, ry = np.concatenate([rx, np.zeros(40_000, np.int64)]), np.concatenate([ry, np.full(40_000, 100)])
        sy, sz = np.concatenate([sy, np.full(40_000, 101)]), np.concatenate([sz, np.zeros(40_000, np.int64)])

    def values(m):
        v = rng.integers(1, 1 << (20 if spread else 5), m) * (1 - 2.0 * rng.integers(0, 2, m))
        return np.ldexp(v, -rng.integers(0, spread + 1, m))

    u = [a.astype(np.uint32) for a in (rx, ry, sy, sz)]
    return u[:2], values(len(rx)), u[2:], values(len(sy))


# value spreads that give from two to eight 32-bit digits with these counts
@pytest.mark.parametrize("spread", [0, 10, 30, 45, 60, 75])
@pytest.mark.parametrize("repeat", ["none", "some", "long"])
@pytest.mark.parametrize("groups", [50, 3000])
def test_slots_equal_sort(lh, spread, repeat, groups):
    rng = synth.rng_for(300 + spread)
    r, rv, s, sv = relations(rng, 6000, groups, spread, repeat)
    tr = lh.trie_build(r, [rv], bag=True)
    ts = lh.trie_build(s, [sv], bag=True)
    for agg in ("sum", "count"):
        out = {}
        for impl in ("sort", "dense", "hash"):
            p = lh.plan(3, [(tr, [0, 1], 0), (ts, [1, 2], 0)], out=[2], agg=agg, attr_order=[0, 1, 2], policy="fixed",
                        group_impl=impl)
            print(spread, repeat, groups, agg, impl, "digits", p.info()["exact_digits"], file=sys.stderr, flush=True)
            out[impl] = lh.join_aggregate([p])[0].to_host()
            p.free()
        for impl in ("dense", "hash"):
            for k in ("keys", "counts"):
                assert np.array_equal(out[impl][k], out["sort"][k])
            if agg == "sum":
                assert np.array_equal(out[impl]["sums"].view(np.uint64), out["sort"]["sums"].view(np.uint64))
            assert out[impl]["n_join"] == out["sort"]["n_join"]
    tr.free()
    ts.free()


def test_noalloc_falls_back_to_small_slots(lh):
    """A dense array that fits the static scratch only without padding runs."""
    import torch
    rng = synth.rng_for(8)
    n, space = 2000, 1_060_000
    a, b = rng.integers(0, 50, n).astype(np.uint32), rng.integers(0, space, n).astype(np.uint32)
    b[0] = space - 1
    # values of one digit pair: 36 bytes per entry before padding to 4 words
    x = np.ldexp(rng.integers(1, 1 << 20, n).astype(np.float64), -rng.integers(0, 20, n))
    tr = lh.trie_build([a], [x[:n]], bag=True)
    ts = lh.trie_build([a, b], [x], bag=True)
    p = lh.plan(2, [(ts, [0, 1], 0), (tr, [0], -1)], out=[1], agg="sum", attr_order=[0, 1], policy="fixed",
                group_impl="dense")
    print("digits", p.info()["exact_digits"], file=sys.stderr, flush=True)
    want = lh.join_aggregate([p])[0].to_host()
    cap = len(want["counts"])
    keys = [torch.zeros(cap, dtype=torch.int32, device="cuda")]
    counts = torch.zeros(cap, dtype=torch.int64, device="cuda")
    sums = torch.zeros(cap, dtype=torch.float64, device="cuda")
    assert lh.join_aggregate_noalloc(p, keys, counts, sums) == cap
    assert np.array_equal(keys[0].cpu().numpy().view(np.uint32), want["keys"][:, 0])
    assert np.array_equal(sums.cpu().numpy().view(np.uint64), want["sums"].view(np.uint64))
    assert np.array_equal(counts.cpu().numpy().view(np.uint64), want["counts"])
    p.free()
