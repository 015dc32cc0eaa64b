"""Joins from several host threads at once, each on a stream of its own, and
from many short-lived threads: what a thread reads back is its own, in every
form of query.  Every result is compared with the same query run alone."""
import sys
import threading

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


def queries(lh, seed):
    """Builds, plans and runs one of each kind; its results, as plain values."""
    rng = synth.rng_for(seed)
    n = 2000 + 100 * (seed % 7)
    i, j = (rng.integers(0, 300, n).astype(np.uint32) for _ in range(2))
    v, x = rng.integers(-80, 81, n) / 8.0, rng.integers(-8, 9, 300) / 8.0
    ta, te = lh.trie_build([i, j], [v], bag=True), lh.trie_build([i, j])
    tx = lh.trie_build([np.arange(300, dtype=np.uint32)], [x], bag=True)
    plans = [lh.plan(2, [(ta, [0, 1], 0), (tx, [1], 0)], out=[0], agg="sum"),
             lh.plan(3, [(ta, [0, 1], 0), (ta, [1, 2], 0)], out=[0, 2], agg="sum"),
             lh.plan(3, [(te, [0, 1], -1), (te, [1, 2], -1), (te, [0, 2], -1)], agg="count"),
             lh.plan(3, [(te, [0, 1], -1), (te, [1, 2], -1)], out=[0, 1, 2], agg="count"),
             lh.plan(2, [(ta, [0, 1], 0), (tx, [1], 0)], out=[], agg="sum")]
    got = []
    for p in plans:
        o = lh.join_aggregate([p])[0].to_host()
        got.append((o["keys"].tobytes(), o["counts"].tobytes(), None if o["sums"] is None else o["sums"].tobytes(),
                    o["n_join"]))
    return got


def in_threads(work, n):
    wrong = []

    def guard(k):
        try:
            work(k)
        except BaseException as e:  # noqa: BLE001 (shown by the assertion below)
            wrong.append((k, repr(e)))

    threads = [threading.Thread(target=guard, args=(k,)) for k in range(n)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong


@pytest.mark.parametrize("own_stream", [True, False])
def test_concurrent_joins(lh, own_stream):
    import torch
    print("own streams", own_stream, file=sys.stderr, flush=True)
    seeds = list(range(200, 206))
    want = {s: queries(lh, s) for s in seeds}

    def work(k):
        stream = torch.cuda.Stream() if own_stream else torch.cuda.current_stream()
        with torch.cuda.stream(stream):
            for r in range(12):
                s = seeds[(k + r) % len(seeds)]
                assert queries(lh, s) == want[s], (k, r, s)

    in_threads(work, 6)


def test_short_lived_threads(lh):
    want = queries(lh, 300)
    for r in range(20):
        in_threads(lambda k: (queries(lh, 300) == want) or pytest.fail("another result"), 3)


def test_ended_threads_leave_nothing(lh):
    """Host memory mapped for a thread's words is there for the next thread."""
    import torch
    key = torch.arange(100, device="cuda", dtype=torch.int32)

    def mapped():
        with open("/proc/self/maps") as f:
            return len(f.readlines())

    for r in range(10):
        in_threads(lambda k: lh.trie_build([key]).free(), 2)
    before = mapped()
    for r in range(200):
        in_threads(lambda k: lh.trie_build([key]).free(), 2)
    assert mapped() < before + 100
