"""Calls that reach each path and each of its lengths, with the path asserted: by
chunk_terms, the terms per block of the grid path (one less than a power of two),
4 for the direct path, and a chunk of many terms for the term sums."""
import numpy as np
import pytest

import oracle
import paper_2101_11157_amd as wv
from paper_2101_11157_amd.workloads import next_prime

START = 9 * 2 ** 23   # the grid path's


def near(lo, n):
    out, x = [], lo
    while len(out) < n:
        x = next_prime(x)
        out.append(x)
        x += 1
    return out


@pytest.fixture(scope="module")
def ctxs():
    with wv.Context(0) as c, wv.Context(0) as terms:
        terms.set_block(28, 36)
        yield c, terms


@pytest.mark.gpu
@pytest.mark.parametrize("lo, n, k", [
    # more primes than take a shorter length than their own class
    (START, 400, 1023), (2 ** 27 - 1000, 300, 1023), (2 ** 28 - 9000, 300, 1023), (3 * 10 ** 8, 300, 2047),
    (5 * 10 ** 8, 300, 2047), (2 ** 30 + 10 ** 6, 300, 2047), (15 * 10 ** 8, 300, 4095), (2 ** 32 + 10 ** 9, 300, 8191),
    (10 ** 10, 300, 8191), (10 ** 11 - 10 ** 6, 300, 16383), (2 ** 39 - 20000, 300, 16383), (2 ** 39 + 1, 280, 8191),
    # few primes, but more than little work
    (2 ** 27, 100, 1023), (2 ** 30, 12, 2047)])
def test_lists_reach_every_length(ctxs, lo, n, k):
    c, terms = ctxs
    ps = near(lo, n)
    print(f"case: grid, {n} primes at {lo}", flush=True)
    got = c.eval_primes(ps)
    s = c.stats()
    assert s["chunk_terms"] == k and s["n_primes"] == n
    pick = slice(None) if lo < 2 ** 33 else slice(None, None, 12)
    assert np.array_equal(got[pick], terms.eval_primes(ps[pick]))


@pytest.mark.gpu
@pytest.mark.parametrize("lo, hi, k", [
    # a segment of 2^20 that starts below goes to the term sums whole, the next one to the grid path
    (START - 30000, START + 30000, None), (START - 30000, START + 2 ** 20, 1023), (START, START + 20000, 1023),
    (START - 20000, START, None), (2 * 10 ** 8 - 50, 2 * 10 ** 8 + 30000, 1023),
    # across the first change of length
    (28032 * 10 ** 4 - 40000, 28032 * 10 ** 4 + 40000, 2047)])
def test_windows_on_both_sides_of_the_start(ctxs, lo, hi, k):
    """Searched, in a batch of windows, and through the statistics."""
    c, terms = ctxs
    print(f"case: window [{lo}, {hi})", flush=True)
    got, _ = c.search_range(lo, hi)
    last = c.stats()["chunk_terms"]
    assert last == k if k else c.stats()["n_chunks"] > 0
    want, _ = terms.search_range(lo, hi)
    assert np.array_equal(got, want) and len(got) == len(oracle.primes(lo, hi))
    both = c.search_windows([hi, lo], [hi + 20000, hi])
    assert np.array_equal(both[1], want) and np.array_equal(both[0], terms.search_range(hi, hi + 20000)[0])
    a, b = c.range_stats(lo, hi, bins=64, near=2000), terms.range_stats(lo, hi, bins=64, near=2000)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2]) and a[3] == b[3]


@pytest.mark.gpu
def test_server_ranges_on_both_sides_of_the_start(ctxs):
    c, terms = ctxs
    reqs = [(START - 3000, START + 3000), (START, START + 4000), (START - 4000, START), (28032 * 10 ** 4 - 3000, 28032 * 10 ** 4 + 3000)]
    print(f"case: server, ranges {reqs}", flush=True)
    with wv.Server(c) as srv:
        ids = [srv.submit_range(*r) for r in reqs]
        got = {}
        for _ in range(1000):
            srv.step()
            got.update({i: r[0] for i in ids if i not in got for r in [srv.result(i)] if r is not None})
            if len(got) == len(ids):
                break
    for r, i in zip(reqs, ids):
        assert np.array_equal(got[i], terms.search_range(*r)[0])
