"""The sieve's primes at the edges of its scheme: words, segments, the primes
whose multiples come as patterns, and ranges around the sizes at which a prime
is strided by a wave or by a lane."""
import random

import pytest

import oracle
import paper_2101_11157_amd as wv


@pytest.fixture(scope="module")
def ctx():
    with wv.Context(0) as c:
        yield c


def windows(kind):
    rng = random.Random(kind)
    if kind == "first":      # the patterns' own primes, single integers, words
        return [(5, 6), (5, 7), (6, 7), (7, 32), (29, 38), (31, 33), (33, 37), (5, 64), (5, 65), (5, 66), (63, 130),
                (5, 1024), (1000, 3000), (5, 48 * 37 * 2), (5, 48 * 37 * 2 + 4), (961, 962), (1369, 1370)]
    if kind == "segments":   # around multiples of 2^20
        out = []
        for s in (1 << 20, 1 << 21, 7 << 20, 95367 << 20):
            out += [(s - 1, s + 1), (s, s + 1), (s, s + 2), (s - 3, s + 64), (s - 65, s + 1), (s - 70000, s + 70000)]
        return out
    if kind == "ranges":     # 48 multiples of the primes near 37, 1000, 8000
        return [(lo, lo + 2 * 48 * q + d) for q in (37, 41, 997, 1009) for lo in (10 ** 6 + 1, 10 ** 11 - 10 ** 7)
                for d in (-2, -1, 0, 1, 2)]
    return [(lo, lo + rng.randrange(1, 300_000)) for lo in (rng.randrange(5, 10 ** rng.randrange(2, 12)) for _ in range(12))]


def squares():
    """Windows that begin, end or hold just the square of a prime."""
    return [(q * q + a, q * q + b) for q in (37, 101, 1021, 8191, 316223) for a, b in ((0, 1), (-1, 1), (0, 300), (-300, 0))]


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["first", "segments", "ranges", "random", "squares"])
def test_windows_hold_the_primes(ctx, kind):
    for lo, hi in squares() if kind == "squares" else windows(kind):
        print(f"case: sieve [{lo}, {hi})", flush=True)
        want = [p for p in oracle.primes(lo, hi) if p >= 5]
        assert ctx.count_primes(lo, hi) == len(want), (lo, hi)
        if hi - lo <= 200:
            assert [int(p) for p in ctx.search_range(lo, hi)[0]["p"]] == want, (lo, hi)


@pytest.mark.gpu
@pytest.mark.parametrize("lo,hi", [(5, 70_000), (999_000, 1_030_000), ((1 << 20) - 9000, (1 << 20) + 9001)])
def test_compaction_is_ascending_and_complete(ctx, lo, hi):
    print(f"case: compaction [{lo}, {hi})", flush=True)
    assert [int(p) for p in ctx.search_range(lo, hi)[0]["p"]] == oracle.primes(lo, hi)
