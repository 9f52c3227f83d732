"""Every index of a prime by transforms: the automatic path of the all-index
calls against the power sums taken one by one and against the oracle, at the
edges of the blocks, lengths and moduli."""
import numpy as np
import pytest

import oracle
import paper_2101_11157_amd as wv


def say(s):
    print(s, flush=True)


@pytest.fixture(scope="module")
def ctx():
    with wv.Context(0) as c:
        yield c


def blocks_and_length(h):
    """The modelled choice of block length for a transform of h values."""
    best = None
    for logl in range(9, 15):
        a, L = -(-h // (1 << (logl - 1))), 1 << logl
        w = L * ((6 * a - 1) * (14 + 2.6 * logl) + 2 * a * a * 16)
        if best is None or w < best[0]:
            best = (w, a, logl)
    return best[1:]


def edges():
    """Primes on both sides of every change of (blocks, length) up to 2^17, and
    of the change of moduli at 2^16."""
    ps = oracle.primes(5, 1 << 17)
    out = {5, 7, 11, 13, 65521, 65537}
    for a, b in zip(ps, ps[1:]):
        if blocks_and_length((a - 1) // 2) != blocks_and_length((b - 1) // 2):
            out |= {a, b}
    return sorted(out)


def test_edges_reach_every_length():
    seen = [blocks_and_length((p - 1) // 2) for p in edges()]
    assert {l for _, l in seen} == set(range(9, 15)) and max(a for a, _ in seen) >= 3


@pytest.mark.gpu
@pytest.mark.parametrize("part", range(4))
def test_transforms_equal_power_sums(ctx, part):
    for p in edges()[part::4]:
        say(f"case: every index by transforms, p = {p}")
        b, e = ctx.bernoulli_euler_all(p)
        ctx.set_irregular_path(1)
        try:
            wb, we = ctx.bernoulli_euler_all(p)
        finally:
            ctx.set_irregular_path(0)
        assert np.array_equal(b, wb) and np.array_equal(e, we), p
        if p < 700:
            assert [int(x) for x in b] == oracle.bernoulli_all(p) and [int(x) for x in e] == oracle.euler_all(p)


@pytest.mark.gpu
@pytest.mark.parametrize("lo,hi", [(5, 13), (5, 1500), (1000, 1030), (1500, 5600), (65000, 66200), (130900, 131300)])
def test_census_by_transforms(ctx, lo, hi):
    """Several lengths and both numbers of moduli within one window, joined into
    the larger ones; windows too small for transforms."""
    say(f"case: census by transforms, [{lo}, {hi})")
    got = ctx.irregular_pairs(lo, hi)
    ctx.set_irregular_path(1)
    try:
        want = ctx.irregular_pairs(lo, hi)
    finally:
        ctx.set_irregular_path(0)
    assert np.array_equal(got[0], want[0]) and got[1:] == want[1:]
