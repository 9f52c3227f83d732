"""Batches of little work in one launch: against the term sums (a context with
a forced shape) and the oracle, at the ends of its ranges, of its groups of four
terms and of the workgroups per prime."""
import numpy as np
import pytest
import torch   # before the library: it loads its own HIP runtime first

import oracle
import paper_2101_11157_amd as wv


@pytest.fixture(scope="module")
def ctxs():
    with wv.Context(0) as direct, wv.Context(0) as sums:
        sums.set_block(28, 36)
        yield direct, sums


@pytest.mark.gpu
def test_first_primes_equal_the_oracle(ctxs):
    """Every prime below 400: sums of no term, one, two and three."""
    print("case: direct, primes below 400", flush=True)
    ps = oracle.primes(5, 400)
    got = ctxs[0].eval_primes(ps)
    assert ctxs[0].stats()["chunk_terms"] == 4
    for r in got:
        p = int(r["p"])
        assert int(r["b"]) == oracle.bernoulli_all(p)[(p - 3) // 2 - 1] and int(r["e"]) == oracle.euler_all(p)[(p - 3) // 2 - 1]


# primes near which the arithmetic, the threads per prime or the path change
EDGES = [11, 1000, 65536, 10 ** 6, 1 << 21, 1 << 24, (1 << 27) - 700, 1 << 27, 10 ** 9, 6 * 10 ** 9]


@pytest.mark.gpu
@pytest.mark.parametrize("at", EDGES)
@pytest.mark.parametrize("n", [1, 2, 7, 40])
def test_short_lists_equal_the_term_sums(ctxs, at, n):
    if at * n > 1.2e10:
        pytest.skip("more work than the path takes")
    print(f"case: direct, {n} primes at {at}", flush=True)
    ps = oracle.primes(at, at + 3000)[:n]
    got = ctxs[0].eval_primes(ps)
    want = ctxs[1].eval_primes(ps)
    assert np.array_equal(got, want)
    a, b = ctxs[0].stats(), ctxs[1].stats()
    if a["chunk_terms"] == 4:
        assert (a["n_terms"], a["n_terms_b"], a["n_sums"]) == (b["n_terms"], b["n_terms_b"], b["n_sums"])


@pytest.mark.gpu
@pytest.mark.parametrize("lo,hi", [(5, 30_000), (5, 6), (8, 10), (10 ** 6, 10 ** 6 + 20_000), ((1 << 20) - 500, (1 << 20) + 500),
                                   ((1 << 27) - 2000, (1 << 27) + 2000), (10 ** 9, 10 ** 9 + 300)])
def test_windows_equal_the_term_sums(ctxs, lo, hi):
    """Searched alone (a captured sequence, run three times) and in a batch."""
    print(f"case: direct, window [{lo}, {hi})", flush=True)
    want, want_hits = ctxs[1].search_range(lo, hi)
    for _ in range(3):
        got, hits = ctxs[0].search_range(lo, hi)
        assert np.array_equal(got, want) and np.array_equal(hits, want_hits)
        ctxs[0].count_primes(5, 2000)
    both = ctxs[0].search_windows([lo, 5], [hi, 300])
    assert np.array_equal(both[0], want) and [int(p) for p in both[1]["p"]] == oracle.primes(5, 300)


@pytest.mark.gpu
def test_lists_hold_primes_only(ctxs):
    """Strong pseudoprimes to the first bases, squares and products of the
    smallest primes a trial division does not catch are refused; the bases of the
    test themselves are primes."""
    print("case: primality of list entries", flush=True)
    for n in (41 * 41, 41 * 43, 1373653, 25326001, 161304001, 960946321, 1157839381, 3215031751,
              118670087467, 307768373641, 546348519181):
        with pytest.raises(wv.WvError) as e:
            ctxs[0].eval_primes([n])
        assert e.value.status == wv.WV_ENOTPRIME, n
    got = ctxs[0].eval_primes([13, 23, 41, 43, 1662803, 1093, 3511])
    assert [int(p) for p in got["p"]] == [13, 23, 41, 43, 1662803, 1093, 3511]


@pytest.mark.gpu
@pytest.mark.parametrize("at,n", [(5, 1), (5, 40), (10 ** 5, 1), (10 ** 5, 600), (10 ** 6, 4200), (1 << 27, 3), (10 ** 9, 2),
                                  (3 * 10 ** 7, 700), (10 ** 8, 300)])
def test_device_lists_equal_the_term_sums(ctxs, at, n):
    """The call that leaves the choice to the device, on both sides of it, with
    rejected entries among the primes."""
    print(f"case: direct, device list of {n} at {at}", flush=True)
    ps = oracle.primes(at, at + 40 * n + 2000)[:n]
    ps[len(ps) // 2:len(ps) // 2] = [0, 4, 2 ** 40 + 15]
    d = torch.tensor(ps, dtype=torch.int64, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    got = []
    for c in ctxs:
        o = torch.zeros((len(ps), 4), dtype=torch.int64, device="cuda")
        for _ in range(2):
            c.eval_primes_static(d.data_ptr(), len(ps), o.data_ptr(), st)
        torch.cuda.synchronize()
        got.append(o.cpu().numpy())
    assert np.array_equal(got[0], got[1])
    assert int(np.count_nonzero(got[0][:, 0] == 0)) == 3
