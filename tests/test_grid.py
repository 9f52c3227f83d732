"""The grid path (fast evaluation at block starts): plan and exact arithmetic on
the CPU, residues on the GPU against the term-sum path and the oracle."""
import os
import random
import subprocess

import numpy as np
import pytest

import oracle
import paper_2101_11157_amd as wv
from paper_2101_11157_amd.workloads import is_prime, next_prime

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plan_and_arithmetic_on_host(tmp_path):
    exe = tmp_path / "test_grid"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2101_11157_amd", "csrc"), "-o", str(exe),
                    os.path.join(ROOT, "tests", "cpp", "test_grid.cpp")], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


def primes_from(lo, n):
    out, x = [], lo
    while len(out) < n:
        x = next_prime(x)
        out.append(x)
        x += 1
    return out


def primes_below(hi, n):
    out, x = [], hi - 1
    while len(out) < n:
        if is_prime(x):
            out.append(x)
        x -= 1
    return out


@pytest.fixture(scope="module")
def grid():
    with wv.Context(0) as c:
        yield c


@pytest.fixture(scope="module")
def terms():
    """A context held to the term-sum kernels (a forced block shape)."""
    with wv.Context(0) as c:
        c.set_block(28, 36)
        yield c


def rows(res):
    return [(int(r["p"]), int(r["b"]), int(r["e"]), int(r["flags"])) for r in res]


# sizes on both sides of the path's start and of its changes of length and
# congruences, and the largest primes allowed, where the transforms' integers
# are largest
SIZES = [2 ** 27, 2 ** 28 - 200, 3 * 10 ** 8, 5 * 10 ** 8, 2 ** 30, 15 * 10 ** 8, 2 ** 32, 10 ** 10, 3 * 10 ** 10,
         10 ** 11, 4 * 10 ** 11]


@pytest.mark.gpu
@pytest.mark.parametrize("lo", SIZES)
def test_grid_equals_term_sums(grid, terms, lo):
    ps = primes_from(lo - 100, 5)
    print(f"case: grid path at {ps[0]}", flush=True)
    got = grid.eval_primes(ps)
    assert rows(got) == rows(terms.eval_primes(ps))
    assert grid.stats()["n_primes"] == len(ps) and grid.stats()["n_terms"] > 0


@pytest.mark.gpu
def test_grid_largest_primes(grid, terms):
    ps = primes_below(2 ** 40, 3)
    print(f"case: grid path at {ps}", flush=True)
    assert rows(grid.eval_primes(ps)) == rows(terms.eval_primes(ps))


@pytest.mark.gpu
def test_grid_mixed_list_keeps_input_order(grid, terms):
    """Primes of every class and below the grid path's start, shuffled, with a
    repeat: results in input order, and the paper's printed near misses among
    them."""
    rng = random.Random(11)
    ps = [5, 7, 11, 16843, 2124679, 1025793739, 1025793739]
    for lo in SIZES[:9] + [10 ** 6, 10 ** 7, 10 ** 8]:
        ps += primes_from(lo, 3)
    rng.shuffle(ps)
    print(f"case: {len(ps)} primes of all sizes", flush=True)
    got = grid.eval_primes(ps)
    assert rows(got) == rows(terms.eval_primes(ps))
    i = ps.index(1025793739)
    assert wv.symmetric(got[i]["b"], ps[i]) == -9
    one = [p for p in ps if 10 ** 8 < p < 10 ** 9][0]
    want = oracle.residues([one], method="table")[0]
    assert (int(got[ps.index(one)]["b"]), int(got[ps.index(one)]["e"])) == want


@pytest.mark.gpu
@pytest.mark.parametrize("lo, width", [(2 ** 27 - 5000, 10000), (2 ** 28 - 20000, 40001), (10 ** 10, 3000),
                                       (10 ** 11 - 10 ** 6, 20000)])
def test_grid_windows(grid, terms, lo, width):
    """Windows that straddle the path's start, a change of class, and one whose
    workspace is cut into sub-batches: every prime, identical to the term
    sums (a sample of the largest window), and the same through the statistics."""
    print(f"case: window [{lo}, {lo + width})", flush=True)
    got, hits = grid.search_range(lo, lo + width)
    assert [int(p) for p in got["p"]] == oracle.primes(lo, lo + width)
    pick = got if len(got) < 300 or lo < 10 ** 9 else got[::17]
    assert rows(pick) == rows(terms.eval_primes(pick["p"]))
    hb, he, near, n = grid.range_stats(lo, lo + width, bins=7, near=0)
    assert n == len(got) and int(hb.sum()) == int(he.sum()) == n


@pytest.mark.gpu
def test_other_settings_keep_the_term_sums(terms):
    """A forced chunk, other tables or a progress callback are honoured."""
    ps = primes_from(10 ** 9, 4)
    ref = rows(terms.eval_primes(ps))
    with wv.Context(0) as c:
        c.set_chunk_terms(4096)
        assert rows(c.eval_primes(ps)) == ref and c.stats()["chunk_terms"] == 4096
        c.set_chunk_terms(0)
        c.set_tables("BB6", "EE9")
        assert rows(c.eval_primes(ps)) == ref and c.stats()["n_sums"] == 15 * len(ps)
        c.set_tables("BB30", "EE33")
        seen = []
        c.set_progress(lambda d, t: seen.append((d, t)), terms_per_launch=1 << 28)
        assert rows(c.eval_primes(ps)) == ref and seen
        c.set_progress(None)
        assert rows(c.eval_primes(ps)) == ref


def drain(srv, ids, out):
    for _ in range(100000):
        for rid in ids:
            if rid not in out:
                r = srv.result(rid)
                if r is not None:
                    out[rid] = r[0]
        if len(out) == len(ids):
            return
        srv.step()
    raise AssertionError("server did not drain")


@pytest.mark.gpu
@pytest.mark.parametrize("step_terms, fault", [(0, None), (1 << 30, None), (1 << 30, 1)])
def test_server_mixes_both_paths(grid, terms, step_terms, fault):
    """Requests of every class, below the grid path's start, across it (the term
    sums serve those) and empty, in one server, with whole-request and cut-up
    steps and a forced failure: each equals the same primes on the term sums."""
    print(f"case: server, step_terms {step_terms}, fault {fault}", flush=True)
    reqs = [primes_from(lo, 1 + k % 3) for k, lo in enumerate(SIZES[:9])]
    reqs += [(2 ** 27 - 1500, 2 ** 27 + 1500), (3 * 10 ** 9, 3 * 10 ** 9 + 900), (10 ** 6, 10 ** 6 + 2000), (24, 29),
             primes_from(10 ** 6, 4) + primes_from(10 ** 9, 2)]
    errors = 0
    with wv.Server(grid, step_terms=step_terms) as srv:
        if fault is not None:
            srv.inject_fault(fault)
        ids = []
        for i, r in enumerate(reqs):
            ids.append(srv.submit_range(*r) if isinstance(r, tuple) else srv.submit_primes(r))
            if i % 5 == 4:
                try:
                    srv.step()
                except wv.WvError:
                    errors += 1
        out = {}
        for _ in range(3):
            try:
                drain(srv, ids, out)
                break
            except wv.WvError:
                errors += 1
        st = srv.stats()
    assert errors == (0 if fault is None else 1)
    assert st["failed"] == 0 and st["completed"] == len(reqs) and st["terms_done"] > 0
    for r, rid in zip(reqs, ids):
        ps = oracle.primes(*r) if isinstance(r, tuple) else r
        assert [int(p) for p in out[rid]["p"]] == ps
        if ps:
            assert rows(out[rid]) == rows(terms.eval_primes(ps))


@pytest.mark.gpu
@pytest.mark.parametrize("lo,n", [(9 * 2 ** 23, 400), (10 ** 10, 40), (3 * 10 ** 10, 40), (10 ** 11 - 5000, 40),
                                  (5 * 10 ** 9, 5), (2 * 10 ** 10, 9), (10 ** 11 - 8000, 300), (2 ** 39 - 700, 20), (2 ** 39 + 1, 12)])
def test_ends_of_the_path_and_of_split_transforms(lo, n):
    """The first primes of the path, and batches large enough for transforms
    split into two, up to where they end."""
    print(f"case: grid, {n} primes at {lo}", flush=True)
    ps = [p for p in oracle.primes(lo, lo + 12000)][:n]
    with wv.Context(0) as grid, wv.Context(0) as sums:
        sums.set_block(28, 36)
        got = grid.eval_primes(ps)
        assert grid.stats()["chunk_terms"] in ([16383] if (lo, n) in [(10 ** 11 - 8000, 300), (2 ** 39 - 700, 20)] else [1023, 2047, 4095, 8191, 16383, 4])
        assert np.array_equal(got, sums.eval_primes(ps))
