"""Little work and lists of mixed sizes: the rules on the CPU, lists on the GPU
against a context held to the term sums."""
import os
import subprocess

import numpy as np
import pytest
import torch   # before the library: it loads its own HIP runtime first

import oracle
import paper_2101_11157_amd as wv
from paper_2101_11157_amd.workloads import next_prime

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("name", ["test_direct_plan", "test_list_plan"])
def test_rules_on_host(tmp_path, name):
    exe = tmp_path / name
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2101_11157_amd", "csrc"), "-o", str(exe),
                    os.path.join(ROOT, "tests", "cpp", name + ".cpp")], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.gpu
def test_list_longer_than_a_launch():
    """More small primes, with repeats, than one launch holds threads for."""
    few = np.array(oracle.primes(5, 300), dtype=np.uint64)
    n = (1 << 26) + 77
    print(f"case: direct, list of {n} entries", flush=True)
    with wv.Context(0) as c, wv.Context(0) as terms:
        terms.set_block(28, 36)
        want = terms.eval_primes(few)
        got = c.eval_primes(np.resize(few, n))
        assert c.stats()["n_primes"] == n and c.stats()["chunk_terms"] == 4
    whole = n // len(few) * len(few)
    assert bool((got[:whole].reshape(-1, len(few)) == want).all())
    assert np.array_equal(got[whole:], want[:n - whole])


def near(lo, n):
    out, x = [], lo
    while len(out) < n:
        x = next_prime(x)
        out.append(x)
        x += 1
    return out


# the paths a list takes by chunk_terms of its last part: a grid block, 4 (direct), or a chunk of term sums
MIXED = [("grid, little work below it", near(10 ** 4, 100) + near(2 * 10 ** 10, 2), 4),
         ("grid, term sums below it", near(5 * 10 ** 7, 3000) + near(10 ** 9, 30), None),
         ("direct, of sizes 1e5 to 2e9", near(10 ** 5, 5) + near(10 ** 7, 3) + near(2 * 10 ** 9, 1), 4),
         ("term sums: a chain each would be longer", near(15 * 10 ** 7, 60) + near(7 * 10 ** 9, 1), None)]


@pytest.mark.gpu
@pytest.mark.parametrize("what, ps, chunk", MIXED, ids=[m[0] for m in MIXED])
def test_lists_of_mixed_sizes(what, ps, chunk):
    print(f"case: {what}", flush=True)
    ps = ps[1::2] + ps[::2]
    with wv.Context(0) as c, wv.Context(0) as terms:
        terms.set_block(28, 36)
        got = c.eval_primes(ps)
        s = c.stats()
        assert s["n_primes"] == len(ps) and (s["chunk_terms"] == chunk if chunk else s["n_chunks"] > 0)
        assert np.array_equal(got, terms.eval_primes(ps))


# a list in device memory: one large prime among many small ones would leave its few lanes
# with most of the work, so such lists stay with the term sums
@pytest.mark.gpu
@pytest.mark.parametrize("n, lo, m, hi", [(500, 10 ** 5, 1, 4 * 10 ** 9), (5000, 10 ** 4, 1, 10 ** 9), (8, 10 ** 5, 1, 2 * 10 ** 9),
                                          (1, 7, 1, 5 * 10 ** 9), (300, 10 ** 6, 2, 5 * 10 ** 7), (99, 10 ** 4, 1, 2 * 10 ** 8)])
def test_device_lists_of_mixed_sizes(n, lo, m, hi):
    print(f"case: device list, {n} primes at {lo} and {m} at {hi}", flush=True)
    ps = near(lo, n) + near(hi, m)
    ps = ps[1::2] + ps[::2]
    d = torch.tensor(ps, dtype=torch.int64, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    got, ms = [], []
    with wv.Context(0) as c, wv.Context(0) as terms:
        terms.set_block(28, 36)
        for x in (c, terms):
            o = torch.zeros((n + m, 4), dtype=torch.int64, device="cuda")
            t = []
            for _ in range(5):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                x.eval_primes_static(d.data_ptr(), n + m, o.data_ptr(), st)
                b.record()
                torch.cuda.synchronize()
                t.append(a.elapsed_time(b))
            got.append(o.cpu().numpy())
            ms.append(min(t))
    assert np.array_equal(got[0], got[1])
    # (0.1 to 0.6 ms by term sums; 6.5 and 25 ms when the first two went direct)
    assert ms[0] < 2.0 * ms[1]


# windows that form several parts, that go as one batch, and that overlap, in any order
WINDOWS = [[(10 ** 6, 400), (3 * 10 ** 7, 400), (8 * 10 ** 7, 400), (2 * 10 ** 8, 400), (10 ** 9, 400), (9 * 10 ** 9, 200)],
           [(9 * 2 ** 23 - 300, 300), (9 * 2 ** 23, 300), (9 * 2 ** 23 - 100, 200)],
           [(2 * 10 ** 9, 3000), (2 * 10 ** 9 + 1, 2999), (2 * 10 ** 9 + 1000, 50), (5, 100), (2 * 10 ** 9 - 64, 9000)],
           [(10 ** 8 + 7 * 10 ** 6 * k, 1500) for k in range(12)] + [(10 ** 10, 30), (2 * 10 ** 7, 3000)],
           [(24, 5), (10 ** 10, 40), (90, 7), (4 * 10 ** 9, 700), (113 * 10 ** 7, 700)]]


@pytest.mark.gpu
@pytest.mark.parametrize("k", range(len(WINDOWS)))
def test_windows_of_mixed_sizes(k):
    """Each window of a call, whatever parts its primes run in, is what the term sums give."""
    los = [lo for lo, _ in WINDOWS[k]]
    his = [lo + w for lo, w in WINDOWS[k]]
    print(f"case: windows {WINDOWS[k]}", flush=True)
    with wv.Context(0) as c, wv.Context(0) as terms:
        terms.set_block(28, 36)
        want = terms.search_windows(los, his)
        for order in (list(range(len(los))), list(range(len(los)))[::-1], list(range(1, len(los), 2)) + list(range(0, len(los), 2))):
            got = c.search_windows([los[i] for i in order], [his[i] for i in order])
            for i, g in zip(order, got):
                assert [int(p) for p in g["p"]] == oracle.primes(los[i], his[i])
                assert np.array_equal(g, want[i])
        lo, hi = min(los), max(his)
        if hi - lo < 10 ** 5:
            assert c.range_stats(lo, hi, bins=10, near=0)[3] == len(oracle.primes(lo, hi))


@pytest.mark.gpu
@pytest.mark.parametrize("lo, width", [(9 * 2 ** 23 + 1, 1), (3 * 10 ** 8, 2), (10 ** 9 + 6, 2), (10 ** 9, 20), (10 ** 8, 33),
                                       (10 ** 9 + 1, 64), (10 ** 7, 300), (10 ** 6, 7000), (10 ** 6, 9000)])
def test_narrow_windows(lo, width):
    """One window with as many slots as it may hold primes, or 16: three captured
    replays each, between other calls."""
    print(f"case: direct, window [{lo}, {lo + width})", flush=True)
    with wv.Context(0) as c, wv.Context(0) as terms:
        terms.set_block(28, 36)
        for a in (lo, lo + 12, lo + 2):
            got, _ = c.search_range(a, a + width)
            ps = oracle.primes(a, a + width)
            assert [int(p) for p in got["p"]] == ps
            if ps:
                assert c.stats()["chunk_terms"] == 4 and c.stats()["n_primes"] == len(ps)
                assert np.array_equal(got, terms.eval_primes(ps))
            c.count_primes(5, 3000)
