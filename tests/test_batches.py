"""Lists and ranges whose primes differ widely in size: their batches on the
CPU, their residues on the GPU against a context held to the term sums."""
import os
import random
import subprocess

import numpy as np
import pytest

import paper_2101_11157_amd as wv
from paper_2101_11157_amd.workloads import next_prime

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_batches_on_host(tmp_path):
    exe = tmp_path / "test_batches"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2101_11157_amd", "csrc"), "-o", str(exe),
                    os.path.join(ROOT, "tests", "cpp", "test_batches.cpp")], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


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


# primes that, at the length of the largest beside them, meet a point that is p away from a node
SPREAD = [[76007749] + near(9 * 10 ** 10, 1), near(5 * 10 ** 10, 7) + [75510511], [75505151] + near(9 * 10 ** 10, 50)]


@pytest.mark.gpu
@pytest.mark.parametrize("step_terms", [0, 1 << 34])
def test_server_lists_of_spread_primes(ctxs, step_terms):
    """In the caller's order, with repeats, beside requests of single primes; whole and
    cut up by a budget of a few primes a step."""
    c, terms = ctxs
    rng = random.Random(3)
    lists = [list(ps) for ps in SPREAD]
    lists.append(near(113 * 10 ** 7, 2) + near(44 * 10 ** 8, 2))
    lists += [near(int(10 ** e), 2) for e in (7.9, 8.4, 9.1, 9.7, 10.6)]
    lists.append([p for ps in lists for p in ps[:3]] + [76007749, 75510511])
    for ps in lists[3:]:
        rng.shuffle(ps)
    with wv.Server(c, step_terms=step_terms) as srv:
        ids = [srv.submit_primes(ps) for ps in lists]
        got = {}
        for _ in range(10000):
            print("step", flush=True)
            srv.step()
            got.update({i: r[0] for i in ids if i not in got for r in [srv.result(i)] if r is not None})
            if len(got) == len(ids):
                break
    for ps, i in zip(lists, ids):
        print(f"case: server list of {len(ps)} primes from {min(ps)} to {max(ps)}", flush=True)
        assert np.array_equal(got[i], terms.eval_primes(ps))


@pytest.mark.gpu
@pytest.mark.parametrize("ps", SPREAD + [near(113 * 10 ** 7, 2) + near(44 * 10 ** 8, 2) + near(5 * 10 ** 10, 20),
                                         near(10 ** 6, 3) + near(9 * 2 ** 23 - 50, 8) + near(3 * 10 ** 9, 40)])
def test_lists_of_spread_primes(ctxs, ps):
    """One call for the whole list, as it stands and shuffled, with a repeat; among them
    one of a class that serves two ranges of sizes beside a longer one's primes."""
    c, terms = ctxs
    print(f"case: list of {len(ps)} primes from {min(ps)} to {max(ps)}", flush=True)
    for seed in (0, 1):
        ps = ps + ps[:1]
        assert np.array_equal(c.eval_primes(ps), terms.eval_primes(ps))
        ps = random.Random(seed).sample(ps, len(ps))
