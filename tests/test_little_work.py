"""Little work: the direct path's rule on the CPU, its longest lists on the GPU."""
import os
import subprocess

import numpy as np
import pytest

import oracle
import paper_2101_11157_amd as wv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rule_on_host(tmp_path):
    exe = tmp_path / "test_direct_plan"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2101_11157_amd", "csrc"), "-o", str(exe),
                    os.path.join(ROOT, "tests", "cpp", "test_direct_plan.cpp")], check=True)
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
