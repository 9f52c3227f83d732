"""Every index of one prime: sizes that one index a lane and eight serve, and those of
the longer transforms, against the power sums and the term sums."""
import numpy as np
import pytest

import paper_2101_11157_amd as wv
from paper_2101_11157_amd.workloads import next_prime

# without queued indices (5003, 6007) and with, on both sides of 2^19, and above 2^24
SIZES = [5, 7, 11, 131, 5003, 6007, 300007, (1 << 19) - 1, next_prime(1 << 19), 1000003, 4000037, next_prime(1 << 24)]


@pytest.mark.gpu
@pytest.mark.parametrize("p", SIZES)
def test_every_index(p):
    print(f"case: every index of {p}", flush=True)
    with wv.Context(0) as c, wv.Context(0) as terms:
        terms.set_block(28, 36)
        b, e = c.bernoulli_euler_all(p)
        assert len(b) == len(e) == (p - 3) // 2 and c.stats()["n_primes"] == 1
        r = terms.eval_primes([p])[0]
        assert (int(b[-1]), int(e[-1])) == (int(r["b"]), int(r["e"]))   # B_{p-3}, E_{p-3}
        assert int(e.max()) < p and int(b[b != np.uint64(2 ** 64 - 1)].max()) < p
        if p < 1 << 22:
            c.set_irregular_path(2)
            sums = c.bernoulli_euler_all(p)
            assert np.array_equal(b, sums[0]) and np.array_equal(e, sums[1])
