"""Calls on a device whose memory others hold: the workspaces of the grid path and
of the transforms of every index are cut to what is left, and the results stay
what they are with memory to spare."""
import numpy as np
import pytest
import torch   # before the library: it loads its own HIP runtime first

import paper_2101_11157_amd as wv
from paper_2101_11157_amd.workloads import next_prime

GIB = 1 << 30


def hold_all_but(left):
    """Tensors that leave about `left` bytes of the device free."""
    held = []
    while True:
        free, _ = torch.cuda.mem_get_info()
        if free - left < GIB // 8:
            return held
        held.append(torch.empty(min(free - left, 64 * GIB), dtype=torch.uint8, device="cuda"))


@pytest.mark.gpu
def test_calls_with_little_memory_left():
    p = next_prime(16_000_000)
    lo, hi = 10 ** 11 - 10 ** 6, 10 ** 11 - 10 ** 6 + 8192
    with wv.Context(0) as c:
        print("case: memory to spare", flush=True)
        window, _ = c.search_range(lo, hi)
        pairs = c.irregular_pairs(10 ** 6, 10 ** 6 + 1500)
        every = c.bernoulli_euler_all(p)
    with wv.Context(0) as c:
        c.search_range(5, 10 ** 5)   # the runtime's own buffers
        c.eval_primes([10 ** 9 + 7])
        c.irregular_pairs(30_000, 30_500)
        held = hold_all_but(4 * GIB)
        try:
            print("case: 4 GiB left, a window whose primes' workspace is 7 GiB", flush=True)
            got, _ = c.search_range(lo, hi)
            assert np.array_equal(got, window)
            assert c.stats()["chunk_terms"] == 16383   # the grid path's longest blocks all the same
        finally:
            del held
            torch.cuda.empty_cache()
    with wv.Context(0) as c:
        c.irregular_pairs(30_000, 30_500)
        held = hold_all_but(4 * GIB)
        try:
            print("case: 4 GiB left, a census window of 8 GiB groups", flush=True)
            got = c.irregular_pairs(10 ** 6, 10 ** 6 + 1500)
            assert np.array_equal(got[0], pairs[0]) and got[1:] == pairs[1:]
        finally:
            del held
            torch.cuda.empty_cache()
    with wv.Context(0) as c:
        c.irregular_pairs(30_000, 30_500)
        c.set_irregular_path(2)
        c.irregular_pairs(30_000, 30_500)
        c.set_irregular_path(0)
        held = hold_all_but(2 * GIB)
        try:
            print("case: 2 GiB left, a prime whose transforms need more", flush=True)
            got = c.bernoulli_euler_all(p)
            assert np.array_equal(got[0], every[0]) and np.array_equal(got[1], every[1])
        finally:
            del held
            torch.cuda.empty_cache()
