"""Calls that a user of this framework makes, with the sizes they are made with.

Each case is one call (or, for the request server, one run of requests) through
the public Python entry points: ranges searched from the first primes to the
ceiling of the paper's search at 1e11, single primes and short lists, batches
of uneven windows, residue statistics, prime counts, the request server, the
device-pointer call of callers that must not allocate, and the irregular-pair
census.  Every output is a whole number.

Contexts are kept for the life of the process, as a program that searches
keeps its own; inputs are made from the seed alone.
"""
import math
import random

import numpy as np
import torch

import paper_2101_11157_amd as wv
from paper_2101_11157_amd.workloads import next_prime

# Terms of the printed congruences (eqnBB30 + eqnEE33: 0.0878 p per prime) that
# one drawn case may hold: below the largest listed one.
TERM_COST = 0.0878
MAX_TERMS = 2.5e12


def listed():
    return [
        # every prime below 1e5: the smallest search, where launches count
        {"name": "search_small", "kind": "search", "tables": "printed", "lo": 5, "width": 100_000},
        # a window of the paper's middle range, tens of thousands of primes
        {"name": "search_1e9", "kind": "search", "tables": "printed", "lo": 10 ** 9, "width": 400_003},
        # one sub-window at the ceiling of the paper's search, default context
        {"name": "search_1e11", "kind": "search", "tables": "printed", "lo": 10 ** 11 - 10 ** 6, "width": 8192},
        # the same with the shipped ladders of derived congruences
        {"name": "search_1e11_derived", "kind": "search", "tables": "derived", "lo": 10 ** 11 - 10 ** 6, "width": 8192},
        # one large prime: the latency of a single query
        {"name": "eval_single", "kind": "eval", "lo": 5 * 10 ** 10, "hi": 6 * 10 ** 10, "n": 1},
        # uneven windows over the whole range in one batched call
        {"name": "windows", "kind": "windows", "n": 12, "len_lo": 1000, "len_hi": 10_000, "lo": 10 ** 6,
         "hi": 10 ** 11},
        # mixed requests through the server: 70 % single primes, 30 % intervals
        {"name": "serve", "kind": "serve", "n": 24, "lo": 10 ** 8, "hi": 5 * 10 ** 10, "len_lo": 100,
         "len_hi": 10_000},
        # a list of mid-size primes in device memory, no allocation in the call
        {"name": "static_list", "kind": "static", "lo": 10 ** 6, "hi": 10 ** 8, "n": 1000},
        # histograms and near misses of a range, no per-prime results
        {"name": "stats_1e8", "kind": "stats", "lo": 10 ** 8, "width": 1_000_000, "bins": 2000, "near": 50},
        # the irregular-pair census, one window of the benchmark's size
        {"name": "census", "kind": "census", "lo": 1 << 15, "width": 4096},
        # every B_{2k}, E_{2k} of one prime
        {"name": "all_index", "kind": "all_index", "lo": 100_000, "hi": 300_000},
        # prime count of a wide range at the ceiling
        {"name": "count_1e11", "kind": "count", "lo": 10 ** 11 - 10 ** 9, "width": 10 ** 9},
    ]


def _log_int(rng, a, b):
    return int(math.exp(rng.uniform(math.log(a), math.log(b))))


def _width(rng, lo, a, b):
    """A width in [a, b] whose primes near lo hold at most MAX_TERMS terms."""
    w = _log_int(rng, a, b)
    per = max(1.0, lo) * TERM_COST / math.log(max(lo, 10))
    return max(1, min(w, int(MAX_TERMS / per)))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "eval", "windows", "serve", "static", "stats", "census",
                       "all_index", "count"])
    if kind == "search":
        lo = _log_int(rng, 5, 10 ** 11)
        return {"kind": kind, "tables": "printed", "lo": lo, "width": _width(rng, lo, 1000, 10 ** 6)}
    if kind == "eval":
        lo = _log_int(rng, 10 ** 4, 9 * 10 ** 10)
        return {"kind": kind, "lo": lo, "hi": lo + lo // 5 + 100, "n": _log_int(rng, 1, 100)}
    if kind == "windows":
        a = _log_int(rng, 10 ** 3, 10 ** 4)
        return {"kind": kind, "n": rng.randint(2, 12), "len_lo": a, "len_hi": a + rng.randint(1, a), "lo": 10 ** 6,
                "hi": _log_int(rng, 10 ** 8, 10 ** 11)}
    if kind == "serve":
        return {"kind": kind, "n": rng.randint(4, 24), "lo": 10 ** 7, "hi": _log_int(rng, 10 ** 8, 5 * 10 ** 10),
                "len_lo": 100, "len_hi": rng.randint(200, 10_000)}
    if kind == "static":
        lo = _log_int(rng, 10 ** 3, 10 ** 9)
        return {"kind": kind, "lo": lo, "hi": 2 * lo, "n": min(8000, _log_int(rng, 1, 2 * 10 ** 11 // lo))}
    if kind == "stats":
        lo = _log_int(rng, 10 ** 4, 10 ** 10)
        return {"kind": kind, "lo": lo, "width": _width(rng, lo, 1000, 10 ** 6), "bins": rng.randint(1, 4000),
                "near": rng.randint(0, 1000)}
    if kind == "census":
        lo = _log_int(rng, 5, 1 << 17)
        return {"kind": kind, "lo": lo, "width": rng.randint(100, 8192)}
    if kind == "all_index":
        lo = _log_int(rng, 10 ** 3, 10 ** 6)
        return {"kind": kind, "lo": lo, "hi": lo + lo // 5}
    lo = _log_int(rng, 5, 10 ** 11)
    return {"kind": "count", "lo": lo, "width": _log_int(rng, 10 ** 3, 10 ** 9)}


_contexts = {}


def _context(which):
    """The process's context with the printed tables (the default), the shipped
    ladders ("derived") or for the server."""
    if which not in _contexts:
        c = wv.Context(0)
        if which == "derived":
            c.use_derived_tables()
        _contexts[which] = c
    return _contexts[which]


_server = []


def _the_server():
    if not _server:
        _server.append(wv.Server(_context("server")))
    return _server[0]


def _primes(rng, lo, hi, n):
    return [next_prime(rng.randrange(lo, hi)) for _ in range(n)]


def _table(width, words):
    """Room for the results of the primes of `width` integers (a fixed share of
    the odd ones where there are many)."""
    return np.zeros((width // 2 + 8 if width < 1000 else width // 4 + 300, words), dtype=np.int64)


def prepare(case, seed):
    rng = random.Random(f"{case['kind']} {seed}")
    kind = case["kind"]
    s = {"kind": kind}
    if kind in ("search", "stats", "census", "count"):
        # another seed, another window: a shifted start, or, from the first
        # primes on, another end
        shift = rng.randrange(1, 2 + max(1, case["width"] // 4))
        lo = case["lo"] if case["lo"] == 5 else case["lo"] + shift
        hi = case["lo"] + case["width"] + shift
        if case["lo"] > 10 ** 11 - 10 ** 10:   # stay below the ceiling
            lo, hi = case["lo"] - shift, case["lo"] + case["width"] - shift
        s.update(lo=lo, hi=hi)
    if kind == "search":
        s.update(ctx=_context(case["tables"]), table=_table(case["width"], 4), hits=np.zeros((64, 1), dtype=np.int64))
    elif kind == "eval":
        s.update(ctx=_context("printed"),
                 primes=np.array(_primes(rng, case["lo"], case["hi"], case["n"]), dtype=np.uint64))
    elif kind == "windows":
        los, his = [], []
        for i in range(case["n"]):
            # positions spread over the range (one per equal step of its logarithm)
            a, b = math.log(case["lo"]), math.log(case["hi"])
            u = a + (b - a) * (i + rng.random()) / case["n"]
            lo = min(int(math.exp(u)), case["hi"] - case["len_hi"])
            los.append(lo)
            his.append(lo + _log_int(rng, case["len_lo"], case["len_hi"]))
        order = list(range(case["n"]))
        rng.shuffle(order)
        s.update(ctx=_context("printed"), los=[los[i] for i in order], his=[his[i] for i in order],
                 table=_table(case["n"] * case["len_hi"], 4))
    elif kind == "serve":
        reqs = []
        for i in range(case["n"]):
            u = rng.randrange(case["lo"], case["hi"])
            if i % 10 < 7:
                reqs.append(np.array([next_prime(u)], dtype=np.uint64))
            else:
                reqs.append((u, u + _log_int(rng, case["len_lo"], case["len_hi"])))
        s.update(server=_the_server(), requests=reqs, table=_table(case["n"] * case["len_hi"], 4))
    elif kind == "static":
        ps = np.array(_primes(rng, case["lo"], case["hi"], case["n"]), dtype=np.int64)
        s.update(ctx=_context("printed"), n=case["n"], d_primes=torch.from_numpy(ps).cuda(),
                 d_out=torch.zeros((case["n"], 4), dtype=torch.int64, device="cuda"))
    elif kind == "stats":
        # near misses of both sides: a few per prime at most
        s.update(ctx=_context("printed"), bins=case["bins"], near=case["near"], table=_table(2 * case["width"], 3))
    elif kind == "census":
        s.update(ctx=_context("printed"), table=_table(4 * case["width"], 2))
    elif kind == "all_index":
        s.update(ctx=_context("printed"), p=_primes(rng, case["lo"], case["hi"], 1)[0],
                 table=np.zeros((case["hi"] + 1000, 1), dtype=np.int64))
    elif kind == "count":
        s.update(ctx=_context("printed"))
    return s


def _rows(a, words):
    """A record array as rows of 64-bit words (no copy)."""
    return a.view(np.int64).reshape(-1, words)


def _collect(buf, parts, words):
    """The caller's own table of results: the parts one after another in a table
    of fixed size, and how many rows each has."""
    at, counts = 0, []
    for a in parts:
        r = _rows(a, words)
        buf[at:at + len(r)] = r
        at += len(r)
        counts.append(len(r))
    return {"rows": buf, "counts": np.array(counts, dtype=np.int64)}


def run(s):
    kind = s["kind"]
    if kind == "search":
        res, hits = s["ctx"].search_range(s["lo"], s["hi"])
        return [_collect(s["table"], [res], 4), _collect(s["hits"], [hits], 1)]
    if kind == "eval":
        return _rows(s["ctx"].eval_primes(s["primes"]), 4)
    if kind == "windows":
        return _collect(s["table"], s["ctx"].search_windows(s["los"], s["his"]), 4)
    if kind == "serve":
        srv = s["server"]
        ids = [srv.submit_range(*r) if isinstance(r, tuple) else srv.submit_primes(r) for r in s["requests"]]
        out = [None] * len(ids)
        while any(o is None for o in out):
            srv.step()
            for i, rid in enumerate(ids):
                if out[i] is None:
                    r = srv.result(rid)
                    if r is not None:
                        out[i] = r[0]
        return _collect(s["table"], out, 4)
    if kind == "static":
        s["ctx"].eval_primes_static(s["d_primes"].data_ptr(), s["n"], s["d_out"].data_ptr(),
                                    torch.cuda.current_stream().cuda_stream)
        return s["d_out"]
    if kind == "stats":
        hb, he, near, n = s["ctx"].range_stats(s["lo"], s["hi"], bins=s["bins"], near=s["near"])
        return [hb.view(np.int64), he.view(np.int64), _collect(s["table"], [near], 3), n]
    if kind == "census":
        pairs, n_primes, unresolved = s["ctx"].irregular_pairs(s["lo"], s["hi"])
        return [_collect(s["table"], [pairs], 2), n_primes, unresolved]
    if kind == "all_index":
        b, e = s["ctx"].bernoulli_euler_all(s["p"])
        return [_collect(s["table"], [b, e], 1)]
    return s["ctx"].count_primes(s["lo"], s["hi"])


def work(case):
    """What a pass cannot do without.  Two residues of one prime p take at least
    about sqrt(p) log2(p) products mod p by the fastest method known for one
    prime (products over arithmetic progressions by fast evaluation), six
    operations each; every index of one prime about p log2(p) (one convolution
    of that length); a prime count one operation per odd integer.  Bytes: the
    results, 32 per prime (16 per index; one bit per odd integer counted)."""
    kind = case["kind"]

    def one(p):
        p = max(p, 10.0)
        return 6.0 * math.sqrt(p) * math.log2(p)

    def count(lo, width):
        mid = max(lo + width / 2, 10.0)
        return max(1.0, width / math.log(mid))

    if kind in ("search", "stats"):
        n = count(case["lo"], case["width"])
        return {"bytes": 32 * n, "flops": n * one(case["lo"] + case["width"] / 2)}
    if kind in ("eval", "static"):
        return {"bytes": 32 * case["n"], "flops": case["n"] * one((case["lo"] + case["hi"]) / 2)}
    if kind in ("windows", "serve"):
        mean_len = (case["len_hi"] - case["len_lo"]) / max(1e-9, math.log(case["len_hi"] / case["len_lo"]))
        share = 1.0 if kind == "windows" else 0.3
        n = flops = 0.0
        for i in range(case["n"]):
            f = (i + 0.5) / case["n"]
            p = (math.exp(math.log(case["lo"]) * (1 - f) + math.log(case["hi"]) * f) if kind == "windows" else
                 case["lo"] * (1 - f) + case["hi"] * f)
            k = share * count(p, mean_len) + (1 - share)
            n += k
            flops += k * one(p)
        return {"bytes": 32 * n, "flops": flops}
    if kind == "census":
        p = max(case["lo"] + case["width"] / 2, 10.0)
        n = count(case["lo"], case["width"])
        return {"bytes": 32 * n, "flops": n * 6.0 * p * math.log2(p)}
    if kind == "all_index":
        p = (case["lo"] + case["hi"]) / 2
        return {"bytes": 8 * p, "flops": 6.0 * p * math.log2(p)}
    return {"bytes": case["width"] / 16, "flops": case["width"] / 2}


def _plain_primes(lo, hi):
    lo = max(lo, 5)
    if hi <= lo:
        return []
    keep = np.ones(hi - lo, dtype=bool)
    for q in range(2, math.isqrt(hi) + 1):
        keep[max(q * q, -(-lo // q) * q) - lo::q] = False
    return [lo + int(i) for i in np.flatnonzero(keep)]


def _plain_residues(p):
    """B_{p-3} and E_{p-3} mod p from H_{p-1} == -(p^2 / 3) B_{p-3} (mod p^3) and
    -4 E_{p-3} == sum_{0 < s < p/4} s^-2 (mod p)."""
    m = p ** 3
    h = sum(pow(k, -1, m) for k in range(1, p)) % m
    b = -3 * (h // (p * p)) % p
    e = -pow(4, -1, p) * sum(pow(s, -2, p) for s in range(1, p // 4 + 1)) % p
    return b, e


def exact(case, seed):
    """Whole numbers from their definitions, where the primes are small and few
    enough; every output is an integer, so nothing else is needed elsewhere."""
    kind = case["kind"]
    if kind == "count" and case["width"] <= 10 ** 6 and case["lo"] + case["width"] <= 10 ** 9:
        s = prepare(case, seed)
        return len(_plain_primes(s["lo"], s["hi"]))
    if kind == "search" and case["lo"] + case["width"] <= 6000:
        s = prepare(case, seed)
        rows, hits = [], []
        for p in _plain_primes(s["lo"], s["hi"]):
            b, e = _plain_residues(p)
            rows.append((p, b, e, (b == 0) | 2 * (e == 0)))
            if b == 0 or e == 0:
                hits.append(p)
        table, found = _table(case["width"], 4), np.zeros((64, 1), dtype=np.int64)
        table[:len(rows)] = np.array(rows, dtype=np.int64).reshape(-1, 4)
        found[:len(hits), 0] = hits
        return [{"rows": table, "counts": np.array([len(rows)])}, {"rows": found, "counts": np.array([len(hits)])}]
    return None
