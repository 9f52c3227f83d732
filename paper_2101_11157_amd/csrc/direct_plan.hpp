// direct_plan.hpp -- which batches go the direct way and in what launches: plain
// host code, unit-tested without a GPU.
#pragma once
#include <algorithm>
#include <cstdint>

#include "mont.hpp"

namespace wv {

// The direct path (wv_direct.hip): batches of little work, contexts as for the
// grid path.  Measured on MI355X, ms a call, term sums (or grid path) / direct:
//   n primes below 2^27, by their terms in all: 4e6 x 4096 (1.4e9 terms) 0.95 /
//   0.80, 1e7 x 1024 (0.9e9) 0.70 / 0.46, x 4096 (3.6e9) 1.43 / 1.76, 2e7 x 1024
//   (1.8e9) 0.86 / 0.80, 4e7 x 256 (0.9e9) 0.66 / 0.53, 8e7 x 256 (1.8e9) 0.88 /
//   0.96, one prime at 1e8 0.53 / 0.08;
//   every batch of small primes, whose (prime, sum) records cost more than the
//   terms: 1e6 x 20000 1.97 / 1.01, 4e6 x 20000 2.83 / 2.83;
//   from 2^27 on, where a product is six operations: 1.4e8 x 64 (0.8e9) 0.58 / 0.53,
//   3e8 x 16 (0.4e9) 0.40 / 0.31, x 64 (1.7e9) 0.52 / 0.91, one prime at 3e9 (0.26e9)
//   0.39 / 0.22, at 1e10 (0.9e9) 0.50 / 0.54.
constexpr int kDirectWaves = 4;     // of a workgroup, at most
constexpr uint64_t kDirectSmallP = 1ull << 27;   // products exact in double precision below
constexpr uint64_t kDirectAllP = 3ull << 20;
constexpr double kDirectSmallTerms = 1.6e9, kDirectTerms = 5e8;
// Lanes the primes of a batch share, and the least terms for one: 2^20 are 16
// waves for each SIMD, rounds enough to even out the ends (2e7 x 1024: 0.80 ms,
// with 2^19 0.98 ms).
constexpr double kDirectLanes = 1048576.0, kDirectLaneTerms = 48.0;
// Every prime of a batch gets as many lanes, so the largest of a list of mixed
// sizes ends last: terms a lane at most, n primes like the largest at kDirectLanes.
// A lane takes 40 ns a term, 80 where the sums are short: 500 primes near 1e5 and
// one near 4e9 (171,000 a lane) 6.5 ms, by term sums 0.58.
constexpr double kDirectLaneMost = 2048.0;
struct DirectShape {
    bool small;              // p < kDirectSmallP
    uint32_t G, threads;     // workgroups per prime and their threads
    uint64_t key() const { return (uint64_t)G << 32 | threads << 1 | (small ? 1 : 0); }
};
constexpr uint64_t kDirectParts = 1 << 14;   // fractions held where only the device knows the primes

// Whether a batch of n primes <= pmax, sum in all, whose congruences hold cost p
// terms a prime, goes this way; the host's rule and the device's.
__host__ __device__ inline bool direct_rule(double n, uint64_t pmax, double sum, double cost) {
    return pmax <= kDirectAllP || (sum * cost <= (pmax <= kDirectSmallP ? kDirectSmallTerms : kDirectTerms) &&
                                   (double)pmax * cost * n <= kDirectLaneMost * kDirectLanes);
}

// Lanes of each prime: the chip's, and kDirectLaneTerms (about twelve groups of
// four) for each at least.
__host__ __device__ inline double direct_lanes(double n, uint64_t pmax, double cost) {
    const double share = kDirectLanes / n, own = (double)pmax * cost / kDirectLaneTerms;
    return share < own ? share : own;
}

inline bool direct_shape(uint64_t n, uint64_t pmax, double sum, double cost, DirectShape *d) {
    if (n == 0) return false;
    d->small = pmax <= kDirectSmallP;
    if (!direct_rule((double)n, pmax, sum, cost)) return false;
    const double lanes = direct_lanes((double)n, pmax, cost);
    uint32_t w = 64;
    while (2.0 * w <= lanes && w < 64 * kDirectWaves) w *= 2;
    uint32_t G = 1;
    while (2.0 * G * w <= lanes && G < 1024) G *= 2;
    d->threads = w;
    d->G = G;
    return true;
}

// Primes per launch at most: a launch holds fewer than 2^32 threads, and a
// list (of small primes, with repeats) may be longer.
inline uint32_t direct_launch_primes(const DirectShape &d) { return (1u << 31) / (d.G * d.threads); }

// Slots of a captured search of at most n_bound primes: every one has its
// workgroups, G of them, whether it holds a prime or not, and 2^18 that hold none
// take 0.25 ms.  Up to 1024 a power of two (few captures), then a multiple of 1024:
// windows of 2 integers near 1e9, 1024 slots / these, 0.34 / 0.09 ms (term sums
// 0.32), of 20 near 8e7 0.16 / 0.08.
inline uint64_t direct_pad(uint64_t n_bound) {
    uint64_t n = 16;
    while (n < n_bound && n < 1024) n *= 2;
    return n < n_bound ? (n_bound + 1023) & ~1023ull : n;
}

}  // namespace wv
