// wv_grid.hip -- both residues of a batch of primes by fast evaluation along
// arithmetic progressions.
//
// Each sum of a congruence (Sections 3 and 5) is cut into blocks of K
// consecutive s.  With F(x) = prod_{j<K} (x + j) and its Taylor coefficients
// g_0 .. g_3 (F(x + h) = sum g_k h^k), a block that starts at x enters the
// sum's pair as P = g_0^d, Q as in sum_core.hpp.  Instead of stepping the g_k
// from block to block, their values at all block starts x = lo + K t are taken
// from their values at K + 1 fixed nodes by Lagrange's formula,
//   g(X) = prod_i (X - Y_i) sum_i u_i / (X - Y_i),
//   u_i = g(Y_i) / prod_{m != i} (Y_i - Y_m),
// whose nodes and points both advance by K, so that the sum over i is a
// convolution of u with 1 / (lo + K n), done exactly by number-theoretic
// transforms (ntt.hpp).  The factor prod (X - Y_i) is common to g_0 .. g_3 at
// one point and drops out of c1 / c0.  A sum of len terms costs about
// len / K^2 transforms of length 2 K instead of len steps: for a prime p about
// sqrt(p) log p operations per transform-sized share instead of p.
//
// Nodes Y_i = -K (K + 1 - i), i = 0 .. K: below every point, so every
// difference X - Y_i is a positive integer below p (p >= 4 (2 K + 2)^2).
//
// Node values (products of K consecutive integers with derivatives) are built
// by doubling: blocks of k = 255 directly, then from k to 2 k + 1 as
//   P_{2k+1}(Y) = P_k(Y) P_k(Y + k) (Y + 2 k),
// where the nodes already known give P_k at Y_t + k and at the next k + 1
// nodes by the same convolutions (here with the factor prod (X - Y_i)).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "grid_plan.hpp"
#include "ntt.hpp"
#include "wave_ops.hpp"
#include "wv_ctx.hpp"

namespace wv {
namespace {

constexpr int kBaseK = 255;   // blocks whose node values are multiplied out

// ---------------------------------------------------------------------------
// plan: shifts per sum
// ---------------------------------------------------------------------------

// One thread per (prime, run), laid out as the sums are (s^-3 runs of prime i at
// i rB + r, then the s^-2 ones): its first term and length, and the shifts of
// W block starts it needs; the terms of each side added to terms[0] (all) and
// terms[1] (s^-3 side).
__global__ void __launch_bounds__(256) k_grid_runs(const SegRec *__restrict__ segs, uint32_t n, int nB, int nE,
                                                   const GridRuns *__restrict__ tabs, int tb, int te, uint64_t K,
                                                   int logw, SegRec *__restrict__ runs, uint64_t *__restrict__ cnt,
                                                   unsigned long long *__restrict__ terms) {
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    const uint32_t rB = tabs[tb].n, rE = tabs[te].n;
    uint64_t len = 0, len_b = 0;
    if (i < (uint64_t)n * (rB + rE)) {
        const bool bern = i < (uint64_t)n * rB;
        const uint64_t k = bern ? i : i - (uint64_t)n * rB;
        const uint32_t prime = (uint32_t)(k / (bern ? rB : rE)), r = (uint32_t)(k % (bern ? rB : rE));
        const GridRuns &g = tabs[bern ? tb : te];
        const uint64_t base = bern ? (uint64_t)prime * nB : (uint64_t)n * nB + (uint64_t)prime * nE;
        SegRec s = segs[base + g.first[r]];
        const SegRec e = segs[base + g.last[r]];
        s.len = e.lo + e.len - s.lo;   // 0 for a rejected prime (every sum empty)
        runs[i] = s;
        cnt[i] = (s.len / K + (1ull << logw) - 1) >> logw;
        len = s.len;
        len_b = bern ? s.len : 0;
    }
    for (int o = 32; o >= 1; o >>= 1) {
        len += shfl_xor_u64(len, o);
        len_b += shfl_xor_u64(len_b, o);
    }
    if ((threadIdx.x & 63) == 0 && len) {
        atomicAdd(&terms[0], (unsigned long long)len);
        if (len_b) atomicAdd(&terms[1], (unsigned long long)len_b);
    }
}

// ---------------------------------------------------------------------------
// inverses along a progression
// ---------------------------------------------------------------------------

// inv[e] = 1 / (lo + K n) mod p for n = 0 .. (R + 1) W - 1 of every run with R
// shifts, at (off[slot] + slot) W + n.  A wave takes 64 C consecutive entries
// of one run, each lane C of them: products up, one Fermat inverse, products
// down.
template <int C>
__global__ void __launch_bounds__(256) k_grid_inv(const SegRec *__restrict__ segs, const uint64_t *__restrict__ off,
                                                  uint32_t nseg, const PrimeRec *__restrict__ pr, uint64_t K, int logw,
                                                  double *__restrict__ inv) {
    const int lane = threadIdx.x & 63;
    const uint64_t units = ((off[nseg] + nseg) << logw) / (64 * C);
    const uint64_t nwaves = (uint64_t)gridDim.x * 4;
    for (uint64_t u0 = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6); u0 < units; u0 += nwaves) {
        const uint64_t u = readfirst_u64(u0);
        const uint64_t e0 = u * (64 * C), g = e0 >> logw;
        uint32_t lo = 0, hi = nseg;   // the slot whose entries hold granule g
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (off[mid] + mid <= g) lo = mid;
            else hi = mid;
        }
        if (off[lo + 1] == off[lo]) continue;   // no shift: entries never read
        const SegRec s = segs[lo];
        const uint64_t p = pr[s.prime].p;
        const Fmod f = fmod_of(p);
        const uint64_t n0 = e0 - ((off[lo] + lo) << logw);
        const double a0 = (double)(s.lo + K * (n0 + lane)), step = (double)(64 * K);
        double pre[C];
        double acc = 1.0;
WV_UNROLL
        for (int c = 0; c < C; c++) {
            pre[c] = acc;
            acc = f_mulmod(acc, fma((double)c, step, a0), f);   // the entry, an integer below p
        }
        double r = f_pow_u(acc, p - 2, f);
WV_UNROLL
        for (int c = C - 1; c >= 0; c--) {
            inv[e0 + (uint64_t)c * 64 + lane] = f_mulmod(r, pre[c], f);
            r = f_mulmod(r, fma((double)c, step, a0), f);
        }
    }
}

// Prefix products A_i of get(0 .. 256 C - 1) over a workgroup of 256 threads,
// and their inverses: thread t holds entries [t C, t C + C).  prev: A before
// its first entry.
template <int C, class Get>
__device__ __forceinline__ void prefix_inverses(const Fmod &f, uint64_t p, double *__restrict__ s, Get get,
                                                double (&A)[C], double (&iA)[C], double &prev) {
    const int tid = threadIdx.x;
    double v[C];
WV_UNROLL
    for (int i = 0; i < C; i++) {
        v[i] = get(tid * C + i);
        A[i] = i ? f_mulmod(A[i ? i - 1 : 0], v[i], f) : v[0];
    }
    s[tid] = A[C - 1];
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const double u = tid >= o ? s[tid - o] : 1.0;
        __syncthreads();
        s[tid] = f_mulmod(s[tid], u, f);
        __syncthreads();
    }
    prev = tid ? s[tid - 1] : 1.0;
    double r = f_pow_u(s[tid], p - 2, f);   // inverse of the prefix up to this thread's last entry
    __syncthreads();                        // s is free
WV_UNROLL
    for (int i = 0; i < C; i++) A[i] = f_mulmod(A[i], prev, f);
WV_UNROLL
    for (int i = C - 1; i >= 0; i--) {
        iA[i] = r;
        r = f_mulmod(r, v[i], f);
    }
}

// A thread's C consecutive entries of an array of 256 C through LDS (one pad
// per 16), so that memory sees whole lines: stored entry by entry they took
// most of the time of the kernels below.
__host__ __device__ constexpr int stage_at(int i) { return i + (i >> 4); }
template <int C>
struct Stage {
    double v[stage_at(256 * C)];
};

template <int C, int N>
__device__ __forceinline__ void stage_store(Stage<C> &s, double *__restrict__ out) {
    __syncthreads();
WV_UNROLL
    for (int i = 0; i < (N + 255) / 256; i++) {
        const int at = i * 256 + (int)threadIdx.x;
        if (at < N) out[at] = s.v[stage_at(at)];
    }
    __syncthreads();
}

// Factorials and their inverses mod p up to K = 256 C - 1 (a workgroup per
// prime): fact[i], fact[(K + 1) + i].
template <int C>
__global__ void __launch_bounds__(256) k_grid_fact(const PrimeRec *__restrict__ pr, double *__restrict__ fact) {
    __shared__ Stage<C> s;
    const int tid = threadIdx.x;
    const uint64_t p = pr[blockIdx.x].p;
    const Fmod f = fmod_of(p);
    double *F = fact + (size_t)blockIdx.x * 2 * (256 * C);
    double A[C], iA[C], prev;
    prefix_inverses<C>(f, p, s.v, [](int i) { return i ? (double)i : 1.0; }, A, iA, prev);
WV_UNROLL
    for (int i = 0; i < C; i++) s.v[stage_at(tid * C + i)] = A[i];
    stage_store<C, 256 * C>(s, F);
WV_UNROLL
    for (int i = 0; i < C; i++) s.v[stage_at(tid * C + i)] = iA[i];
    stage_store<C, 256 * C>(s, F + 256 * C);
}

// Level arrays of one doubling step (blocks of k terms, L = 2 (k + 1) = 256
// C): for shift s of prime i, a(n) = K n (s = 0: the next k + 1 nodes), k + K
// (n - L/2) (s = 1: the nodes moved by k) or k + K n (s = 2: both); beta[n] =
// 1 / a(n), n >= 1, and pi[t] = prod_{t < n <= t + L/2} a(n), the factor
// prod (X - Y_i) at point t.  cst[i] = K^-k.
template <int C>
__global__ void __launch_bounds__(256) k_grid_level(const PrimeRec *__restrict__ pr, uint32_t K,
                                                    double *__restrict__ beta, double *__restrict__ pi,
                                                    double *__restrict__ cst) {
    constexpr int L = 256 * C, k = L / 2 - 1;
    __shared__ Stage<C> s;
    const int tid = threadIdx.x;
    const uint32_t i = blockIdx.x / 3, sh = blockIdx.x - 3 * i;
    const uint64_t p = pr[i].p;
    const Fmod f = fmod_of(p);
    const double Kd = (double)K;
    const double a0 = sh == 0 ? 0.0 : (sh == 1 ? (double)k - Kd * (double)(k + 1) : (double)k);
    double A[C], iA[C], prev;
    prefix_inverses<C>(f, p, s.v, [&](int n) { return n ? fma((double)n, Kd, a0) : 1.0; }, A, iA, prev);
WV_UNROLL
    for (int e = 0; e < C; e++) s.v[stage_at(tid * C + e)] = f_mulmod(iA[e], e ? A[e ? e - 1 : 0] : prev, f);
    stage_store<C, L>(s, beta + (size_t)blockIdx.x * L);
    // A of the upper half meets 1 / A of the lower half
    if (tid >= 128) {
WV_UNROLL
        for (int e = 0; e < C; e++) s.v[stage_at((tid - 128) * C + e)] = A[e];
    }
    __syncthreads();
    if (tid < 128) {
WV_UNROLL
        for (int e = 0; e < C; e++) s.v[stage_at(tid * C + e)] = f_mulmod(s.v[stage_at(tid * C + e)], iA[e], f);
    }
    stage_store<C, L / 2>(s, pi + (size_t)blockIdx.x * (L / 2));
    if (sh == 0) {
        const double c = f_pow_u(f_pow_u(Kd, p - 2, f), k, f);
        if (tid == 0) cst[i] = c;
    }
}

// ---------------------------------------------------------------------------
// node values
// ---------------------------------------------------------------------------

// Values of g_0 .. g_3 of blocks of kBaseK terms at the first kBaseK + 1 nodes,
// multiplied out (one thread per node, one workgroup per prime).
__global__ void __launch_bounds__(256) k_grid_base(const PrimeRec *__restrict__ pr, uint32_t K, double *__restrict__ node) {
    const uint64_t p = pr[blockIdx.x].p;
    const Fmod f = fmod_of(p);
    const int t = threadIdx.x;
    const double y = -(double)K * (double)(K + 1 - t);
    double g0 = 1.0, g1 = 0.0, g2 = 0.0, g3 = 0.0;
    for (int j = 0; j < kBaseK; j++) {
        const double a = y + (double)j;   // |a| <= K (K + 1) < p
        g3 = f_mulmod(g3, a, f) + g2;     // |g_k| < (0.574 + 0.574 k) p
        g2 = f_mulmod(g2, a, f) + g1;
        g1 = f_mulmod(g1, a, f) + g0;
        g0 = f_mulmod(g0, a, f);
    }
    double *o = node + (size_t)blockIdx.x * 4 * (kBaseK + 1) + t;
    o[0] = f_reduce(g0, f);
    o[kBaseK + 1] = f_reduce(g1, f);
    o[2 * (kBaseK + 1)] = f_reduce(g2, f);
    o[3 * (kBaseK + 1)] = f_reduce(g3, f);
}

// u_i / L of one value vector at the k + 1 = L/2 nodes, transformed (a
// workgroup per prime, vector and modulus): out[((prime 4 + j) 2 + q) L + ...]
// in the transform's own layout.
template <int LOGL>
__global__ void __launch_bounds__(NttShape<LOGL>::T, 4) k_grid_fwd(const PrimeRec *__restrict__ pr,
                                                                   const double *__restrict__ node,
                                                                   const double *__restrict__ fact, uint32_t K,
                                                                   const double *__restrict__ tab,
                                                                   double *__restrict__ out) {
    using S = NttShape<LOGL>;
    constexpr int E = S::E, T = S::T, L = S::L;
    __shared__ NttLds<LOGL> lds;
    const int tid = threadIdx.x;
    const uint32_t i = blockIdx.x >> 3, j = (blockIdx.x >> 1) & 3, q = blockIdx.x & 1;
    const Fmod fp = fmod_of(pr[i].p);
    const Fmod f = ntt_mod(q);
    const VecBuf tb = vec_buf(tab, 2 * S::STRIDE);
    const VecBuf v = vec_buf(node + ((size_t)i * 4 + j) * (L / 2), L / 2);
    const VecBuf iF = vec_buf(fact + (size_t)i * 2 * (K + 1) + (K + 1), K + 1);
    double x[E];
WV_UNROLL
    for (int e = 0; e < E / 2; e++) {
        // n = tid + T e: (-1)^(k-n) / (n! (k-n)!), k = L/2 - 1 odd, T even
        const double u = f_mulmod(f_mulmod(vec_load(v, tid, T * e), vec_load(iF, tid, T * e), fp),
                                  vec_load(iF, T - 1 - tid, L / 2 - T - T * e), fp);
        x[e] = (tid & 1) ? u : -u;
        x[E / 2 + e] = 0.0;
    }
    ntt_lds_tables<LOGL>(lds, tb, (int)q, tid);
    ntt_forward<LOGL>(x, lds, tb, (int)q, f, tid);
    // 1 / L mod q = -(q - 1) / L
    const double li = -(f.p - 1.0) / (double)L;
    const VecBuf o = vec_buf(out + (((size_t)i * 4 + j) * 2 + q) * L, L);
WV_UNROLL
    for (int m = 0; m < E; m++) vec_store(o, tid, m * T, f_mulmod(x[m], li, f));
}

// ---------------------------------------------------------------------------
// values at the block starts
// ---------------------------------------------------------------------------

struct ShiftArgs {
    const PrimeRec *pr;
    const double *beta;       // kernel entries
    const double *uhat;       // transformed node vectors
    const double *tab;
    double *out;              // level: residues mod q; runs: values mod p
    const SegRec *runs;       // runs only, from here
    const uint64_t *off;
    unsigned long long *counters;   // 8, one per XCD's share, zero at launch
    uint32_t nruns, nruns_b;
};

// One shift of a doubling step: residues mod q of every value vector at the
// L/2 points, out[((item 4 + j) 2 + q) L/2 + t]; a workgroup per (item =
// prime 3 + shift, modulus).
template <int LOGL>
__global__ void __launch_bounds__(NttShape<LOGL>::T, 4) k_grid_level_shift(ShiftArgs A) {
    using S = NttShape<LOGL>;
    constexpr int E = S::E, T = S::T, L = S::L;
    __shared__ NttLds<LOGL> lds;
    const int tid = threadIdx.x;
    const uint32_t item = blockIdx.x >> 1, q = blockIdx.x & 1, i = item / 3;
    const Fmod f = ntt_mod(q);
    const VecBuf tab = vec_buf(A.tab, 2 * S::STRIDE);
    double w[E], x[E], t1[E];
    load_vec<LOGL>(w, A.beta + (size_t)item * L, tid);
    ntt_lds_tables<LOGL>(lds, tab, (int)q, tid);
    const double *uh = A.uhat + ((size_t)i * 8 + q) * L;   // vector j at 2 j L
    ntt_forward<LOGL>(w, lds, tab, (int)q, f, tid);
    twiddle1_load<LOGL>(t1, tab, ntt_inverse_tw1<LOGL>((int)q), tid);
WV_NO_UNROLL
    for (int j = 0; j < 4; j++) {
        load_vec<LOGL>(x, uh + (size_t)(2 * j) * L, tid);
        mulmod_range<kNttGroup, 0, E>(x, w, f);
        ntt_inverse<LOGL>(x, t1, lds, (int)q, f, tid);
        const VecBuf o = vec_buf(A.out + (((size_t)item * 4 + j) * 2 + q) * (L / 2), L / 2);
WV_UNROLL
        for (int e = 0; e < E / 2; e++) vec_store(o, tid, e * T, f_reduce(x[E / 2 + e], f));
    }
}

// Where the values of an item's vectors start: W per vector, four vectors for
// an s^-3 shift, three for an s^-2 one (the s^-3 items, items_b of them, come
// first).
__device__ __forceinline__ uint64_t value_base(uint64_t item, uint64_t items_b, uint32_t W) {
    return (item < items_b ? 4 * item : items_b + 3 * item) * W;
}

// The next of `total` items for this workgroup: those of its XCD (one eighth,
// in order), then those the others have left; part counts the shares used up.
__device__ __forceinline__ bool next_item(unsigned long long *counters, uint64_t total, uint32_t &part,
                                          unsigned long long *ticket, uint64_t &item) {
    while (part < 8) {
        const uint32_t X = (blockIdx.x + part) & 7;
        __syncthreads();   // LDS free
        if (threadIdx.x == 0) *ticket = atomicAdd(&counters[X], 1ull);
        __syncthreads();
        item = total * X / 8 + readfirst_u64(*ticket);
        if (item < total * (X + 1) / 8) return true;
        part++;
    }
    return false;
}

// What bounds this kernel: issue of f64 operations (about 66 per element of a
// transform, 0.58 of the issue slots at L = 2^14), then the vector loads of
// node vectors, twiddles and values between them.  One transform at a time
// stays in a workgroup's registers (16 values a thread, four waves per SIMD);
// at L = 2^14 a workgroup fills a CU.
//
// The shifts of every run (persistent; the items split evenly over the eight
// XCDs, taken one by one, so that neighbouring items, which share a prime's
// node vectors, meet in one L2): values of g_0 .. g_d mod p at the W block
// starts, up to a factor common to one block start.
template <int LOGL>
__global__ void __launch_bounds__(NttShape<LOGL>::T, 4) k_grid_shift(ShiftArgs A) {
    using S = NttShape<LOGL>;
    constexpr int E = S::E, T = S::T, L = S::L, W = L / 2;
    __shared__ NttLds<LOGL> lds;
    __shared__ unsigned long long ticket;
    const int tid = threadIdx.x;
    const uint64_t total = A.off[A.nruns], items_b = A.off[A.nruns_b];
    const VecBuf tab = vec_buf(A.tab, 2 * S::STRIDE);
    uint32_t part = 0;
    uint64_t item;
    while (next_item(A.counters, total, part, &ticket, item)) {
        const uint32_t slot = __builtin_amdgcn_readfirstlane(find_seg(A.off, A.nruns, item));
        const uint32_t prime = __builtin_amdgcn_readfirstlane(A.runs[slot].prime);
        const int np = slot < A.nruns_b ? 4 : 3;
        const Fmod fp = fmod_of(readfirst_u64(A.pr[prime].p));
        const double q1p = f_reduce((double)kNttQ[0], fp);   // q1 mod p, balanced
        const double *beta = A.beta + (slot + item) * W;      // entry off[slot] + slot + (item - off[slot])
        const double *uh = A.uhat + (size_t)prime * 8 * L;   // vector j modulo q at (2 j + q) L
        const VecBuf out = vec_buf(A.out + value_base(item, items_b, W), np * W);
        double w[E], x[E], t1[E];
WV_NO_UNROLL
        for (int q = 0; q < 2; q++) {
            const Fmod f = ntt_mod(q);
            load_vec<LOGL>(w, beta, tid);
            ntt_lds_tables<LOGL>(lds, tab, q, tid);
            ntt_forward<LOGL>(w, lds, tab, q, f, tid);
            twiddle1_load<LOGL>(t1, tab, ntt_inverse_tw1<LOGL>(q), tid);
WV_NO_UNROLL
            for (int j = 0; j < np; j++) {
                load_vec<LOGL>(x, uh + (size_t)(2 * j + q) * L, tid);
                mulmod_range<kNttGroup, 0, E>(x, w, f);
                ntt_inverse<LOGL>(x, t1, lds, q, f, tid);
                // the residues mod q1 wait where the values go
                const int o = j * W;
                if (q == 0) {
WV_UNROLL
                    for (int e = 0; e < E / 2; e++) vec_store(out, tid, o + e * T, f_reduce(x[E / 2 + e], f));
                } else {
                    double r[E / 2];
WV_UNROLL
                    for (int e = 0; e < E / 2; e++) r[e] = vec_load(out, tid, o + e * T);
                    __builtin_amdgcn_sched_barrier(0);
WV_UNROLL
                    for (int e = 0; e < E / 2; e++)
                        vec_store(out, tid, o + e * T, ntt_crt(r[e], x[E / 2 + e], kNttQ1Inv, q1p, f, fp));
                }
            }
        }
    }
}

// Convolutions of length 2 N, N = 2^kNttMaxLog, modulo X^2N - 1 = (X^N - 1)
// (X^N + 1): of the halves' sum and difference, by transforms of N.  Of c's
// halves, c[N + n] = (c+[n] - c-[n]) / 2.
constexpr int kSplitN = 1 << kNttMaxLog;

// u_i / 2 N of one value vector, as k_grid_fwd: out[(((prime 4 + j) 2 + q) 2 + sub)
// N + ...], a workgroup each.
__global__ void __launch_bounds__(NttShape<kNttMaxLog>::T, 4) k_grid_fwd_split(
    const PrimeRec *__restrict__ pr, const double *__restrict__ node, const double *__restrict__ fact,
    const double *__restrict__ tab, const double *__restrict__ neg, double *__restrict__ out) {
    using S = NttShape<kNttMaxLog>;
    constexpr int E = S::E, T = S::T, N = S::L;
    __shared__ NttLds<kNttMaxLog> lds;
    const int tid = threadIdx.x;
    const uint32_t i = blockIdx.x >> 4, j = (blockIdx.x >> 2) & 3, q = (blockIdx.x >> 1) & 1, sub = blockIdx.x & 1;
    const Fmod fp = fmod_of(pr[i].p);
    const Fmod f = ntt_mod(q);
    const VecBuf tb = vec_buf(tab, 2 * S::STRIDE);
    const VecBuf v = vec_buf(node + ((size_t)i * 4 + j) * N, N);
    const VecBuf iF = vec_buf(fact + (size_t)i * 2 * N + N, N);   // K + 1 = N
    double x[E];
WV_UNROLL
    for (int e = 0; e < E; e++) {
        const double u = f_mulmod(f_mulmod(vec_load(v, tid, T * e), vec_load(iF, tid, T * e), fp),
                                  vec_load(iF, T - 1 - tid, N - T - T * e), fp);
        x[e] = (tid & 1) ? u : -u;
    }
    ntt_lds_tables<kNttMaxLog>(lds, tb, (int)q, tid);
    if (sub) ntt_forward_neg<kNttMaxLog>(x, lds, tb, neg, (int)q, f, tid);
    else ntt_forward<kNttMaxLog>(x, lds, tb, (int)q, f, tid);
    const double li = -(f.p - 1.0) / (double)(2 * N);   // 1 / 2 N mod q
    const VecBuf o = vec_buf(out + (size_t)blockIdx.x * N, N);
WV_UNROLL
    for (int m = 0; m < E; m++) vec_store(o, tid, m * T, f_mulmod(x[m], li, f));
}

// k_grid_shift for W = N block starts: 2 N terms of the kernel, two transforms
// of N each way per modulus and vector, so twice the work of a shift of N / 2
// block starts for four times its terms.  Bound by its memory traffic, which no
// longer stays in the L2s: of each vector and modulus 2 N values of the node
// vectors, and N of c+, which wait in the workgroup's share of half (np N
// values) for c-: 3.5 TB/s past the L2s, 0.44 of the f64 issue slots.  Shifts of 310
// primes near 1e11: 16.5 ms, by whole transforms 17.4.  (With c+ in registers, the
// kernel's transforms and the twiddles read again for every vector, 18.4; with
// the weights psi^n of X^N + 1 from memory instead of in the twiddles, 21.0.)
__global__ void __launch_bounds__(NttShape<kNttMaxLog>::T, 4) k_grid_shift_split(ShiftArgs A,
                                                                                 const double *__restrict__ neg,
                                                                                 double *__restrict__ half) {
    using S = NttShape<kNttMaxLog>;
    constexpr int E = S::E, T = S::T, N = S::L, LG = kNttMaxLog, G = 8;
    __shared__ NttLds<LG> lds;
    __shared__ unsigned long long ticket;
    const int tid = threadIdx.x;
    const uint64_t total = A.off[A.nruns], items_b = A.off[A.nruns_b];
    const VecBuf tab = vec_buf(A.tab, 2 * S::STRIDE);
    const VecBuf hb = vec_buf(half + (size_t)blockIdx.x * 4 * N, 4 * N);
    uint32_t part = 0;
    uint64_t item;
    while (next_item(A.counters, total, part, &ticket, item)) {
        const uint32_t slot = __builtin_amdgcn_readfirstlane(find_seg(A.off, A.nruns, item));
        const uint32_t prime = __builtin_amdgcn_readfirstlane(A.runs[slot].prime);
        const int np = slot < A.nruns_b ? 4 : 3;
        const Fmod fp = fmod_of(readfirst_u64(A.pr[prime].p));
        const double q1p = f_reduce((double)kNttQ[0], fp);
        const double *beta = A.beta + (slot + item) * N;      // 2 N entries
        const double *uh = A.uhat + (size_t)prime * 16 * N;   // vector j modulo q, part sub at ((2 j + q) 2 + sub) N
        const VecBuf out = vec_buf(A.out + value_base(item, items_b, N), np * N);
        double w[E], x[E], t1[E];
WV_NO_UNROLL
        for (int q = 0; q < 2; q++) {
            const Fmod f = ntt_mod(q);
            load_vec<LG>(w, beta, tid);
            load_vec<LG>(x, beta + N, tid);
WV_UNROLL
            for (int e = 0; e < E; e++) w[e] += x[e];
            ntt_lds_tables<LG>(lds, tab, q, tid);
            ntt_forward<LG>(w, lds, tab, q, f, tid);
            twiddle1_load<LG>(t1, tab, ntt_inverse_tw1<LG>(q), tid);
WV_NO_UNROLL
            for (int j = 0; j < np; j++) {
                load_vec<LG>(x, uh + (size_t)(2 * j + q) * 2 * N, tid);
                mulmod_range<kNttGroup, 0, E>(x, w, f);
                ntt_inverse<LG>(x, t1, lds, q, f, tid);
WV_UNROLL
                for (int e = 0; e < E; e++) vec_store(hb, tid, j * N + e * T, x[e]);
            }
            load_vec<LG>(w, beta, tid);
            load_vec<LG>(x, beta + N, tid);
WV_UNROLL
            for (int e = 0; e < E; e++) w[e] -= x[e];
            ntt_forward_neg<LG>(w, lds, tab, neg, q, f, tid);
            neg_twiddle1_load<LG>(t1, neg, 2 * q + 1, tid);
WV_NO_UNROLL
            for (int j = 0; j < np; j++) {
                load_vec<LG>(x, uh + ((size_t)(2 * j + q) * 2 + 1) * N, tid);
                mulmod_range<kNttGroup, 0, E>(x, w, f);
                ntt_inverse<LG, true>(x, t1, lds, q, f, tid);
                const int o = j * N;
WV_UNROLL
                for (int e0 = 0; e0 < E; e0 += G) {
                    double h[G];
WV_UNROLL
                    for (int e = 0; e < G; e++) h[e] = vec_load(hb, tid, o + (e0 + e) * T);
                    __builtin_amdgcn_sched_barrier(0);
WV_UNROLL
                    for (int e = 0; e < G; e++) x[e0 + e] = f_reduce(h[e] - x[e0 + e], f);   // < 20.6 q before
                }
                // the residues mod q1 wait where the values go
                if (q == 0) {
WV_UNROLL
                    for (int e = 0; e < E; e++) vec_store_stream(out, tid, o + e * T, x[e]);
                } else {
WV_UNROLL
                    for (int e0 = 0; e0 < E; e0 += G) {
                        double r[G];
WV_UNROLL
                        for (int e = 0; e < G; e++) r[e] = vec_load_stream(out, tid, o + (e0 + e) * T);
                        __builtin_amdgcn_sched_barrier(0);
WV_UNROLL
                        for (int e = 0; e < G; e++)
                            vec_store_stream(out, tid, o + (e0 + e) * T, ntt_crt(r[e], x[e0 + e], kNttQ1Inv, q1p, f, fp));
                    }
                }
            }
        }
    }
}

// Node values of the next doubling step: P_{2k+1} at 2 (k + 1) nodes from P_k at
// the first k + 1 (node), at the next ones (shift 0) and moved by k (shifts 1,
// 2).  One thread per (prime, node).
__global__ void __launch_bounds__(256) k_grid_combine(const PrimeRec *__restrict__ pr, uint32_t n, uint32_t K, uint32_t k,
                                                      const double *__restrict__ node, const double *__restrict__ res,
                                                      const double *__restrict__ pi, const double *__restrict__ cst,
                                                      double *__restrict__ next) {
    const uint64_t g = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    const uint32_t h = k + 1, L = 2 * h;
    if (g >= (uint64_t)n * L) return;
    const uint32_t i = (uint32_t)(g / L), t = (uint32_t)(g - (uint64_t)i * L);
    const Fmod fp = fmod_of(pr[i].p);
    const Fmod f2 = ntt_mod(1);
    const double q1p = f_reduce((double)kNttQ[0], fp);
    const uint32_t tt = t < h ? t : t - h;
    // values of shift s at point tt, times prod (X - Y_i) K^-k
    auto shifted = [&](uint32_t s, double (&v)[4]) {
        const size_t item = (size_t)i * 3 + s;
        const double w = f_mulmod(pi[item * h + tt], cst[i], fp);
        for (int j = 0; j < 4; j++) {
            const double r1 = res[((item * 4 + j) * 2) * h + tt], r2 = res[((item * 4 + j) * 2 + 1) * h + tt];
            v[j] = f_mulmod(ntt_crt(r1, r2, kNttQ1Inv, q1p, f2, fp), w, fp);
        }
    };
    double x[4], y[4];
    if (t < h) {
        for (int j = 0; j < 4; j++) x[j] = node[((size_t)i * 4 + j) * h + t];
        shifted(1, y);
    } else {
        shifted(0, x);
        shifted(2, y);
    }
    double z[4];
    z[0] = f_mulmod(x[0], y[0], fp);
    z[1] = f_mulmod(x[0], y[1], fp) + f_mulmod(x[1], y[0], fp);
    z[2] = f_mulmod(x[0], y[2], fp) + f_mulmod(x[1], y[1], fp) + f_mulmod(x[2], y[0], fp);
    z[3] = f_mulmod(x[0], y[3], fp) + f_mulmod(x[1], y[2], fp) + f_mulmod(x[2], y[1], fp) + f_mulmod(x[3], y[0], fp);
    const double last = (double)(2 * k) - (double)K * (double)(K + 1 - t);   // Y_t + 2 k
    double *o = next + (size_t)i * 4 * L + t;
    o[0] = f_reduce(f_mulmod(z[0], last, fp), fp);
    for (int j = 1; j < 4; j++) o[(size_t)j * L] = f_reduce(f_mulmod(z[j], last, fp) + z[j - 1], fp);
}

// Every (prime, sum): its blocks' pairs, from the values at their starts, and
// the terms of the blocks that hold its endpoints, joined (NW waves per sum;
// one where a sum has few blocks).  Reads each value once.
template <int NW>
__global__ void __launch_bounds__(NW == 1 ? 256 : 64 * NW) k_grid_join(
    const SegRec *__restrict__ segs, uint32_t n, int nB, int nE, const GridRuns *__restrict__ tabs, int tb, int te,
    const SegRec *__restrict__ runs, const uint64_t *__restrict__ off, const PrimeRec *__restrict__ pr,
    const double *__restrict__ vals, uint32_t K, int logw, Pair *__restrict__ seg_pairs) {
    __shared__ Pair part[NW];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint64_t nseg = (uint64_t)n * (nB + nE);
    const uint64_t j = NW == 1 ? (uint64_t)blockIdx.x * 4 + wave : blockIdx.x;
    const bool live = j < nseg;   // NW > 1: the grid has a workgroup per sum
    uint64_t c0 = 1, c1 = 0;
    Mont m;
    if (live) {
        const bool bern = j < (uint64_t)n * nB;
        const uint32_t k = (uint32_t)(bern ? j : j - (uint64_t)n * nB);
        const uint32_t i = k / (uint32_t)(bern ? nB : nE), sum = k - i * (uint32_t)(bern ? nB : nE);
        const uint32_t rB = tabs[tb].n, rE = tabs[te].n;
        const uint32_t slot = bern ? i * rB + tabs[tb].run[sum] : n * rB + i * rE + tabs[te].run[sum];
        const SegRec s = segs[j];
        const uint64_t run0 = runs[slot].lo;
        const PrimeRec P = pr[s.prime];
        m = mont_of(P);
        const Fmod f = fmod_of(P.p);
        const uint32_t me = NW == 1 ? lane : threadIdx.x;
        // blocks [b0, b1) of the run lie inside the sum
        const uint64_t d0 = s.len ? s.lo - run0 : 0;
        const uint64_t b0 = (d0 + K - 1) / K, b1 = max((d0 + s.len) / K, b0);
        double a0 = 1.0, a1 = 0.0;
        auto fold = [&](double P0, double Q) {
            a1 = f_mulmod(a0, Q, f) + f_mulmod(a1, P0, f);
            a0 = f_mulmod(a0, P0, f);
        };
        const uint32_t W = 1u << logw;
        const uint64_t first = off[slot], items_b = off[n * rB];
        const double *v0 = vals + value_base(first, items_b, W);
        const uint64_t per = (uint64_t)(bern ? 4 : 3) << logw;   // values of one item
        if (bern) {
            for (uint64_t t = b0 + me; t < b1; t += 64 * NW) {
                const double *v = v0 + (t >> logw) * per + (t & (W - 1));
                const double r0 = v[0], r1 = v[W], r2 = v[2 * W], r3 = v[3 * W];
                const double sq = f_mulmod(r0, r0, f);
                const double u = fma(f_mulmod(r0, r2, f), -3.0, f_mulmod(r1, r1, f));
                fold(f_mulmod(sq, r0, f), fma(f_mulmod(r3, sq, f), 3.0, f_mulmod(r1, u, f)));
            }
        } else {
            for (uint64_t t = b0 + me; t < b1; t += 64 * NW) {
                const double *v = v0 + (t >> logw) * per + (t & (W - 1));
                const double r0 = v[0], r1 = v[W], r2 = v[2 * W];
                const double u = f_mulmod(r0, r2, f);
                fold(f_mulmod(r0, r0, f), f_mulmod(r1, r1, f) - (u + u));
            }
        }
        // the terms before the first block and after the last (all of them
        // when no block fits)
        const uint64_t head = b1 > b0 ? b0 * K - d0 : s.len, gap = b1 > b0 ? (b1 - b0) * K : 0;
        for (uint64_t t = me; t < s.len - gap; t += 64 * NW) {
            const double v = (double)(s.lo + (t < head ? t : t + gap));
            const double v2 = f_mulmod(v, v, f);
            const double u = bern ? f_mulmod(v2, v, f) : v2;
            a1 = f_mulmod(a1, u, f) + a0;   // |a1| < 1.15 p
            a0 = f_mulmod(a0, u, f);
        }
        c0 = f_canon(a0, f);
        c1 = f_canon(a1, f);
        wave_pair_reduce(c0, c1, m);
        if (NW == 1 && lane == 0) seg_pairs[j] = Pair{c0, c1};
    }
    if (NW > 1) {
        if (lane == 0) part[wave] = Pair{c0, c1};
        __syncthreads();
        if (threadIdx.x == 0 && live) {
            for (int v = 1; v < NW; v++) pair_mul(c0, c1, part[v].c0, part[v].c1, m);
            seg_pairs[j] = Pair{c0, c1};
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

uint64_t mulmod_q(uint64_t a, uint64_t b, uint64_t q) { return (uint64_t)((unsigned __int128)a * b % q); }

uint64_t powmod_q(uint64_t a, uint64_t e, uint64_t q) {
    uint64_t r = 1;
    for (; e; e >>= 1, a = mulmod_q(a, a, q))
        if (e & 1) r = mulmod_q(r, a, q);
    return r;
}

double balanced(uint64_t v, uint64_t q) { return v > q / 2 ? -(double)(q - v) : (double)v; }

uint32_t bitrev(uint32_t v, int bits) {
    uint32_t r = 0;
    for (int i = 0; i < bits; i++) r |= ((v >> i) & 1) << (bits - 1 - i);
    return r;
}

// fn(integral_constant<int, c>), c a power of two from MIN on
template <int MIN, class F>
int with_chunks(int c, F &&fn) {
    switch (c) {
    case 2:
        if constexpr (MIN <= 2) return fn(std::integral_constant<int, 2>{});
        return WV_EINVAL;
    case 4: return fn(std::integral_constant<int, 4>{});
    case 8: return fn(std::integral_constant<int, 8>{});
    case 16: return fn(std::integral_constant<int, 16>{});
    case 32: return fn(std::integral_constant<int, 32>{});
    case 64: return fn(std::integral_constant<int, 64>{});
    default: return WV_EINVAL;
    }
}

// Constant data into an empty buffer (waited for; the buffer stays empty if it
// fails).
int upload_once(wv_ctx *c, DevBuf &buf, const void *h, size_t bytes) {
    WV_TRY(ensure(c, buf, bytes));
    const hipError_t e = hipMemcpyAsync(buf.ptr, h, bytes, hipMemcpyHostToDevice, c->stream);
    const hipError_t e2 = hipStreamSynchronize(c->stream);
    if (e != hipSuccess || e2 != hipSuccess) {
        (void)hipFree(buf.ptr);
        buf = DevBuf{};
        return WV_EHIP;
    }
    return WV_OK;
}

}  // namespace

// Twiddle tables of one length (both moduli), uploaded once per context.
int ntt_tables(wv_ctx *c, int logl) {
    DevBuf &buf = c->ntt_tab[logl];
    if (buf.ptr) return WV_OK;
    const uint64_t L = 1ull << logl;
    std::vector<double> h;
    std::vector<uint64_t> pw(L);
    const int rc = with_shape(logl, [&](auto s) -> int {
        using S = NttShape<decltype(s)::value>;
        h.resize(2 * S::STRIDE);
        for (int q = 0; q < 2; q++) {
            const uint64_t Q = kNttQ[q], w = powmod_q(kNttRoot[q], (1ull << 17) / L, Q);
            pw[0] = 1;
            for (uint64_t i = 1; i < L; i++) pw[i] = mulmod_q(pw[i - 1], w, Q);
            double *t = h.data() + (size_t)q * S::STRIDE;
            for (int k = 1; k <= S::NT; k++)
                for (uint64_t i = 0; i < (uint64_t)S::E; i++)
                    for (uint64_t x = 0; x < (uint64_t)S::N(k); x++) {
                        // root of order N(k - 1) to the power x bitrev(i)
                        const uint64_t n = (uint64_t)S::N(k - 1), e = bitrev((uint32_t)i, S::LE) * x % n;
                        t[S::table(k) + i * S::N(k) + x] = balanced(pw[L / n * e], Q);
                        t[S::DIR + S::table(k) + i * S::N(k) + x] = balanced(pw[L / n * ((n - e) % n)], Q);
                    }
        }
        return WV_OK;
    });
    WV_TRY(rc);
    return upload_once(c, buf, h.data(), h.size() * sizeof(double));
}

namespace {

// Product 1's twiddles modulo X^N + 1 of both moduli: those of ntt_tables times
// psi^t (forward) and psi^-t (inverse), psi of order 2 N, for thread t.
int split_table(wv_ctx *c) {
    if (c->ntt_split.ptr) return WV_OK;
    using S = NttShape<kNttMaxLog>;
    constexpr uint64_t N = S::L, T = S::T, M = 2 * N;
    std::vector<double> h(4 * N);
    std::vector<uint64_t> pw(M);
    for (int q = 0; q < 2; q++) {
        const uint64_t Q = kNttQ[q], w = powmod_q(kNttRoot[q], (1ull << 17) / M, Q);
        pw[0] = 1;
        for (uint64_t i = 1; i < M; i++) pw[i] = mulmod_q(pw[i - 1], w, Q);
        for (uint64_t m = 0; m < (uint64_t)S::E; m++)
            for (uint64_t t = 0; t < T; t++) {
                const uint64_t e = (2 * bitrev((uint32_t)m, S::LE) + 1) * t % M;
                h[(2 * q) * N + m * T + t] = balanced(pw[e], Q);
                h[(2 * q + 1) * N + m * T + t] = balanced(pw[(M - e) % M], Q);
            }
    }
    return upload_once(c, c->ntt_split, h.data(), h.size() * sizeof(double));
}

// The runs of the compiled tables, uploaded once per context.
int runs_table(wv_ctx *c) {
    if (c->grid_tabs.ptr) return WV_OK;
    std::vector<GridRuns> h(WV_TABLE_EE33 + 1);
    for (int i = 0; i <= WV_TABLE_EE33; i++) h[i] = grid_runs(i);
    return upload_once(c, c->grid_tabs, h.data(), h.size() * sizeof(GridRuns));
}

// Bytes of device memory a batch of n primes needs besides the plan's records.
struct GridLayout {
    size_t node0, node1, fact, beta, pi, cst, uhat, res, inv, vals, counters, half, total;
};

size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

GridLayout grid_layout(const GridClass &g, uint64_t n, uint64_t pmax, unsigned blocks) {
    const uint64_t L = 1ull << g.logl, W = L / 2;
    const uint64_t nruns = n * (grid_runs(g.tb).n + grid_runs(g.te).n);
    const uint64_t items_b = n * grid_shifts(g.tb, (double)pmax, g.logl);
    const uint64_t items_e = n * grid_shifts(g.te, (double)pmax, g.logl);
    GridLayout y;
    size_t at = 0;
    auto take = [&](size_t &where, size_t doubles) {
        where = at;
        at += up256(doubles * sizeof(double));
    };
    take(y.node0, n * 4 * W);
    take(y.node1, n * 4 * W);
    take(y.fact, n * 2 * W);
    take(y.beta, n * 3 * W);
    take(y.pi, n * 3 * W / 2);
    take(y.cst, n);
    take(y.uhat, n * 8 * L);
    take(y.res, n * 12 * W);
    take(y.inv, (items_b + items_e + nruns) * W);
    take(y.vals, (4 * items_b + 3 * items_e) * W);
    take(y.counters, 8);
    take(y.half, g.logl > kNttMaxLog ? (size_t)blocks * 4 * W : 0);   // a share per workgroup of the shifts
    y.total = at;
    return y;
}

constexpr size_t kGridBytes = (size_t)8 << 30;   // workspace of one sub-batch, at most

// Workgroups of the persistent kernel: four waves per SIMD of 128 registers.
unsigned grid_blocks(const wv_ctx *c, int logl) {
    const int T = (1 << std::min(logl, kNttMaxLog)) / (logl >= 10 ? 16 : 8);
    return (unsigned)std::max(8, c->num_cus * (1024 / T) / 8 * 8);
}

template <int C>
void launch_inv(hipStream_t st, unsigned grid, const SegRec *segs, const uint64_t *off, uint32_t nseg,
                const PrimeRec *pr, uint64_t K, int logw, double *inv) {
    hipLaunchKernelGGL(k_grid_inv<C>, dim3(grid), dim3(256), 0, st, segs, off, nseg, pr, K, logw, inv);
}

// One sub-batch of n primes, enqueued on st: results into d_out, terms summed
// added to terms (2 words on the device).
int grid_sub(wv_ctx *c, GridWork &b, hipStream_t st, const GridClass &g, const GridLayout &y, const uint64_t *d_primes,
             uint32_t n, unsigned long long *terms, wv_result *d_out) {
    const uint32_t K = (uint32_t)grid_k(g.logl);
    const int logw = g.logl - 1;
    const int nB = kTables[g.tb].n, nE = kTables[g.te].n;
    const uint64_t nseg = (uint64_t)n * (nB + nE);
    if (nseg >= (1ull << 31) || (uint64_t)n * (K + 1) >= (1ull << 31)) return WV_EINVAL;
    PrimeRec *pr = as<PrimeRec>(b.pr);
    SegRec *segs = as<SegRec>(b.segs), *runs = as<SegRec>(b.runs);
    uint64_t *off = as<uint64_t>(b.off);
    const GridRuns *tabs = as<GridRuns>(c->grid_tabs);
    const uint32_t nruns_b = n * grid_runs(g.tb).n, nruns = nruns_b + n * grid_runs(g.te).n;
    char *ws = as<char>(b.ws);
    auto at = [&](size_t o) { return reinterpret_cast<double *>(ws + o); };
    WV_HIP(launch_plan(st, d_primes, n, g.tb, g.te, g.tb, g.te, nB, nE, table_store(c), pr, segs,
                       as<uint64_t>(b.terms), as<uint64_t>(b.coefs), as<uint64_t>(b.lhsmod), 0));
    hipLaunchKernelGGL(k_grid_runs, dim3((nruns + 255) / 256), dim3(256), 0, st, segs, n, nB, nE, tabs, g.tb, g.te,
                       (uint64_t)K, logw, runs, as<uint64_t>(b.cnt), terms);
    WV_HIP(launch_scan(st, as<uint64_t>(b.cnt), nruns, off, as<uint64_t>(b.tiles)));
    const unsigned inv_grid = (unsigned)c->num_cus * 8;
    double *inv = at(y.inv);
    switch (logw) {
    case 10: launch_inv<16>(st, inv_grid, runs, off, nruns, pr, K, logw, inv); break;
    default: launch_inv<32>(st, inv_grid, runs, off, nruns, pr, K, logw, inv); break;
    }
    WV_TRY(with_chunks<(1 << kGridMinLog) / 512>((int)(K + 1) / 256, [&](auto c) -> int {
        hipLaunchKernelGGL(k_grid_fact<decltype(c)::value>, dim3(n), dim3(256), 0, st, pr, at(y.fact));
        return WV_OK;
    }));
    hipLaunchKernelGGL(k_grid_base, dim3(n), dim3(256), 0, st, pr, K, at(y.node0));
    double *node = at(y.node0), *next = at(y.node1);
    auto fwd = [&](int logl) -> int {
        return with_shape(logl, [&](auto s) -> int {
            constexpr int LG = decltype(s)::value;
            hipLaunchKernelGGL(k_grid_fwd<LG>, dim3(n * 8), dim3(NttShape<LG>::T), 0, st, pr, node, at(y.fact), K,
                               as<double>(c->ntt_tab[LG]), at(y.uhat));
            return WV_OK;
        });
    };
    for (int l = kNttMinLog; l < g.logl; l++) {
        const uint32_t k = (uint32_t)grid_k(l);
        WV_TRY(with_chunks<(1 << kNttMinLog) / 256>((1 << l) / 256, [&](auto c) -> int {
            hipLaunchKernelGGL(k_grid_level<decltype(c)::value>, dim3(3 * n), dim3(256), 0, st, pr, K, at(y.beta),
                               at(y.pi), at(y.cst));
            return WV_OK;
        }));
        WV_TRY(fwd(l));
        WV_TRY(with_shape(l, [&](auto s) -> int {
            constexpr int LG = decltype(s)::value;
            ShiftArgs a{};
            a.beta = at(y.beta);
            a.uhat = at(y.uhat);
            a.tab = as<double>(c->ntt_tab[LG]);
            a.out = at(y.res);
            hipLaunchKernelGGL(k_grid_level_shift<LG>, dim3(6 * n), dim3(NttShape<LG>::T), 0, st, a);
            return WV_OK;
        }));
        const uint64_t points = (uint64_t)n * 2 * (k + 1);
        hipLaunchKernelGGL(k_grid_combine, dim3((unsigned)((points + 255) / 256)), dim3(256), 0, st, pr, n, K, k, node,
                           at(y.res), at(y.pi), at(y.cst), next);
        std::swap(node, next);
    }
    const bool split = g.logl > kNttMaxLog;
    if (split)
        hipLaunchKernelGGL(k_grid_fwd_split, dim3(n * 16), dim3(NttShape<kNttMaxLog>::T), 0, st, pr, node, at(y.fact),
                           as<double>(c->ntt_tab[kNttMaxLog]), as<double>(c->ntt_split), at(y.uhat));
    else
        WV_TRY(fwd(g.logl));
    WV_HIP(launch_set_u64(st, reinterpret_cast<uint64_t *>(at(y.counters)), 8, 0));
    ShiftArgs a{};
    a.pr = pr;
    a.beta = inv;
    a.uhat = at(y.uhat);
    a.tab = as<double>(c->ntt_tab[std::min(g.logl, kNttMaxLog)]);
    a.out = at(y.vals);
    a.runs = runs;
    a.off = off;
    a.counters = reinterpret_cast<unsigned long long *>(at(y.counters));
    a.nruns = nruns;
    a.nruns_b = nruns_b;
    if (split)
        hipLaunchKernelGGL(k_grid_shift_split, dim3(grid_blocks(c, g.logl)), dim3(NttShape<kNttMaxLog>::T), 0, st, a,
                           as<double>(c->ntt_split), at(y.half));
    else WV_TRY(with_shape(g.logl, [&](auto s) -> int {
        constexpr int LG = decltype(s)::value;
        if constexpr (LG >= kGridMinLog) {
            hipLaunchKernelGGL(k_grid_shift<LG>, dim3(grid_blocks(c, LG)), dim3(NttShape<LG>::T), 0, st, a);
            return WV_OK;
        }
        return WV_EINVAL;
    }));
    auto join = [&](auto nw) {
        constexpr int NW = decltype(nw)::value;
        hipLaunchKernelGGL(k_grid_join<NW>, dim3(NW == 1 ? (unsigned)((nseg + 3) / 4) : (unsigned)nseg),
                           dim3(NW == 1 ? 256 : 64 * NW), 0, st, segs, n, nB, nE, tabs, g.tb, g.te, runs, off, pr,
                           at(y.vals), K, logw, as<Pair>(b.seg_pairs));
    };
    // a wave's reduction costs about what 50 of its terms or blocks do, so
    // batches of many sums take few waves each (those of 2416 primes near 1e9 1.24
    // ms with eight, 0.75 with two), small ones enough to end soon
    if (nseg < 2048) join(std::integral_constant<int, 8>{});
    else if (K < 2047) join(std::integral_constant<int, 1>{});
    else if (K < 8191) join(std::integral_constant<int, 2>{});
    else join(std::integral_constant<int, 8>{});
    WV_HIP(hipGetLastError());
    WV_HIP(launch_finalize(st, table_store(c), pr, as<Pair>(b.seg_pairs), as<uint64_t>(b.coefs),
                           as<uint64_t>(b.lhsmod), n, nB, nE, d_out, nullptr));
    return WV_OK;
}

}  // namespace

// The path serves contexts with the default congruences, whose residues any
// printed congruence gives; a table the caller chose or defined, a forced shape
// or chunk, and a progress callback (called between term-sum launches) keep the
// term sums.
bool grid_allowed(const wv_ctx *c, int tb, int te) {
    return tb == WV_TABLE_BB30 && te == WV_TABLE_EE33 && !c->shape_forced && !c->chunk_cfg && !c->progress;
}

bool grid_takes(const wv_ctx *c, uint64_t p, GridClass *g) {
    if (p < kGridMinP || !grid_allowed(c, c->tb, c->te)) return false;
    *g = grid_class(p);
    return true;
}

int grid_enqueue(wv_ctx *c, GridWork &b, hipStream_t st, const GridClass &own, const uint64_t *d_primes, uint32_t n,
                 uint64_t pmin, uint64_t pmax, unsigned long long *terms, wv_result *d_out) {
    if (n == 0) return WV_OK;
    // a difference of two points could be p, and its inverse and those found with it 0
    if (!grid_fits(pmin, own.logl) || (own.logl > kNttMaxLog && pmax > kGridSplitMaxP)) return WV_EINVAL;
    const GridClass g = grid_batch_class(own, n, pmax);   // no longer than own
    for (int l = kNttMinLog; l <= std::min(g.logl, kNttMaxLog); l++) WV_TRY(ntt_tables(c, l));
    if (g.logl > kNttMaxLog) WV_TRY(split_table(c));
    WV_TRY(runs_table(c));
    // sub-batches within the workspace bound, or within what the device has left
    const unsigned blocks = grid_blocks(c, g.logl);
    const size_t one = grid_layout(g, 64, pmax, 0).total / 64 + 1;
    uint32_t step = (uint32_t)std::min<uint64_t>(n, std::max<uint64_t>(1, kGridBytes / one));
    step = std::min<uint32_t>(step, 1u << 16);
    GridLayout y;
    auto reserve = [&]() -> int {
        y = grid_layout(g, step, pmax, blocks);
        const uint64_t nseg = (uint64_t)step * (kTables[g.tb].n + kTables[g.te].n);
        WV_TRY(ensure(c, b.pr, step * sizeof(PrimeRec)));
        WV_TRY(ensure(c, b.segs, nseg * sizeof(SegRec)));
        WV_TRY(ensure(c, b.runs, nseg * sizeof(SegRec)));   // no more runs than sums
        WV_TRY(ensure(c, b.terms, nseg * sizeof(uint64_t)));
        WV_TRY(ensure(c, b.cnt, nseg * sizeof(uint64_t)));
        WV_TRY(ensure(c, b.off, (nseg + 1) * sizeof(uint64_t)));
        WV_TRY(ensure(c, b.tiles, ((nseg + kScanTile - 1) / kScanTile + 1) * sizeof(uint64_t)));
        WV_TRY(ensure(c, b.seg_pairs, nseg * sizeof(Pair)));
        WV_TRY(ensure(c, b.coefs, nseg * sizeof(uint64_t)));
        WV_TRY(ensure(c, b.lhsmod, 2 * (size_t)step * sizeof(uint64_t)));
        return ensure(c, b.ws, y.total);
    };
    for (;;) {
        const uint32_t parts = (n + step - 1) / step;
        step = (n + parts - 1) / parts;
        const int rc = reserve();
        if (rc == WV_OK) break;
        if (rc != WV_ENOMEM || step == 1) return rc;
        step = (step + 1) / 2;
    }
    for (uint32_t i = 0; i < n; i += step)
        WV_TRY(grid_sub(c, b, st, g, y, d_primes + i, std::min(step, n - i), terms, d_out + i));
    return WV_OK;
}

void grid_free(GridWork &b) {
    DevBuf *bufs[] = {&b.pr, &b.segs, &b.runs, &b.terms, &b.cnt, &b.off, &b.tiles, &b.seg_pairs, &b.coefs, &b.lhsmod, &b.ws};
    for (DevBuf *x : bufs)
        if (x->ptr) (void)hipFree(x->ptr);
}

int grid_batch_sync(wv_ctx *c, const GridClass &own, const uint64_t *d_primes, uint32_t n, uint64_t pmin,
                    uint64_t pmax, wv_result *d_out) {
    if (n == 0) return WV_OK;
    const GridClass g = grid_batch_class(own, n, pmax);   // as grid_enqueue takes it
    hipStream_t st = c->stream;
    auto *terms = as<unsigned long long>(c->scal);
    WV_HIP(hipEventRecord(c->ev[EV_PLAN0], st));
    WV_HIP(launch_set_u64(st, as<uint64_t>(c->scal), 8, 0));
    WV_TRY(grid_enqueue(c, c->grid, st, own, d_primes, n, pmin, pmax, terms, d_out));
    WV_HIP(hipEventRecord(c->ev[EV_FINAL], st));
    uint64_t host[2];
    WV_HIP(hipMemcpyAsync(host, terms, sizeof(host), hipMemcpyDeviceToHost, st));
    WV_HIP(hipStreamSynchronize(st));
    wv_stats &s = c->stats;
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, c->ev[EV_PLAN0], c->ev[EV_FINAL]);
    s.ms_total += ms;
    s.ms_sum += ms;   // the phases are not timed apart
    s.n_primes += n;
    s.n_sums += (uint64_t)n * (kTables[g.tb].n + kTables[g.te].n);
    s.n_terms += host[0];
    s.n_terms_b += host[1];
    s.chunk_terms = grid_k(g.logl);
    s.block_k_b = (uint32_t)sum_variant_kb(c->variant);
    s.block_k_e = (uint32_t)sum_variant_ke(c->variant);
    s.grid = grid_blocks(c, g.logl);
    return WV_OK;
}

// ---------------------------------------------------------------------------
// request server: primes of a step out of the pool, results into it
// ---------------------------------------------------------------------------

namespace {

// Pool slot of prime q of a step: span[a] holds primes q0 .. q0 + cnt - 1 at
// pool slots i0 .. (spans ascending in q0).
__device__ __forceinline__ uint32_t span_slot(const StepSpan *__restrict__ sp, uint32_t nsp, uint32_t q) {
    uint32_t a = 0, b = nsp;
    while (b - a > 1) {
        const uint32_t m = (a + b) >> 1;
        if (sp[m].q0 <= q) a = m;
        else b = m;
    }
    return sp[a].i0 + (q - sp[a].q0);
}

__global__ void __launch_bounds__(256) k_pool_gather(const StepSpan *__restrict__ sp, uint32_t nsp, uint32_t n,
                                                     const uint64_t *__restrict__ plist, uint64_t *__restrict__ out) {
    const uint32_t q = blockIdx.x * 256 + threadIdx.x;
    if (q < n) out[q] = plist[span_slot(sp, nsp, q)];
}

__global__ void __launch_bounds__(256) k_pool_scatter(const StepSpan *__restrict__ sp, uint32_t nsp, uint32_t n,
                                                      const wv_result *__restrict__ res, wv_result *__restrict__ pool) {
    const uint32_t q = blockIdx.x * 256 + threadIdx.x;
    if (q < n) pool[span_slot(sp, nsp, q)] = res[q];
}

// Results of finished requests (pool slots base .. base + n - 1) to out + out0.
__global__ void __launch_bounds__(256) k_pool_results(const FinReq *__restrict__ fr, uint32_t nfr,
                                                      const wv_result *__restrict__ pool, wv_result *__restrict__ out) {
    const FinReq f = fr[blockIdx.x];
    for (uint32_t i = threadIdx.x; i < f.n; i += 256) out[f.out0 + i] = pool[f.base + i];
}

}  // namespace

hipError_t launch_pool_gather(hipStream_t st, const StepSpan *sp, uint32_t nsp, uint32_t n, const uint64_t *plist,
                              uint64_t *out) {
    hipLaunchKernelGGL(k_pool_gather, dim3((n + 255) / 256), dim3(256), 0, st, sp, nsp, n, plist, out);
    return hipGetLastError();
}

hipError_t launch_pool_scatter(hipStream_t st, const StepSpan *sp, uint32_t nsp, uint32_t n, const wv_result *res,
                               wv_result *pool) {
    hipLaunchKernelGGL(k_pool_scatter, dim3((n + 255) / 256), dim3(256), 0, st, sp, nsp, n, res, pool);
    return hipGetLastError();
}

hipError_t launch_pool_results(hipStream_t st, const FinReq *fr, uint32_t nfr, const wv_result *pool, wv_result *out) {
    hipLaunchKernelGGL(k_pool_results, dim3(nfr), dim3(256), 0, st, fr, nfr, pool, out);
    return hipGetLastError();
}

}  // namespace wv
