// wv_irregular.hip -- irregular and E-irregular pairs: B_{2k} mod p and
// E_{2k} mod p for every 2 <= 2k <= p - 3 (Section 1), from the paper's
// congruences for general index:
//
//   C_k(a,b,c) B_{2k} == sum_i S_{2k-1}(x_i, y_i)   (mod p)     (Section 2:
//     the family (2, b, b+1) over sum_{m <= b/2} (m/(b+1), m/b): b = 3, i.e.
//     (1/4, 1/3), for every k, then b = 4, 5, ... where C_k(2,3,4) vanishes),
//   C_k(a,b,c) = (a^{p-2k} + b^{p-2k} - c^{p-2k} - 1) / (4k),
//   (-1)^k 4^{k-1} (9^k + 1) E_t == 2^t (S_t(0, 1/12) - S_t(5/12, 1/2))
//     (mod p), t = p - 1 - 2k  (eqnEMac2, Section 4: McIntosh's congruence
//     with one subdivision), and where 9^k == -1 (mod p)
//   (-1)^k 4^{2k-1} E_t == S_t(0, 1/4)   (mod p)  (eqnE1, sign read as (-1)^k),
//
// with S_l(x, y) = sum_{xp < s < yp} s^l (eqnDefnS) for positive l.  Every k
// needs its own exponent, so the power sums of each range are computed for all
// exponents at once: a wave owns 1024 consecutive s (16 per lane) and a block
// of up to 2048 exponents, steps x <- x s^2 through them, and the partial sums
// go through LDS (one transpose per 32 exponents) into exact double-precision
// totals (integers below 2^53, so the order of the atomic additions does not
// matter).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "ntt.hpp"
#include "sum_core.hpp"
#include "wave_ops.hpp"
#include "wv_ctx.hpp"

namespace wv {
namespace {

struct IrrTask {          // +- sum_{lo <= s < hi} s^t for t = t0, t0 + 2, ..., t0 + 2 (nt - 1)
    uint64_t p, lo, hi;
    uint64_t out;         // index in V of the first exponent's total (tasks may share it)
    uint32_t t0, nt;
    uint32_t ct;          // matrix-core path: exponents per row = 16 ct (1 <= ct <= 8)
    uint32_t neg;         // 1: the sums enter V negated
};

struct IrrPrime {         // one prime of a batch
    uint64_t p;
    uint64_t vb, ve;      // its Bernoulli (odd t = 2k - 1) and Euler (even t = 2k) totals in V
    uint64_t res;         // index of its first residue in the b / e output arrays
    uint32_t nt;          // (p - 3) / 2
    uint32_t pad;
};

struct IrrFix {           // an index whose first congruence degenerates (its left side is 0 mod p)
    uint32_t prime, k;    // Bernoulli side: B_{2k}; Euler side: E_{2k}
};

constexpr int kIrrLaneS = 16;                        // s per lane
constexpr uint64_t kIrrWaveS = 64 * kIrrLaneS;       // s per wave (one work unit)
constexpr int kIrrBlock = 32;                        // exponents per transpose
constexpr uint32_t kIrrUnitT = 2048;                 // exponents per work unit
constexpr int kIrrStride = 65;                       // LDS row stride (doubles)
constexpr uint64_t kIrrMaxV = 1ull << 27;            // totals per batch (1 GiB)
constexpr uint64_t kIrrMaxUnits = (1ull << 24) - 64;  // units per launch (fewer than 2^32 work-items)

__host__ __device__ inline uint64_t floor_div(uint64_t a, uint64_t b) { return a / b; }

// first and one-past-last s of x p < s < y p, x = xa/xb, y = ya/yb (p prime > xb, yb)
__host__ __device__ inline void open_range(uint64_t p, uint64_t xa, uint64_t xb, uint64_t ya, uint64_t yb,
                                           uint64_t &lo, uint64_t &hi) {
    lo = floor_div(xa * p, xb) + 1;
    hi = ya * p % yb ? floor_div(ya * p, yb) + 1 : ya * p / yb;   // s < y p
    if (hi < lo) hi = lo;
}

__device__ inline double fpow_e(double a, uint64_t e, const Fmod &f) {
    double r = 1.0;
    while (e) {
        if (e & 1) r = f_mulmod(r, a, f);
        a = f_mulmod(a, a, f);
        e >>= 1;
    }
    return r;
}

// a^e for e < 8 without branches
__device__ inline double fpow_lt8(double a, uint32_t e, const Fmod &f) {
    const double a2 = f_mulmod(a, a, f), a4 = f_mulmod(a2, a2, f);
    double r = (e & 1) ? a : 1.0;
    const double r2 = f_mulmod(r, a2, f);
    r = (e & 2) ? r2 : r;
    const double r4 = f_mulmod(r, a4, f);
    return (e & 4) ? r4 : r;
}

__device__ inline uint64_t u_pow(uint64_t a, uint64_t e, const Fmod &f) {
    return f_canon(fpow_e((double)a, e, f), f);
}

// C_k(a, b, c) mod p for 1 <= k <= (p - 3) / 2
__device__ inline uint64_t c_k(uint64_t a, uint64_t b, uint64_t c, uint64_t k, const Fmod &f, uint64_t p) {
    const uint64_t e = p - 2 * k;
    double num = fpow_e((double)a, e, f) + fpow_e((double)b, e, f) - fpow_e((double)c, e, f) - 1.0;
    const uint64_t n = f_canon(f_reduce(num, f), f);
    const uint64_t inv4k = u_pow((4 * k) % p, p - 2, f);
    return f_canon(f_mulmod((double)n, (double)inv4k, f), f);
}

// ---------------------------------------------------------------------------
// power sums for all exponents
// ---------------------------------------------------------------------------

__global__ void __launch_bounds__(256) k_irr_sum(const IrrTask *__restrict__ tasks,
                                                 const uint64_t *__restrict__ unit_off, uint32_t ntask,
                                                 uint64_t nunits, double *__restrict__ V) {
    __shared__ double lds[4][kIrrBlock * kIrrStride];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint64_t unit = (uint64_t)blockIdx.x * 4 + wave;   // wave-uniform
    if (unit >= nunits) return;
    const uint32_t j = __builtin_amdgcn_readfirstlane(find_seg(unit_off, ntask, unit));
    const IrrTask T = tasks[j];
    Fmod f;
    f.p = (double)T.p;
    f.pinv = 1.0 / f.p;
    // unit = (s chunk, exponent block): 1024 s times at most kIrrUnitT exponents
    const uint32_t nblk = (T.nt + kIrrUnitT - 1) / kIrrUnitT;
    const uint64_t u = unit - unit_off[j];
    const uint32_t e_first = (uint32_t)(u % nblk) * kIrrUnitT;
    const uint32_t e_end = min(T.nt, e_first + kIrrUnitT);
    const uint64_t s0 = T.lo + (u / nblk) * kIrrWaveS + lane;
    double x[kIrrLaneS], sq[kIrrLaneS];
WV_UNROLL
    for (int m = 0; m < kIrrLaneS; m++) {
        const uint64_t s = s0 + 64 * (uint64_t)m;
        const double sd = (double)s;
        const double s2 = f_mulmod(sd, sd, f);
        const bool in = s < T.hi;
        // s^(t0 + 2 e_first)
        const double xs = fpow_e(sd, T.t0 + 2 * (uint64_t)e_first, f);
        x[m] = in ? xs : 0.0;
        sq[m] = in ? s2 : 0.0;
    }
    double *L = lds[wave];
    for (uint32_t b0 = e_first; b0 < e_end; b0 += kIrrBlock) {
#pragma unroll 2
        for (int e = 0; e < kIrrBlock; e++) {
            double a = 0.0;
WV_UNROLL
            for (int m = 0; m < kIrrLaneS; m++) a += x[m];   // |a| < 16 * 0.574 p, exact
WV_UNROLL
            for (int m = 0; m < kIrrLaneS; m++) x[m] = f_mulmod(x[m], sq[m], f);
            L[e * kIrrStride + lane] = a;
        }
        // the wave's own LDS rows: complete its writes before reading across lanes
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // lane l and l + 32 each sum half of exponent (l & 31)'s row
        const int row = lane & 31, half = lane >> 5;
        double t = 0.0;
        for (int m = 0; m < 32; m++) t += L[row * kIrrStride + half * 32 + m];
        t += __shfl_xor(t, 32, 64);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (half == 0 && b0 + row < e_end) atomicAdd(&V[T.out + b0 + row], T.neg ? -t : t);
    }
}

// The same totals as a dense contraction on the matrix cores, for p < 2^24:
// with e = N m + j (N = 16 ct exponents per row, ct chosen per task so that
// the rows fill whole row blocks), s^(t0 + 2e) = A[m][s] B[s][j],
// A[m][s] = s^(t0 + 2N m), B[s][j] = s^(2j), so V[m][j] = sum_s A[m][s] B[s][j].  Residues below 0.574p
// make every product an integer below 0.33 p^2 (< 2^46.4), so the f64
// multiply-adds are exact while a partial sum stays below 2^53: the
// accumulators are reduced mod p after every `period` chunks of 32 s, the
// most whose products stay below 2^52 (32 chunks = 1024 s for p < 2^21, one
// chunk near 2^24), and before their atomic additions.  A
// workgroup takes (task, 128 rows of m, kMmaSb s) with twelve waves in two roles: four producer waves
// build the A (128 x 32) and transposed B (N x 32) slices of the next 32 s in
// one LDS buffer while eight consumer waves run v_mfma_f64_16x16x4 on the
// other (each its 16 rows x N columns, ct operations per 4 s), one barrier per
// 32 s.  Each SIMD holds two consumer waves (one issues while the other waits
// on LDS) and one producer wave, so the table arithmetic on the vector ALU
// overlaps the matrix cores.
constexpr int kMmaRows = 128;                // rows of m per workgroup
constexpr int kMmaKc = 32;                   // s per LDS chunk
constexpr uint64_t kMmaSb = 1024;            // s per workgroup
constexpr uint32_t kMmaReduceMax = 1024 / kMmaKc;   // chunks between reductions of the accumulators, at most
constexpr uint64_t kIrrMmaMaxP = 1ull << 24;
constexpr int kMmaConsumers = 512;           // 8 consumer waves, 16 rows each
constexpr int kMmaThreads = kMmaConsumers + 256;   // and 4 producer waves
constexpr uint64_t kMmaMaxGrid = 1ull << 22;       // workgroups per launch (2^22 x 768 < 2^32 work-items)
// LDS row stride (doubles) of A and of the transposed B: a wave's fragment
// reads (16 rows x 4 s) then touch each bank pair at most twice
constexpr int kMmaAs = kMmaKc + 4;

typedef double v4d __attribute__((ext_vector_type(4)));

// One 32-s chunk of a consumer wave: its 16 rows x 16 CT columns.  CT is
// compile-time; the LDS operands of the next 4-s step are read while the
// matrix operations of the current one run (two register sets; the group
// barriers put the reads (mask 0x100) ahead of the matrix operations (mask
// 0x8), the fence keeps them from being hoisted further).
template <int CT>
__device__ __forceinline__ void mma_chunk(const double *A, const double *B, int wave, int lane, v4d (&acc)[8]) {
    double a[2], b[2][CT];
    const double *Ar = A + (16 * wave + (lane & 15)) * kMmaAs + (lane >> 4);
    const double *Br = B + (lane & 15) * kMmaAs + (lane >> 4);
    auto load = [&](int kk, int slot) {
        a[slot] = Ar[4 * kk];
WV_UNROLL
        for (int n = 0; n < CT; n++) b[slot][n] = Br[16 * n * kMmaAs + 4 * kk];
    };
    load(0, 0);
WV_UNROLL
    for (int kk = 0; kk < kMmaKc / 4; kk++) {
        const int cur = kk & 1;
        if (kk + 1 < kMmaKc / 4) load(kk + 1, cur ^ 1);
WV_UNROLL
        for (int n = 0; n < CT; n++)
            acc[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[cur], b[cur][n], acc[n], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1 + CT, 0);
        __builtin_amdgcn_sched_group_barrier(0x8, CT, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The workgroup's unit (task T, row block rb of M rows, s in [sb0, sb1)) with
// N = 16 CT exponents per row; CT is compile-time so that each width has its
// own accumulators and straight-line matrix code.
template <int CT>
__device__ __forceinline__ void irr_mma_unit(const IrrTask &T, const Fmod &f, uint32_t period, uint32_t rb, uint32_t M,
                                             uint64_t sb0, uint64_t sb1, double (&As)[2][kMmaRows * kMmaAs],
                                             double (&Bs)[2][kMmaRows * kMmaAs], double *__restrict__ V) {
    constexpr uint32_t N = 16 * CT;
    const uint32_t m0 = rb * kMmaRows;
    const uint32_t nchunk = (uint32_t)((sb1 - sb0 + kMmaKc - 1) / kMmaKc);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const bool producer = tid >= kMmaConsumers;   // wave-uniform
    const int ptid = tid - kMmaConsumers;

    // tables of chunk c into buffer c & 1: producer thread (q, g) takes
    // s = sb0 + 32c + q and writes rows 16g .. 16g + 15 of A (A[m][s] =
    // s^(t0 + 2N(m0 + m))) and of the transposed B (Bt[j][s] = s^(2j); rows
    // j >= N are written and never read).  Every power comes from s^2, s^16,
    // s^32, s^(2N) = (s^32)^CT and its squares; the 16 entries of each table
    // run as two chains of 8, so a thread carries four independent chains.
    auto produce = [&](uint32_t c) {
        double *A = As[c & 1];
        double *Bt = Bs[c & 1];
        const int q = ptid & 31, g = ptid >> 5;
        const uint64_t sv = sb0 + (uint64_t)c * kMmaKc + q;
        const bool in = sv < sb1;
        const double sd = (double)sv;
        const double s2 = f_mulmod(sd, sd, f);
        double s16 = s2;
WV_UNROLL
        for (int i = 0; i < 3; i++) s16 = f_mulmod(s16, s16, f);   // s^16
        const double h = f_mulmod(s16, s16, f);                    // s^32
        const double step = fpow_e(h, CT, f);                      // s^(2N)
        double step8 = step;
WV_UNROLL
        for (int i = 0; i < 3; i++) step8 = f_mulmod(step8, step8, f);   // s^(16N)
        const double h16 = f_mulmod(step8, step8, f);                   // s^(32N)
        double h128 = h16;
WV_UNROLL
        for (int i = 0; i < 3; i++) h128 = f_mulmod(h128, h128, f);   // s^(256N)
        // s^(t0) s^(256N rb) s^(32N g) = s^(t0 + 2N (m0 + 16 g))
        const double base = f_mulmod(fpow_e(h128, rb, f), fpow_e(sd, T.t0, f), f);
        double xa0 = f_mulmod(base, fpow_lt8(h16, (uint32_t)g, f), f);
        double xa1 = f_mulmod(xa0, step8, f);
        double xb0 = fpow_lt8(h, (uint32_t)g, f);                      // s^(32g)
        double xb1 = f_mulmod(xb0, s16, f);
WV_UNROLL
        for (int r = 0; r < 8; r++) {
            A[(16 * g + r) * kMmaAs + q] = in ? xa0 : 0.0;
            A[(16 * g + 8 + r) * kMmaAs + q] = in ? xa1 : 0.0;
            Bt[(16 * g + r) * kMmaAs + q] = in ? xb0 : 0.0;
            Bt[(16 * g + 8 + r) * kMmaAs + q] = in ? xb1 : 0.0;
            xa0 = f_mulmod(xa0, step, f);
            xa1 = f_mulmod(xa1, step, f);
            xb0 = f_mulmod(xb0, s2, f);
            xb1 = f_mulmod(xb1, s2, f);
        }
    };

    const bool live = !producer && m0 + 16 * wave < M;   // wave-uniform
    v4d acc[8];
WV_UNROLL
    for (int n = 0; n < CT; n++) acc[n] = v4d{0.0, 0.0, 0.0, 0.0};
    if (producer) produce(0);
    __syncthreads();
    for (uint32_t c = 0; c < nchunk; c++) {
        if (producer) {
            if (c + 1 < nchunk) produce(c + 1);
        } else if (live) {
            mma_chunk<CT>(As[c & 1], Bs[c & 1], wave, lane, acc);
            if (c % period == period - 1) {
WV_UNROLL
                for (int n = 0; n < CT; n++)
WV_UNROLL
                    for (int r = 0; r < 4; r++) acc[n][r] = f_reduce(acc[n][r], f);
            }
        }
        __syncthreads();
    }
    if (!live) return;
    // element r of lane l of a 16 x 16 tile is row l / 16 + 4 r, column l % 16
WV_UNROLL
    for (int n = 0; n < CT; n++) {
WV_UNROLL
        for (int r = 0; r < 4; r++) {
            const uint32_t m = m0 + 16 * wave + (lane >> 4) + 4 * r;
            const uint64_t e = (uint64_t)N * m + 16 * n + (lane & 15);
            if (m < M && e < T.nt) {
                const double v = f_reduce(acc[n][r], f);
                atomicAdd(&V[T.out + e], T.neg ? -v : v);
            }
        }
    }
}

__global__ void __launch_bounds__(kMmaThreads) k_irr_mma(const IrrTask *__restrict__ tasks,
                                                         const uint64_t *__restrict__ unit_off, uint32_t ntask,
                                                         uint64_t nunits, uint64_t unit_base, double *__restrict__ V) {
    __shared__ double As[2][kMmaRows * kMmaAs];
    __shared__ double Bs[2][kMmaRows * kMmaAs];
    const uint64_t unit = unit_base + blockIdx.x;
    if (unit >= nunits) return;   // whole workgroup
    const uint32_t j = find_seg(unit_off, ntask, unit);
    const IrrTask T = tasks[j];
    Fmod f;
    f.p = (double)T.p;
    f.pinv = 1.0 / f.p;
    const uint32_t N = 16 * T.ct;   // exponents per row
    const uint32_t M = (T.nt + N - 1) / N;
    const uint32_t rbs = (M + kMmaRows - 1) / kMmaRows;
    const uint64_t u = unit - unit_off[j];
    const uint32_t rb = (uint32_t)(u % rbs);
    const uint64_t sb0 = T.lo + (u / rbs) * kMmaSb;
    const uint64_t sb1 = min(T.hi, sb0 + kMmaSb);
    // chunks whose products (each below 0.33 p^2) add up to at most 2^52
    const double chunk_bound = 0.33 * f.p * f.p * kMmaKc;
    const uint32_t period = (uint32_t)fmax(1.0, fmin((double)kMmaReduceMax, floor(4503599627370496.0 / chunk_bound)));
    switch (T.ct) {   // workgroup-uniform
        case 1: irr_mma_unit<1>(T, f, period, rb, M, sb0, sb1, As, Bs, V); break;
        case 2: irr_mma_unit<2>(T, f, period, rb, M, sb0, sb1, As, Bs, V); break;
        case 3: irr_mma_unit<3>(T, f, period, rb, M, sb0, sb1, As, Bs, V); break;
        case 4: irr_mma_unit<4>(T, f, period, rb, M, sb0, sb1, As, Bs, V); break;
        case 5: irr_mma_unit<5>(T, f, period, rb, M, sb0, sb1, As, Bs, V); break;
        case 6: irr_mma_unit<6>(T, f, period, rb, M, sb0, sb1, As, Bs, V); break;
        case 7: irr_mma_unit<7>(T, f, period, rb, M, sb0, sb1, As, Bs, V); break;
        default: irr_mma_unit<8>(T, f, period, rb, M, sb0, sb1, As, Bs, V); break;
    }
}

// ---------------------------------------------------------------------------
// power sums for all exponents as one discrete Fourier transform
// ---------------------------------------------------------------------------
//
// With g a primitive root of p, w = g^2 (of order h = (p - 1) / 2) and s_j the
// one of +-g^j in (0, p/2), s_j^2 = w^j, so over any set of s below p/2
//   sum c(s) s^(2k)   = sum_j c(s_j) w^(jk),
//   sum c(s) s^(2k-1) = sum_j c(s_j) s_j^-1 w^(jk):
// both sides' totals for every k are a transform of length h over F_p.  With
// T(n) = n (n - 1) / 2, jk = T(j + k) - T(j) - T(k), so (Bluestein's method)
//   V_k = w^-T(k) sum_j [c_j w^-T(j)] w^T(j+k),
// a correlation, done in blocks of M = L/2 inputs and outputs by the exact
// transforms of ntt.hpp: output block b = sum over input blocks a of (y_a)
// correlated with the 2 M chirp values from (a + b) M on.  One modulus where h
// products below 0.33 p^2 stay below q/2 (p < 2^16), else two.
// About 450 p operations per prime near 2^15 and 1250 p near 3e5, instead of the
// p^2 / 8 multiply-adds of the power sums taken one by one: a window of 390
// primes near 2^15 takes 0.90 ms (4.8 ms by the matrix cores), one prime near
// 2e5 0.46 ms (0.73 ms; more than half of it the copy of its residues).

struct IrrNtt {
    uint64_t p, vb, ve;   // the prime and its totals V
    uint64_t h;
};

// What the primes of one launch share: A blocks of M = L/2 values.  Prime i's
// sequences: chirp 2 A M, inverse chirp A M, the sides' y A M each; its vectors
// of L: 2 A - 1 chirp segments, A blocks of each side, then A output blocks of
// each side, each with nq moduli.
struct IrrShape {
    uint32_t n, A, M, nq;
    __host__ __device__ uint64_t seq_len() const { return 5ull * A * M; }
    __host__ __device__ uint64_t fwd() const { return 4ull * A - 1; }
    __host__ __device__ uint64_t vecs() const { return 6ull * A - 1; }
    __host__ __device__ uint64_t seq_units() const;
};

constexpr uint64_t kIrrOneQ = 1ull << 16;   // one modulus below this
constexpr int kSeqRun = 32;                 // sequence entries per lane

__host__ __device__ inline uint64_t IrrShape::seq_units() const { return (2ull * A * M + 64 * kSeqRun - 1) / (64 * kSeqRun); }

// A primitive root of each prime (one wave each): the least g >= 2 with
// g^((p-1)/r) != 1 for every prime r | p - 1, eight g at a time (numbers below
// 2^27 have at most eight prime factors).
__global__ void __launch_bounds__(64) k_irr_root(const IrrNtt *__restrict__ pr, double *__restrict__ root) {
    const uint32_t lane = threadIdx.x;
    const uint64_t p = readfirst_u64(pr[blockIdx.x].p);
    const uint32_t m = (uint32_t)(p - 1);
    const Fmod f = fmod_of(p);
    uint32_t rest = m, nr = 0, mine = 1;   // mine: prime factor number lane % 8 (1: none)
    for (uint32_t d0 = 2; (uint64_t)d0 * d0 <= rest; d0 += 64) {
        for (;;) {
            const uint64_t hit = __ballot(rest % (d0 + lane) == 0 && d0 + lane <= rest);
            if (!hit) break;
            const uint32_t r = d0 + (uint32_t)__builtin_ctzll(hit);   // smaller primes are gone: a prime
            if ((lane & 7) == nr) mine = r;
            nr++;
            while (rest % r == 0) rest /= r;
        }
    }
    if (rest > 1 && (lane & 7) == nr) mine = rest;
    for (uint32_t g0 = 2; g0 < (1u << 16); g0 += 8) {   // least primitive roots here are far smaller
        const uint32_t g = g0 + (lane >> 3);
        const bool one = g % p == 0 || (mine > 1 && f_canon(fpow_e((double)(g % p), m / mine, f), f) == 1);
        const uint64_t bad = __ballot(one);
        int k = 0;
        while (k < 8 && ((bad >> (8 * k)) & 0xff)) k++;
        if (k < 8) {
            if (lane == 0) root[blockIdx.x] = (double)(g0 + k);
            break;
        }
    }
}

// The sequences of every prime; a wave takes 64 kSeqRun consecutive n of [0, 2 A
// M) of one prime, stepping each of g^n, g^-n, w^T(n), w^-T(n) by 64 n at a
// time: T(n + 64) - T(n) = 64 n + 2016.
__global__ void __launch_bounds__(256) k_irr_seq(const IrrNtt *__restrict__ pr, IrrShape sh,
                                                 const double *__restrict__ root, double *__restrict__ seq) {
    const uint64_t unit = readfirst_u64((uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6));
    const uint32_t i = (uint32_t)(unit / sh.seq_units());
    if (i >= sh.n) return;
    const int lane = threadIdx.x & 63;
    const IrrNtt P = pr[i];
    const uint64_t p = P.p, m = p - 1, h = P.h;
    const Fmod f = fmod_of(p);
    const uint64_t AM = (uint64_t)sh.A * sh.M;
    double *e = seq + i * sh.seq_len(), *ei = e + 2 * AM, *yb = ei + AM, *ye = yb + AM;
    const double g = root[i], gi = f_pow_u(g, p - 2, f);
    // uniform steps: g^64, g^-64, and w^(64 64) = g^8192
    auto sq = [&](double a, int n) {
        for (int k = 0; k < n; k++) a = f_mulmod(a, a, f);
        return a;
    };
    const double g64 = sq(g, 6), gi64 = sq(gi, 6), d2 = sq(g64, 7), di2 = sq(gi64, 7);
    const double c0 = f_mulmod(sq(g64, 6), gi64, f);      // g^4032 = g^4096 g^-64
    const double ci0 = f_mulmod(sq(gi64, 6), g64, f);
    uint64_t n = unit % sh.seq_units() * (64 * kSeqRun) + lane;
    const uint64_t t2 = (n % m) * ((n + m - 1) % m) % m;                 // 2 T(n) mod p - 1 (products below 2^54)
    double G = fpow_e(g, n % m, f), Gi = fpow_e(gi, n % m, f);
    double x = fpow_e(g, t2, f), xi = fpow_e(gi, t2, f);
    double d = f_mulmod(sq(G, 7), c0, f), di = f_mulmod(sq(Gi, 7), ci0, f);   // w^(64 n + 2016) = g^(128 n + 4032)
    uint64_t b0, b1, e0, e1, z0, z1;
    open_range(p, 1, 4, 1, 3, b0, b1);
    open_range(p, 0, 1, 1, 12, e0, e1);
    open_range(p, 5, 12, 1, 2, z0, z1);
    for (int r = 0; r < kSeqRun && n < 2 * AM; r++, n += 64) {
        e[n] = x;
        if (n < AM) {
            ei[n] = xi;
            double vb = 0.0, ve = 0.0;
            if (n < h) {
                uint64_t s = f_canon(G, f);
                const bool up = s > h;
                if (up) s = p - s;
                if (s >= b0 && s < b1) {
                    vb = f_mulmod(Gi, xi, f);      // s^-1 = +-g^-n
                    if (up) vb = -vb;
                }
                ve = s >= e0 && s < e1 ? xi : (s >= z0 && s < z1 ? -xi : 0.0);
            }
            yb[n] = vb;
            ye[n] = ve;
        }
        G = f_mulmod(G, g64, f);
        Gi = f_mulmod(Gi, gi64, f);
        x = f_mulmod(x, d, f);
        xi = f_mulmod(xi, di, f);
        d = f_mulmod(d, d2, f);
        di = f_mulmod(di, di2, f);
    }
}

// Transforms of every chirp segment and every input block (a workgroup per
// prime, vector and modulus): segment sigma holds entry sigma M + i - 1 at i >=
// 1, block a its M values in reverse, so that output M + t of their product is
// sum_j y_j chirp[(a + b) M + j + t].
template <int LOGL>
__global__ void __launch_bounds__(NttShape<LOGL>::T, 4) k_irr_fwd(IrrShape sh, const double *__restrict__ seq,
                                                                  const double *__restrict__ tab,
                                                                  double *__restrict__ hat) {
    using S = NttShape<LOGL>;
    constexpr int E = S::E, T = S::T, L = S::L, M = L / 2;
    __shared__ NttLds<LOGL> lds;
    const int tid = threadIdx.x;
    const uint32_t A = sh.A, per = (uint32_t)sh.fwd() * sh.nq, i = blockIdx.x / per;
    const uint32_t v = blockIdx.x - i * per, q = v % sh.nq, vec = v / sh.nq;
    const Fmod f = ntt_mod(q);
    const VecBuf tb = vec_buf(tab, 2 * S::STRIDE);
    double x[E];
    const double *base = seq + i * sh.seq_len();
    if (vec < 2 * A - 1) {
        const VecBuf b = vec_buf(base + (uint64_t)vec * M, L);
WV_UNROLL
        for (int e = 0; e < E; e++) {
            const bool first = e == 0 && tid == 0;
            x[e] = e ? vec_load(b, tid, e * T - 1) : vec_load(b, first ? 0 : tid - 1, 0);
            if (first) x[e] = 0.0;
        }
    } else {
        const uint64_t AM = (uint64_t)A * M;   // after the chirp (2 A M) and its inverse (A M): the sides' blocks
        const VecBuf b = vec_buf(base + 3 * AM + (uint64_t)(vec - (2 * A - 1)) * M, M);
WV_UNROLL
        for (int e = 0; e < E / 2; e++) x[e] = vec_load(b, T - 1 - tid, M - T - T * e);
WV_UNROLL
        for (int e = E / 2; e < E; e++) x[e] = 0.0;
    }
    ntt_lds_tables<LOGL>(lds, tb, (int)q, tid);
    ntt_forward<LOGL>(x, lds, tb, (int)q, f, tid);
    const double li = -(f.p - 1.0) / (double)L;   // 1 / L mod q
    const VecBuf o = vec_buf(hat + (i * sh.vecs() * sh.nq + v) * L, L);
    if (vec >= 2 * A - 1) {
WV_UNROLL
        for (int m = 0; m < E; m++) vec_store(o, tid, m * T, f_mulmod(x[m], li, f));
    } else {
WV_UNROLL
        for (int m = 0; m < E; m++) vec_store(o, tid, m * T, f_reduce(x[m], f));
    }
}

// The products in the transform domain: a thread takes one position of one
// prime, modulus and BT consecutive output blocks of both sides, the chirp
// values in a window of BT registers, so that a step over the A input blocks
// loads three values for 2 BT products.  With the products in the workgroup of
// the transform back instead (two loads each), a window of 390 primes near 2^15
// took 393 us where this (at 4.5 TB/s, bound by memory) and the transforms back take
// 163 + 130 us; for one prime near 2e5 15 + 30 us instead of 120.
template <int BT>
__global__ void __launch_bounds__(256) k_irr_mul(IrrShape sh, int logl, double *__restrict__ hat) {
    const uint32_t L = 1u << logl, A = sh.A, nt = (A + BT - 1) / BT, chunks = L / 256;
    uint32_t u = blockIdx.x;
    const uint32_t at = (u % chunks) * 256 + threadIdx.x;
    u /= chunks;
    const uint32_t tile = u % nt;
    u /= nt;
    const uint32_t q = u % sh.nq, i = u / sh.nq;
    const uint32_t b0 = tile * BT;
    const Fmod f = ntt_mod((int)q);
    const uint64_t step = (uint64_t)sh.nq * L;                            // from one vector to the next
    const double *w = hat + (i * sh.vecs() * sh.nq + q) * L + at, *y = w + (2 * A - 1) * step;
    double win[BT], acc[2][BT];
WV_UNROLL
    for (int j = 0; j < BT; j++) {
        win[j] = j + 1 < BT && b0 + j < 2 * A - 1 ? w[(b0 + j) * step] : 0.0;
        acc[0][j] = acc[1][j] = 0.0;
    }
    for (uint32_t a0 = 0; a0 < A; a0 += BT) {
WV_UNROLL
        for (int r = 0; r < BT; r++) {
            const uint32_t a = a0 + r;
            if (a >= A) break;
            const uint32_t s = a + b0 + BT - 1;   // the last tile may reach past the segments
            win[(r + BT - 1) % BT] = s < 2 * A - 1 ? w[s * step] : 0.0;
            const double y0 = y[a * step], y1 = y[(A + a) * step];
WV_UNROLL
            for (int j = 0; j < BT; j++) {
                acc[0][j] += f_mulmod(y0, win[(r + j) % BT], f);   // each below 0.52 q in magnitude
                acc[1][j] += f_mulmod(y1, win[(r + j) % BT], f);
            }
        }
WV_UNROLL
        for (int j = 0; j < BT; j++) {
            acc[0][j] = f_reduce(acc[0][j], f);
            acc[1][j] = f_reduce(acc[1][j], f);
        }
    }
    double *o = hat + ((i * sh.vecs() + 4 * A - 1) * sh.nq + q) * L + at;
WV_UNROLL
    for (int j = 0; j < BT; j++) {
        if (b0 + j >= A) break;
        o[(b0 + j) * step] = acc[0][j];
        o[(A + b0 + j) * step] = acc[1][j];
    }
}

// One output block of one side (a workgroup each): brought back, taken mod p
// and multiplied by w^-T(k): V[k - 1] for 1 <= k < h.
template <int LOGL>
__global__ void __launch_bounds__(NttShape<LOGL>::T, 4) k_irr_out(const IrrNtt *__restrict__ pr, IrrShape sh,
                                                                  const double *__restrict__ seq,
                                                                  const double *__restrict__ hat,
                                                                  const double *__restrict__ tab, double *__restrict__ V) {
    using S = NttShape<LOGL>;
    constexpr int E = S::E, T = S::T, L = S::L, M = L / 2;
    __shared__ NttLds<LOGL> lds;
    const int tid = threadIdx.x;
    const uint32_t A = sh.A, i = blockIdx.x / (2 * A), v = blockIdx.x - i * 2 * A, side = v / A, blk = v - side * A;
    const int nq = (int)sh.nq;
    const uint64_t h = readfirst_u64(pr[i].h), vo = readfirst_u64(side ? pr[i].ve : pr[i].vb);
    const Fmod fp = fmod_of(readfirst_u64(pr[i].p));
    const double q1p = f_reduce((double)kNttQ[0], fp);
    const VecBuf tb = vec_buf(tab, 2 * S::STRIDE);
    // outputs k = k0 + t with 1 <= k < h
    const uint64_t k0 = (uint64_t)blk * M;
    const uint32_t live = (uint32_t)min((uint64_t)M, h > k0 ? h - k0 : 0);   // t < live
    double *out = V + vo + k0;                                               // entry t - 1
    const VecBuf ei = vec_buf(seq + i * sh.seq_len() + 2 * (uint64_t)A * M + k0, M);
WV_NO_UNROLL
    for (int q = 0; q < nq; q++) {
        const Fmod f = ntt_mod(q);
        double x[E], t1[E];
        load_vec<LOGL>(x, hat + ((i * sh.vecs() + 4 * A - 1 + v) * nq + q) * L, tid);
        if (q) __syncthreads();   // the last pass may still read the twiddles
        ntt_lds_tables<LOGL>(lds, tb, q, tid);
        __syncthreads();
        twiddle1_load<LOGL>(t1, tb, ntt_inverse_tw1<LOGL>(q), tid);
        ntt_inverse<LOGL>(x, t1, lds, q, f, tid);
WV_UNROLL
        for (int e = 0; e < E / 2; e++) {
            const uint32_t t = tid + T * e;
            if (t >= live || k0 + t == 0) continue;
            double *o = out + t - 1;
            if (nq == 2 && q == 0) {
                *o = f_reduce(x[E / 2 + e], f);
            } else {
                const double r = nq == 2 ? ntt_crt(*o, x[E / 2 + e], kNttQ1Inv, q1p, f, fp)
                                         : f_reduce(f_reduce(x[E / 2 + e], f), fp);
                *o = f_mulmod(r, vec_load(ei, tid, T * e), fp);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// residues from the totals
// ---------------------------------------------------------------------------

// b = B_{2k} mod p from (2,3,4) unless its C_k vanishes (then queued for
// k_irr_fix), e = E_{2k} mod p from eqnEMac2 unless its left side vanishes (then
// queued for k_irr_fix_e).  Counters: [0] queued Bernoulli indices, [1] pairs,
// [2] unresolved, [3] queued Euler indices.  Zero residues are appended to
// pairs as (p, 2k, kind).
//
// A wave takes 64 R consecutive k of one prime, a lane every 64th of them: the
// powers of 2, 3 and 16 are stepped, and with OUT (the residues themselves are
// wanted) one Fermat inverse serves the lane's 2 R left sides, about 10 products
// an index instead of 70 with its own powers and 130 with its own inverses.
// Bound by the serial steps: 16 indices a lane take 48 us over the 390 primes of
// a window near 2^15, 32 take 59 us (half the waves).  The indices of one prime that
// hardly fill the chip go one to a lane (with eight / with one: p = 5003 18 / 7 us,
// 300007 22 / 15, 1000003 23 / 34).
template <bool OUT, int R>
__global__ void __launch_bounds__(256) k_irr_final(const IrrPrime *__restrict__ pr, const uint64_t *__restrict__ off,
                                                   uint32_t np, const double *__restrict__ V,
                                                   uint64_t *__restrict__ b_out, uint64_t *__restrict__ e_out,
                                                   IrrFix *__restrict__ fix, IrrFix *__restrict__ fix_e,
                                                   unsigned long long *__restrict__ counts,
                                                   wv_irr_pair *__restrict__ pairs, uint64_t pair_cap) {
    const uint64_t unit = readfirst_u64((uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6));
    if (unit >= off[np]) return;
    const uint32_t i = __builtin_amdgcn_readfirstlane(find_seg(off, np, unit));
    const IrrPrime P = pr[i];
    const uint64_t p = P.p;
    const Fmod f = fmod_of(p);
    const uint64_t k1 = (unit - off[i]) * (64 * R) + (threadIdx.x & 63) + 1;
    auto sq = [&](double a, int n) {
        for (int k = 0; k < n; k++) a = f_mulmod(a, a, f);
        return a;
    };
    // steps of 64 in k
    double s2 = 0.0, s3 = 0.0, s3i = 0.0, s16 = 0.0;
    if constexpr (R > 1) {
        s2 = sq((double)((p + 1) / 2), 7);
        s3 = sq(3.0, 7);
        s3i = sq(f_pow_u(3.0, p - 2, f), 7);
        s16 = sq(16.0, 6);
    }
    double x = 0.0, y = 0.0, z = 0.0, p4 = 0.0;
    if (k1 <= P.nt) {
        x = fpow_e(2.0, p - 2 * k1, f);
        y = fpow_e(3.0, p - 2 * k1, f);
        z = fpow_e(3.0, 2 * k1, f);
        if (OUT) p4 = f_mulmod(4.0, fpow_e(16.0, k1, f), f);   // 4^(t+1) = 4 16^k
    }
    auto pair = [&](uint64_t k, uint32_t kind) {
        const unsigned long long at = atomicAdd(&counts[1], 1ull);
        if (at < pair_cap) pairs[at] = wv_irr_pair{p, (uint32_t)(2 * k), kind};
    };
    double c[R], w[R], pe[R];
    constexpr int kUnroll = OUT ? R : 1;
#pragma unroll kUnroll
    for (int r = 0; r < R; r++) {
        const uint64_t k = k1 + 64 * r;
        c[r] = w[r] = 1.0;
        pe[r] = 0.0;
        if (k <= P.nt) {
            // Bernoulli side: odd exponent t = 2k - 1; with x = 2^(p-2k),
            // 4k C_k(2,3,4) = x + 3^(p-2k) - x^2 - 1 =: c and B_{2k} = S 4k / c
            const double cc = (double)f_canon(f_reduce(x + y - f_mulmod(x, x, f) - 1.0, f), f);
            if (cc == 0.0) fix[atomicAdd(&counts[0], 1ull)] = IrrFix{i, (uint32_t)k};
            else if (f_canon(V[P.vb + k - 1], f) == 0) pair(k, 1u);
            // Euler side: even exponent t = 2k, left-side index k' = (p - 1 -
            // t) / 2.  eqnEMac2: (-1)^k' 4^(k'-1) (9^k' + 1) E_t == 2^t T, T =
            // S_t(0, 1/12) - S_t(5/12, 1/2) (the totals); by Fermat 4^(k'-1) =
            // 2^(-2-t) and 9^k' = 3^(-t), so E_t = (-1)^k' 4^(t+1) 3^t T /
            // (3^t + 1), queued for eqnE1 where 3^t == -1.
            const double ww = (double)f_canon(z + 1.0, f);
            if (ww == 0.0) fix_e[atomicAdd(&counts[3], 1ull)] = IrrFix{i, (uint32_t)k};
            else if (f_canon(V[P.ve + k - 1], f) == 0) pair(k, 2u);
            if (OUT) {
                c[r] = cc;
                w[r] = ww;
                pe[r] = f_mulmod(p4, z, f);
            }
        }
        if constexpr (R > 1) {
            x = f_mulmod(x, s2, f);
            y = f_mulmod(y, s3i, f);
            z = f_mulmod(z, s3, f);
            if (OUT) p4 = f_mulmod(p4, s16, f);
        }
    }
    if constexpr (OUT) {
        double pre[2 * R], acc = 1.0;
WV_UNROLL
        for (int r = 0; r < R; r++) {
            pre[2 * r] = acc;
            if (c[r] != 0.0) acc = f_mulmod(acc, c[r], f);
            pre[2 * r + 1] = acc;
            if (w[r] != 0.0) acc = f_mulmod(acc, w[r], f);
        }
        double inv = f_pow_u(acc, p - 2, f);
WV_UNROLL
        for (int r = R - 1; r >= 0; r--) {
            const uint64_t k = k1 + 64 * r;
            const double wi = f_mulmod(inv, pre[2 * r + 1], f);
            if (w[r] != 0.0) inv = f_mulmod(inv, w[r], f);
            const double ci = f_mulmod(inv, pre[2 * r], f);
            if (c[r] != 0.0) inv = f_mulmod(inv, c[r], f);
            if (k > P.nt) continue;
            if (c[r] != 0.0) {
                const double s4k = f_mulmod((double)f_canon(V[P.vb + k - 1], f), (double)((4 * k) % p), f);
                b_out[P.res + k - 1] = f_canon(f_mulmod(s4k, ci, f), f);
            }
            if (w[r] != 0.0) {
                const double num = f_mulmod((double)f_canon(V[P.ve + k - 1], f), pe[r], f);
                uint64_t e = f_canon(f_mulmod(num, wi, f), f);
                if ((((p - 1 - 2 * k) / 2) & 1) && e) e = p - e;
                e_out[P.res + k - 1] = e;
            }
        }
    }
}

// The queued indices, evaluated directly (one power per s):
//   Euler side, eqnE1: (-1)^k' 4^(2k'-1) E_t == S_t(0, 1/4) with t = 2k and k' =
//   (p - 1 - t) / 2; 4^-(2k'-1) = 4^(t+1) by Fermat;
//   Bernoulli side, the next members of the family (2, b, b + 1) of Section 2
//   (C_k(2,b,b+1) B_{2k} == sum_{m=1}^{floor(b/2)} S_{2k-1}(m/(b+1), m/b); b = 5
//   is eqnVandiver) for b = 4, 5, ..., kIrrMaxB with p not dividing b (b + 1).
//   At 2k = (p+1)/2 every C_k is a sum of Legendre symbols, and the first b with
//   (b/p) != ((b+1)/p) (or b = 3 when (2/p) = -1) resolves it.  A k where all of
//   them degenerate is marked with the residue UINT64_MAX and counted in
//   counts[2].
//
// An index is shared by up to 16 workgroups, as many as fill the chip, with four
// powers in flight per lane; the one that finishes last turns the total into the
// residue.  One index of p = 299993 is 2.7 million products, 120 us in one
// workgroup and 1.2 ms in one wave; shared, the kernel takes 17 us, and the 700
// or so queued indices of a window near 2^15 64 us (0.42 ms with a wave each).
constexpr uint64_t kIrrMaxB = 64;
static_assert(kIrrMaxB - 4 < 64, "one candidate b per lane");
constexpr int kFixThreads = 512;
constexpr uint64_t kFixGrid = 1024;       // workgroups: the chip twice over
constexpr uint64_t kIrrOneFin = 1u << 19; // one prime below: an index a lane in k_irr_final
constexpr uint64_t kFixShared = kFixGrid / 2;   // queue lengths up to here are shared; a total and a ticket each
constexpr uint64_t kFixMaxShare = 16;
constexpr uint64_t kFixWords = 4 + 2 * kFixShared;   // the counters, totals and tickets

// this thread's part of sum s^t, lo <= s < hi, threads numbered from first, of
// all.  Exact: fewer than p terms below 0.574 p in magnitude.
__device__ inline double pow_sum_part(uint64_t lo, uint64_t hi, uint64_t t, uint64_t first, uint64_t all, const Fmod &f) {
    double acc = 0.0;
    for (uint64_t s = lo + first; s < hi; s += 4 * all) {
        double a[4], r[4];
WV_UNROLL
        for (int q = 0; q < 4; q++) {
            const uint64_t sq = s + q * all;
            a[q] = sq < hi ? (double)sq : 0.0;   // t >= 1: adds 0
            r[q] = 1.0;
        }
        for (uint64_t e = t; e; e >>= 1) {
            if (e & 1) {
WV_UNROLL
                for (int q = 0; q < 4; q++) r[q] = f_mulmod(r[q], a[q], f);
            }
WV_UNROLL
            for (int q = 0; q < 4; q++) a[q] = f_mulmod(a[q], a[q], f);
        }
        acc += (r[0] + r[1]) + (r[2] + r[3]);
    }
    return acc;
}

__global__ void __launch_bounds__(kFixThreads) k_irr_fix(const IrrPrime *__restrict__ pr, const IrrFix *__restrict__ fix_b,
                                                         const IrrFix *__restrict__ fix_e,
                                                         unsigned long long *__restrict__ counts,
                                                         uint64_t *__restrict__ b_out, uint64_t *__restrict__ e_out,
                                                         wv_irr_pair *__restrict__ pairs, uint64_t pair_cap) {
    __shared__ double part[kFixThreads / 64];
    const uint64_t nb = readfirst_u64(counts[0]), n = nb + readfirst_u64(counts[3]);
    if (n == 0) return;
    const uint64_t share = n <= kFixShared ? min(kFixMaxShare, kFixGrid / n) : 1;
    double *total = reinterpret_cast<double *>(counts + 4);
    unsigned long long *ticket = counts + 4 + kFixShared;
    const int lane = threadIdx.x & 63;
    for (uint64_t w = blockIdx.x; w < n * share; w += gridDim.x) {
        const uint64_t at = w / share, first = w % share * kFixThreads + threadIdx.x, all = share * kFixThreads;
        const bool euler = at >= nb;
        const IrrFix F = euler ? fix_e[at - nb] : fix_b[at];
        const IrrPrime P = pr[F.prime];
        const uint64_t p = readfirst_u64(P.p), k = readfirst_u64((uint64_t)F.k);
        const Fmod f = fmod_of(p);
        uint64_t lo, hi, c = 0;
        double acc = 0.0;
        if (euler) {
            open_range(p, 0, 1, 1, 4, lo, hi);
            acc = pow_sum_part(lo, hi, 2 * k, first, all, f);
        } else {
            const uint64_t cand = 4 + lane;
            uint64_t mine = 0;
            if (cand <= kIrrMaxB && cand % p != 0 && (cand + 1) % p != 0) mine = c_k(2, cand, cand + 1, k, f, p);
            const uint64_t ok = __ballot(mine != 0);
            if (ok) {
                const int l = __builtin_ctzll(ok);
                const uint64_t bb = 4 + l;
                c = __shfl(mine, l, 64);
                for (uint64_t m = 1; m <= bb / 2; m++) {
                    open_range(p, m, bb + 1, m, bb, lo, hi);
                    acc += pow_sum_part(lo, hi, 2 * k - 1, first, all, f);   // the intervals hold fewer than p s together
                }
            }
        }
        for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
        __syncthreads();   // the previous index's part
        if (lane == 0) part[threadIdx.x >> 6] = acc;
        __syncthreads();
        if (threadIdx.x) continue;
        acc = 0.0;
        for (int q = 0; q < kFixThreads / 64; q++) acc += part[q];
        if (share > 1) {   // integers below 2^53: exact in any order
            atomicAdd(&total[at], acc);
            __threadfence();
            if (atomicAdd(&ticket[at], 1ull) != share - 1) continue;
            __threadfence();
            acc = atomicAdd(&total[at], 0.0);
        }
        const double S = (double)f_canon(f_reduce(acc, f), f);
        uint64_t r;
        if (euler) {
            r = f_canon(f_mulmod(S, f_mulmod(4.0, fpow_e(16.0, k, f), f), f), f);
            if ((((p - 1 - 2 * k) / 2) & 1) && r) r = p - r;
            if (e_out) e_out[P.res + k - 1] = r;
        } else {
            r = c ? f_canon(f_mulmod(S, (double)u_pow(c, p - 2, f), f), f) : UINT64_MAX;
            if (b_out) b_out[P.res + k - 1] = r;
            if (!c) atomicAdd(&counts[2], 1ull);
        }
        if (r == 0) {
            const unsigned long long to = atomicAdd(&counts[1], 1ull);
            if (to < pair_cap) pairs[to] = wv_irr_pair{p, (uint32_t)(2 * k), euler ? 2u : 1u};
        }
    }
}

__global__ void k_irr_zero(double *__restrict__ v, uint64_t n) {
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) v[i] = 0.0;
}

unsigned grid_for(uint64_t n, unsigned per) { return (unsigned)((n + per - 1) / per + (n == 0)); }

constexpr uint64_t kMaxWgs = 1ull << 22;   // bound on a launch's workgroups of up to 1024 threads
constexpr double kDftMul = 16.0;       // a product and its share of the loads, in the units of a transform's value

// Blocks of L/2 = 2^(logl - 1) values a transform of length h is cut into, and
// the length of the least modelled work: 6 A - 1 transforms and 2 A^2 products
// per position.
uint32_t dft_blocks(uint64_t h, int logl) { return (uint32_t)((h + (1ull << (logl - 1)) - 1) >> (logl - 1)); }

// Modelled work of one prime's transforms: 6 A - 1 of them and the products of
// its blocks, per modulus.
double dft_work(uint32_t blocks, int logl, uint32_t nq) {
    const double A = blocks, L = (double)(1ull << logl);
    return nq * L * ((6.0 * A - 1.0) * (14.0 + 2.6 * logl) + 2.0 * A * A * kDftMul);
}

int dft_logl(uint64_t h) {
    int best = kNttMaxLog;
    double best_w = 1e300;
    for (int l = kNttMinLog; l <= kNttMaxLog; l++) {
        const double w = dft_work(dft_blocks(h, l), l, 1);
        if (w < best_w) best_w = w, best = l;
    }
    return best;
}

// The totals V of every prime by the transform, enqueued in groups of one shape
// (length, blocks, moduli), each within the workspace bound.  Primes are
// ascending; the smaller ones join the shape of the larger while that costs less
// than a group's launches (about 40 us; 1.5e13 modelled units a second), which is most
// of the time of windows of small primes: [100, 8292) each in its own shape 0.83
// ms, joined 0.67 ([500, 4596) 0.56 and 0.35).  keep: the host data of the queued copies, until the stream is
// waited for.
constexpr double kDftGroup = 6e8;
constexpr double kDftSquares = 2.5e7;
struct DftGroup {
    size_t begin, end;
    int logl;
    uint32_t A, nq;
};

std::vector<DftGroup> dft_groups(const std::vector<IrrPrime> &prs) {
    std::vector<DftGroup> out;
    size_t end = prs.size();
    uint64_t last_k = 0;
    int last_l = 0;
    while (end > 0) {
        auto shape = [&](size_t i) {
            // every block is a multiple of 256 values: so are the ends of the shapes' ranges
            const uint64_t k = ((prs[i].p - 1) / 2 + 255) / 256;
            if (k != last_k) {
                last_k = k;
                last_l = dft_logl(256 * k);
            }
            return DftGroup{i, end, last_l, dft_blocks(256 * k, last_l), prs[i].p < kIrrOneQ ? 1u : 2u};
        };
        DftGroup g = shape(end - 1);
        const double mine = dft_work(g.A, g.logl, g.nq);
        while (g.begin > 0) {
            // the run of one shape before the group
            const DftGroup o = shape(g.begin - 1);
            size_t i = g.begin - 1;
            while (i > 0) {
                const DftGroup q = shape(i - 1);
                if (q.logl != o.logl || q.A != o.A || q.nq != o.nq) break;
                i--;
            }
            const bool same = o.logl == g.logl && o.A == g.A && o.nq == g.nq;
            if (!same && (mine - dft_work(o.A, o.logl, o.nq)) * (double)(g.begin - i) > kDftGroup) break;
            g.begin = i;
        }
        out.push_back(g);
        end = g.begin;
    }
    return out;
}

constexpr uint64_t kDftDoubles = 1ull << 30;   // sequences and transforms held at once (8 GiB), unless one prime needs more

int irr_dft(wv_ctx *c, const std::vector<IrrPrime> &prs, std::vector<std::vector<IrrNtt>> &keep) {
    hipStream_t st = c->stream;
    const std::vector<DftGroup> groups = dft_groups(prs);
    size_t i = groups.empty() ? 0 : groups[0].begin;
    uint64_t held = kDftDoubles;
    for (size_t k = 0; k < groups.size();) {
        const DftGroup &gr = groups[k];
        const int logl = gr.logl;
        const uint64_t L = 1ull << logl;
        IrrShape sh{0, gr.A, (uint32_t)(L / 2), gr.nq};
        const uint64_t each = sh.seq_len() + sh.vecs() * sh.nq * L, wgs = sh.vecs() * sh.nq * std::max<uint64_t>(L / 256, 4);
        // as many primes as the bound allows, or what the device has left
        for (;;) {
            const uint64_t most = std::max<uint64_t>(1, std::min(held / each, kMaxWgs / wgs));
            sh.n = (uint32_t)std::min<uint64_t>(most, gr.end - i);
            int rc = ensure(c, c->irr_seq, sh.n * sh.seq_len() * sizeof(double));
            if (rc == WV_OK) rc = ensure(c, c->irr_hat, sh.n * sh.vecs() * sh.nq * L * sizeof(double));
            if (rc == WV_OK) break;
            if (rc != WV_ENOMEM || sh.n == 1) return rc;
            held = sh.n / 2 * each;
        }
        keep.emplace_back();
        std::vector<IrrNtt> &g = keep.back();
        for (; g.size() < sh.n; i++) g.push_back(IrrNtt{prs[i].p, prs[i].vb, prs[i].ve, (prs[i].p - 1) / 2});
        if (i == gr.end && ++k < groups.size()) i = groups[k].begin;   // gr's shape is in sh
        WV_TRY(ntt_tables(c, logl));
        WV_TRY(ensure(c, c->irr_dft, g.size() * sizeof(IrrNtt)));
        WV_TRY(ensure(c, c->irr_root, g.size() * sizeof(double)));
        WV_HIP(hipMemcpyAsync(c->irr_dft.ptr, g.data(), g.size() * sizeof(IrrNtt), hipMemcpyHostToDevice, st));
        const IrrNtt *pr = as<IrrNtt>(c->irr_dft);
        double *seq = as<double>(c->irr_seq), *hat = as<double>(c->irr_hat);
        hipLaunchKernelGGL(k_irr_root, dim3(sh.n), dim3(64), 0, st, pr, as<double>(c->irr_root));
        hipLaunchKernelGGL(k_irr_seq, dim3(grid_for(sh.n * sh.seq_units(), 4)), dim3(256), 0, st, pr, sh,
                           as<double>(c->irr_root), seq);
        WV_TRY(with_shape(logl, [&](auto s) -> int {
            constexpr int LG = decltype(s)::value;
            hipLaunchKernelGGL(k_irr_fwd<LG>, dim3((unsigned)(sh.n * sh.fwd() * sh.nq)), dim3(NttShape<LG>::T), 0, st, sh,
                               seq, as<double>(c->ntt_tab[LG]), hat);
            // output blocks per thread: of a step over the input blocks, 2 products each and 3 loads
            uint32_t bt = 5;
            auto cost = [&](uint32_t k) { return (sh.A + k - 1) / k * (2 * k + 6); };
            for (uint32_t k = 4; k >= 1; k--)
                if (cost(k) < cost(bt)) bt = k;
            const dim3 mg((unsigned)((uint64_t)sh.n * sh.nq * ((sh.A + bt - 1) / bt) * (L / 256)));
            auto mul = bt == 5   ? k_irr_mul<5>
                       : bt == 4 ? k_irr_mul<4>
                       : bt == 3 ? k_irr_mul<3>
                       : bt == 2 ? k_irr_mul<2>
                                 : k_irr_mul<1>;
            hipLaunchKernelGGL(mul, mg, dim3(256), 0, st, sh, logl, hat);
            hipLaunchKernelGGL(k_irr_out<LG>, dim3(sh.n * 2 * sh.A), dim3(NttShape<LG>::T), 0, st, pr, sh, seq, hat,
                               as<double>(c->ntt_tab[LG]), as<double>(c->irr_v));
            return WV_OK;
        }));
        WV_HIP(hipGetLastError());
    }
    return WV_OK;
}

// One batch of primes (all in [5, WV_IRR_P_MAX)): with b and e (host arrays), the
// residues of every index, prime by prime; else zero pairs appended to the device
// list and the counters {fixups, pairs, unresolved}.
int irr_batch(wv_ctx *c, const std::vector<uint64_t> &ps, uint64_t *b, uint64_t *e, uint64_t pair_cap,
              uint64_t counts_out[3], float *ms_sum, double *pairs_done, bool transforms = true) {
    hipStream_t st = c->stream;
    uint64_t *d_b = b ? as<uint64_t>(c->irr_b) : nullptr, *d_e = b ? as<uint64_t>(c->irr_e) : nullptr;
    std::vector<IrrTask> tasks;
    std::vector<uint64_t> units(1, 0);
    std::vector<IrrPrime> prs;
    std::vector<uint64_t> roff(1, 0);
    uint64_t vn = 0, res = 0;
    double work = 0.0;
    // indices per lane of k_irr_final
    const uint64_t kFin = !d_b ? 16 : ps.size() == 1 && ps[0] < kIrrOneFin ? 1 : 8;
    // Path 0: transforms, but the matrix cores for a batch of so little work that the
    // launches count (p^2 summed over the batch; one prime near 3000 130 us by the
    // matrix cores, 139 by transforms, near 5000 both 140, near 8000 167 and 149).
    // Path 2: the matrix cores while every partial sum stays exact.
    double squares = 0.0;
    for (uint64_t p : ps) squares += (double)p * (double)p;
    const bool dft = c->irr_path == 0 && transforms && squares >= kDftSquares;
    const bool mma = c->irr_path != 1 && !dft && *std::max_element(ps.begin(), ps.end()) < kIrrMmaMaxP;
    // exponents per row 16 ct: the least work over whole row blocks, each row
    // costing its N multiply-adds per s plus about 8 for building its A entry
    // (one modular product), ties to wider rows
    auto cols_of = [](uint64_t nt) -> uint32_t {
        uint32_t best = 8;
        uint64_t best_w = UINT64_MAX;
        for (uint32_t ct = 8; ct >= 1; ct--) {
            const uint64_t N = 16 * ct, M = (nt + N - 1) / N;
            const uint64_t w = (M + kMmaRows - 1) / kMmaRows * kMmaRows * (N + 8);
            if (w < best_w) best_w = w, best = ct;
        }
        return best;
    };
    auto units_of = [&](uint64_t lo, uint64_t hi, uint64_t nt) -> uint64_t {
        if (mma) {
            const uint64_t N = 16 * cols_of(nt), M = (nt + N - 1) / N;
            return (M + kMmaRows - 1) / kMmaRows * ((hi - lo + kMmaSb - 1) / kMmaSb);
        }
        return (hi - lo + kIrrWaveS - 1) / kIrrWaveS * ((nt + kIrrUnitT - 1) / kIrrUnitT);
    };
    std::vector<std::vector<IrrNtt>> keep;
    auto task = [&](IrrTask t) {
        if (dft) return;
        t.ct = cols_of(t.nt);
        tasks.push_back(t);
        units.push_back(units.back() + units_of(t.lo, t.hi, t.nt));
    };
    for (uint64_t p : ps) {
        const uint32_t nt = (uint32_t)((p - 3) / 2);
        IrrPrime P{p, vn, vn + nt, res, nt, 0};
        uint64_t lo, hi;
        open_range(p, 1, 4, 1, 3, lo, hi);   // Bernoulli: (1/4, 1/3), odd exponents from 1
        task(IrrTask{p, lo, hi, vn, 1, nt, 0, 0});   // Bernoulli: +S(1/4, 1/3)
        work += (double)(hi - lo) * nt;
        // Euler (eqnEMac2): S(0, 1/12) - S(5/12, 1/2) into the same totals,
        // even exponents from 2
        open_range(p, 0, 1, 1, 12, lo, hi);
        task(IrrTask{p, lo, hi, vn + nt, 2, nt, 0, 0});
        work += (double)(hi - lo) * nt;
        open_range(p, 5, 12, 1, 2, lo, hi);
        task(IrrTask{p, lo, hi, vn + nt, 2, nt, 0, 1});
        work += (double)(hi - lo) * nt;
        vn += 2 * (uint64_t)nt;
        res += nt;
        prs.push_back(P);
        roff.push_back(roff.back() + (nt + 64 * kFin - 1) / (64 * kFin));
    }
    const uint64_t nunits = units.back();
    const uint32_t ntask = (uint32_t)tasks.size(), np = (uint32_t)prs.size();
    WV_TRY(ensure(c, c->irr_primes, prs.size() * sizeof(IrrPrime)));
    WV_TRY(ensure(c, c->irr_roff, roff.size() * sizeof(uint64_t)));
    WV_TRY(ensure(c, c->irr_v, std::max<uint64_t>(vn, 1) * sizeof(double)));
    WV_TRY(ensure(c, c->irr_fix, 2 * std::max<uint64_t>(res, 1) * sizeof(IrrFix)));   // both sides' queues
    WV_TRY(ensure(c, c->irr_counts, kFixWords * sizeof(unsigned long long)));
    WV_HIP(hipMemcpyAsync(c->irr_primes.ptr, prs.data(), prs.size() * sizeof(IrrPrime), hipMemcpyHostToDevice, st));
    WV_HIP(hipMemcpyAsync(c->irr_roff.ptr, roff.data(), roff.size() * sizeof(uint64_t), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_irr_zero, dim3(grid_for(kFixWords, 256)), dim3(256), 0, st, as<double>(c->irr_counts), kFixWords);
    if (!dft) {
        WV_TRY(ensure(c, c->irr_tasks, tasks.size() * sizeof(IrrTask)));
        WV_TRY(ensure(c, c->irr_units, units.size() * sizeof(uint64_t)));
        WV_HIP(hipMemcpyAsync(c->irr_tasks.ptr, tasks.data(), tasks.size() * sizeof(IrrTask), hipMemcpyHostToDevice,
                              st));
        WV_HIP(hipMemcpyAsync(c->irr_units.ptr, units.data(), units.size() * sizeof(uint64_t), hipMemcpyHostToDevice,
                              st));
        hipLaunchKernelGGL(k_irr_zero, dim3(grid_for(vn, 256)), dim3(256), 0, st, as<double>(c->irr_v), vn);
    }
    WV_HIP(hipEventRecord(c->ev[EV_SUM0], st));
    if (dft) {
        const int rc = irr_dft(c, prs, keep);
        if (rc == WV_ENOMEM) {
            // a prime's transforms (120 bytes times p) need more than there is: the
            // power sums, which need a tenth of that
            WV_HIP(hipStreamSynchronize(st));
            for (DevBuf *x : {&c->irr_seq, &c->irr_hat}) {
                if (x->ptr) WV_HIP(hipFree(x->ptr));
                *x = DevBuf{};
            }
            return irr_batch(c, ps, b, e, pair_cap, counts_out, ms_sum, pairs_done, false);
        }
        WV_TRY(rc);
    } else if (mma) {
        // one workgroup per unit, in launches of fewer than 2^32 work-items
        for (uint64_t u0 = 0; u0 < nunits; u0 += kMmaMaxGrid) {
            const uint64_t g = std::min<uint64_t>(kMmaMaxGrid, nunits - u0);
            hipLaunchKernelGGL(k_irr_mma, dim3((unsigned)g), dim3(kMmaThreads), 0, st, as<IrrTask>(c->irr_tasks),
                               as<uint64_t>(c->irr_units), ntask, nunits, u0, as<double>(c->irr_v));
        }
    } else {
        hipLaunchKernelGGL(k_irr_sum, dim3(grid_for(nunits, 4)), dim3(256), 0, st, as<IrrTask>(c->irr_tasks),
                           as<uint64_t>(c->irr_units), ntask, nunits, as<double>(c->irr_v));
    }
    WV_HIP(hipGetLastError());
    WV_HIP(hipEventRecord(c->ev[EV_SUM], st));
    auto *counts = as<unsigned long long>(c->irr_counts);
    IrrFix *fix_b = as<IrrFix>(c->irr_fix), *fix_e = fix_b + std::max<uint64_t>(res, 1);
    const unsigned fgrid = grid_for(roff.back(), 4);
    hipLaunchKernelGGL((kFin == 16  ? k_irr_final<false, 16>
                        : kFin == 8 ? k_irr_final<true, 8>
                                    : k_irr_final<true, 1>),
                       dim3(fgrid), dim3(256), 0, st, as<IrrPrime>(c->irr_primes), as<uint64_t>(c->irr_roff), np,
                       as<double>(c->irr_v), d_b, d_e, fix_b, fix_e, counts, as<wv_irr_pair>(c->irr_pairs), pair_cap);
    WV_HIP(hipGetLastError());
    // the queues' lengths stay on the device: a fixed grid goes through them
    hipLaunchKernelGGL(k_irr_fix, dim3((unsigned)kFixGrid), dim3(kFixThreads), 0, st, as<IrrPrime>(c->irr_primes), fix_b,
                       fix_e, counts, d_b, d_e, as<wv_irr_pair>(c->irr_pairs), pair_cap);
    WV_HIP(hipGetLastError());
    if (b) {
        WV_TRY(words_to_host(c, d_b, b, d_e, e, res));   // waits
    } else {
        unsigned long long host[4];
        WV_HIP(hipMemcpyAsync(host, counts, sizeof(host), hipMemcpyDeviceToHost, st));
        WV_HIP(hipStreamSynchronize(st));
        for (int q = 0; q < 3; q++) counts_out[q] = host[q];
    }
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, c->ev[EV_SUM0], c->ev[EV_SUM]);
    *ms_sum += ms;
    *pairs_done += work;
    return WV_OK;
}

// Batches of consecutive primes within the device budgets.
template <class F>
int irr_for_batches(const std::vector<uint64_t> &ps, F &&run) {
    size_t i = 0;
    while (i < ps.size()) {
        std::vector<uint64_t> b;
        uint64_t vn = 0, units = 0;
        while (i < ps.size()) {
            const uint64_t p = ps[i];
            const uint64_t v = p - 3;   // two totals per k
            // three tasks of at most p/12 s each (a bound for either kernel's units)
            const uint64_t u = 3 * (p / 12 / kIrrWaveS + 2) * ((p / 2) / kIrrUnitT + 1);
            if (!b.empty() && (vn + v > kIrrMaxV || units + u > kIrrMaxUnits)) break;
            b.push_back(p);
            vn += v;
            units += u;
            i++;
        }
        WV_TRY(run(b));
    }
    return WV_OK;
}

}  // namespace
}  // namespace wv

using namespace wv;

int wv_set_irregular_path(wv_ctx *c, int path) {
    if (!c || path < 0 || path > 2) return WV_EINVAL;
    c->irr_path = path;
    return WV_OK;
}

int wv_bernoulli_euler_all(wv_ctx *c, uint64_t p, uint64_t *b, uint64_t *e) {
    if (!c || !b || !e) return WV_EINVAL;
    if (p < 5 || p >= WV_IRR_P_MAX) return WV_EDOMAIN;
    if (!is_prime_u64(p)) return WV_ENOTPRIME;
    WV_TRY(check_device(c));
    c->stats = wv_stats{};
    const uint64_t nt = (p - 3) / 2;
    WV_TRY(ensure(c, c->irr_b, nt * sizeof(uint64_t)));
    WV_TRY(ensure(c, c->irr_e, nt * sizeof(uint64_t)));
    WV_TRY(ensure(c, c->irr_pairs, 64 * sizeof(wv_irr_pair)));
    float ms = 0.f;
    double work = 0.0;
    WV_TRY(irr_batch(c, std::vector<uint64_t>{p}, b, e, 0, nullptr, &ms, &work));
    c->stats.n_primes = 1;
    c->stats.n_terms = (uint64_t)work;
    c->stats.ms_sum = ms;
    return WV_OK;
}

int wv_irregular_pairs(wv_ctx *c, uint64_t lo, uint64_t hi, wv_irr_pair *out, size_t cap, size_t *n_out,
                       uint64_t *n_primes, uint64_t *n_unresolved) {
    if (!c || !n_out || lo > hi || (cap && !out)) return WV_EINVAL;
    if (hi > WV_IRR_P_MAX) return WV_EDOMAIN;
    WV_TRY(check_device(c));
    c->stats = wv_stats{};
    *n_out = 0;
    // the primes of [lo, hi), sieved on the device in groups of segments
    std::vector<SegDesc> d;
    window_descs(lo, hi, d);
    std::vector<uint64_t> ps;
    for (size_t g = 0; g < d.size(); g += kMaxBatchSegs) {
        const size_t ns = std::min(kMaxBatchSegs, d.size() - g);
        std::vector<uint32_t> counts(ns);
        WV_TRY(sieve_count(c, d.data() + g, ns, true, counts.data()));
        uint64_t np = 0;
        WV_TRY(compact(c, d.data() + g, ns, counts.data(), &np));
        const size_t at = ps.size();
        ps.resize(at + np);
        if (np) {
            WV_HIP(hipMemcpyAsync(ps.data() + at, c->primes.ptr, np * sizeof(uint64_t), hipMemcpyDeviceToHost,
                                  c->stream));
            WV_HIP(hipStreamSynchronize(c->stream));
        }
    }
    std::vector<wv_irr_pair> all;
    uint64_t unresolved = 0;
    float ms = 0.f;
    double work = 0.0;
    const uint64_t pair_cap = 1ull << 20;
    WV_TRY(ensure(c, c->irr_pairs, pair_cap * sizeof(wv_irr_pair)));
    WV_TRY(irr_for_batches(ps, [&](const std::vector<uint64_t> &b) -> int {
        uint64_t counts[3];
        WV_TRY(irr_batch(c, b, nullptr, nullptr, pair_cap, counts, &ms, &work));
        if (counts[1] > pair_cap) return WV_ENOMEM;
        const size_t at = all.size();
        all.resize(at + counts[1]);
        if (counts[1]) {
            WV_HIP(hipMemcpyAsync(all.data() + at, c->irr_pairs.ptr, counts[1] * sizeof(wv_irr_pair),
                                  hipMemcpyDeviceToHost, c->stream));
            WV_HIP(hipStreamSynchronize(c->stream));
        }
        unresolved += counts[2];
        return WV_OK;
    }));
    std::sort(all.begin(), all.end(), [](const wv_irr_pair &a, const wv_irr_pair &b) {
        return a.p != b.p ? a.p < b.p : (a.two_k != b.two_k ? a.two_k < b.two_k : a.kind < b.kind);
    });
    c->stats.n_primes = ps.size();
    c->stats.n_terms = (uint64_t)work;
    c->stats.ms_sum = ms;
    if (n_primes) *n_primes = ps.size();
    if (n_unresolved) *n_unresolved = unresolved;
    *n_out = all.size();
    if (all.size() > cap) return WV_ETRUNC;
    std::copy(all.begin(), all.end(), out);
    return WV_OK;
}
