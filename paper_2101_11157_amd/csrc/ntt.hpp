// ntt.hpp -- exact convolutions mod p on a workgroup: number-theoretic
// transforms modulo two primes q below 2^47 in the exact double-precision
// products of sum_core.hpp, the whole vector held in the workgroup's vector
// registers and exchanged through LDS.
//
// A cyclic convolution of length L = 2^LOGL of residues |u|, |b| < 0.574 p, at
// most 2^13 of them nonzero in u, is an integer below 0.33 p^2 2^13 < 2^91.5
// for p < 2^40; q1 q2 = 2^93.5, so its residues mod q1 and q2 give it exactly
// (ntt_crt) and it is reduced mod p from there.
//
// Shape.  T = L / E threads hold E values each (E = 16, 8 at the shortest);
// passes of radix E and a last one of what is left (16, 16, 16, 4 at L =
// 2^14).  Only the first exchange crosses waves.  Forward (decimation in frequency,
// natural order in, an order of its own out) and inverse (the mirror image)
// are only ever paired with each other, so nothing is put in bit-reversed
// order: the transform domain's layout is (register m, thread).
//
// Bounds (q = 2^46.75).  Every value is reduced between passes, by its twiddle
// product or, where the twiddle is 1, by f_reduce: |x| <= r q entering a pass.
// A radix-16 pass at most doubles per level, so |x| <= 16 r q inside and after
// it.  A product by a twiddle (|w| <= q/2) of x with |x| <= M q leaves at most
// (1/2 + M/2 * 2^-5.25) q, so r = 1/2 + 0.21 r, r < 0.64 and |x| < 10.3 q <
// 2^50.2: an exact integer, and |x w| / q < 2^49.2 is inside f_mulmod's range
// (2^51).
#pragma once
#include <cstdint>
#include <type_traits>

#include "sum_core.hpp"

namespace wv {

constexpr int kNttMinLog = 9, kNttMaxLog = 14;
constexpr uint64_t kNttQ[2] = {118345648832513ull, 118345640181761ull};       // == 1 mod 2^17
constexpr uint64_t kNttRoot[2] = {40319942354732ull, 13109796054582ull};      // of order 2^17
constexpr double kNttQ1Inv = -3586245201047.0;                                 // 1 / q1 mod q2, balanced

template <int LOGL>
struct NttShape {
    static constexpr int L = 1 << LOGL;
    static constexpr int LE = LOGL >= 10 ? 4 : 3;
    static constexpr int E = 1 << LE;             // values per thread
    static constexpr int T = L / E;               // threads
    static constexpr int P = LOGL / LE;           // passes of radix E
    static constexpr int R = 1 << (LOGL % LE);    // radix of the last pass (1: none)
    static constexpr int NT = R > 1 ? P : P - 1;  // inter-pass products
    static constexpr int N(int k) { return L >> (LE * k); }   // length after k passes
    // Tables of one modulus (doubles): inter-pass twiddles 1 .. NT, forward then inverse
    static constexpr int table(int k) {           // start of product k's table (k = NT + 1: size of one direction)
        int at = 0;
        for (int i = 1; i < k; i++) at += N(i - 1);
        return at;
    }
    static constexpr int DIR = table(NT + 1), STRIDE = 2 * DIR;
    // LDS position of element i, one pad per E doubles
    static constexpr int at(int i) { return i + (i >> LE); }
    static constexpr int LDS = L + L / E;         // doubles
};

#if defined(__HIPCC__)

// Powers 0 .. 15 of the 32nd root (kNttRoot^4096), balanced, of modulus q at
// row 2 q and of its inverse at row 2 q + 1: constant memory, so that the
// butterflies read them as scalar operands.
__constant__ double kNttRt[4][16] = {
    {1.0, 58544850336196.0, -44176785110119.0, -49111024221253.0, 15015527830968.0, 47910580647752.0,
     -23442931498315.0, 13558510082084.0, -40119262814941.0, -24608988036415.0, 8642893906784.0,
     -55485761914718.0, -46990119939955.0, -18776382491109.0, 32086972574082.0, 53471972864453.0},
    {1.0, -53471972864453.0, -32086972574082.0, 18776382491109.0, 46990119939955.0, 55485761914718.0,
     -8642893906784.0, 24608988036415.0, 40119262814941.0, -13558510082084.0, 23442931498315.0,
     -47910580647752.0, -15015527830968.0, 49111024221253.0, 44176785110119.0, -58544850336196.0},
    {1.0, -34132951168211.0, 48187060380898.0, -34035946235150.0, -26264991430509.0, 53883104814865.0,
     50919257347632.0, -8712651700733.0, 10232154488834.0, 6299334923269.0, 16276727124048.0,
     43388640257468.0, 24500645441877.0, -10537916538005.0, -46354058269123.0, -20598792386782.0},
    {1.0, 20598792386782.0, 46354058269123.0, 10537916538005.0, -24500645441877.0, -43388640257468.0,
     -16276727124048.0, -6299334923269.0, -10232154488834.0, 8712651700733.0, -50919257347632.0,
     -53883104814865.0, 26264991430509.0, 34035946235150.0, -48187060380898.0, 34132951168211.0}};

__device__ __forceinline__ Fmod ntt_mod(int q) {
    Fmod f;
    f.p = q == 0 ? (double)kNttQ[0] : (double)kNttQ[1];
    f.pinv = q == 0 ? 1.0 / (double)kNttQ[0] : 1.0 / (double)kNttQ[1];
    return f;
}

// A vector of doubles at a wave-uniform address, read and written as element
// i + k with i per lane and k the same for the whole wave: buffer instructions
// take k as a scalar offset, so the 32 accesses of a thread share one address
// register (flat addresses T doubles apart each need their own).
struct VecBuf {
    __amdgpu_buffer_rsrc_t r;
};

typedef unsigned v2u __attribute__((ext_vector_type(2)));

__device__ __forceinline__ VecBuf vec_buf(const double *base, uint32_t n) {
    return VecBuf{__builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(base), 0, (int)(n * 8), 0x00020000)};
}

__device__ __forceinline__ double vec_load(const VecBuf &b, int i, int k) {
    const v2u v = __builtin_amdgcn_raw_buffer_load_b64(b.r, i * 8, k * 8, 0);
    return __builtin_bit_cast(double, v);
}

__device__ __forceinline__ void vec_store(const VecBuf &b, int i, int k, double x) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, x), b.r, i * 8, k * 8, 0);
}

// The same for values read once and too late to be kept in the caches
// (non-temporal).
constexpr int kAuxStream = 2;

__device__ __forceinline__ double vec_load_stream(const VecBuf &b, int i, int k) {
    const v2u v = __builtin_amdgcn_raw_buffer_load_b64(b.r, i * 8, k * 8, kAuxStream);
    return __builtin_bit_cast(double, v);
}

__device__ __forceinline__ void vec_store_stream(const VecBuf &b, int i, int k, double x) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, x), b.r, i * 8, k * 8, kAuxStream);
}

// LDS writes of a wave become visible to the wave's other lanes (LDS
// operations of one wave complete in order; this keeps the compiler to it).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int ilog2(int v) { return v <= 1 ? 0 : 1 + ilog2(v / 2); }

// r[i] = a[i] b[i] mod q, N products in step (f_mulmod's six operations, each
// for all N before the next).  The scheduler orders independent products one
// after another to save registers, so that every operation waits for the one
// before it; the barriers keep them interleaved.
template <int N>
__device__ __forceinline__ void mulmod_step(double (&r)[N], const double (&a)[N], const double (&b)[N], const Fmod &f) {
    double h[N], l[N], k[N];
WV_UNROLL
    for (int i = 0; i < N; i++) h[i] = a[i] * b[i];
    __builtin_amdgcn_sched_barrier(0);
WV_UNROLL
    for (int i = 0; i < N; i++) k[i] = fma(h[i], f.pinv, kRound);
    __builtin_amdgcn_sched_barrier(0);
WV_UNROLL
    for (int i = 0; i < N; i++) l[i] = fma(a[i], b[i], -h[i]);
    __builtin_amdgcn_sched_barrier(0);
WV_UNROLL
    for (int i = 0; i < N; i++) k[i] = k[i] - kRound;
    __builtin_amdgcn_sched_barrier(0);
WV_UNROLL
    for (int i = 0; i < N; i++) h[i] = fma(-k[i], f.p, h[i]);
    __builtin_amdgcn_sched_barrier(0);
WV_UNROLL
    for (int i = 0; i < N; i++) r[i] = h[i] + l[i];
    __builtin_amdgcn_sched_barrier(0);
}

// x[i] <- x[i] t[i] for i in [A, B), N at a time
template <int N, int A, int B, int E>
__device__ __forceinline__ void mulmod_range(double (&x)[E], const double (&t)[E], const Fmod &f) {
    static_assert((B - A) % N == 0, "whole groups");
WV_UNROLL
    for (int i = A; i < B; i += N) {
        double a[N], b[N];
WV_UNROLL
        for (int k = 0; k < N; k++) a[k] = x[i + k], b[k] = t[i + k];
        mulmod_step<N>(a, a, b, f);
WV_UNROLL
        for (int k = 0; k < N; k++) x[i + k] = a[k];
    }
}

constexpr int kNttGroup = 4;   // butterflies in step

// Radix-R transforms of x[0 .. R), x[R .. 2 R), ..., decimation in frequency:
// natural order in, slot i holds frequency bitrev(i).  rt: powers of the 32nd
// root.
template <int R, int E>
__device__ __forceinline__ void ntt_dif(double (&x)[E], const double *rt, const Fmod &f) {
    constexpr int LR = ilog2(R), G = kNttGroup;
WV_UNROLL
    for (int s = 0; s < LR; s++) {
        const int len = R >> (s + 1);
WV_UNROLL
        for (int k0 = 0; k0 < E / 2; k0 += G) {
            double d[G], w[G];
WV_UNROLL
            for (int g = 0; g < G; g++) {
                const int k = k0 + g, j = k & (len - 1), i = ((k - j) << 1) + j;
                const double a = x[i], b = x[i + len];
                x[i] = a + b;
                d[g] = a - b;
                w[g] = rt[j * (16 / len)];
            }
            __builtin_amdgcn_sched_barrier(0);
            if (len > 1) {
                // the trivial root (j = 0) keeps its difference
                double keep = d[0];
                if (G > len) {
                    // groups that hold several j = 0 (len < G)
                    double r[G];
WV_UNROLL
                    for (int g = 0; g < G; g++) r[g] = d[g];
                    double a2[G / 2], w2[G / 2];
WV_UNROLL
                    for (int g = 0; g < G / 2; g++) a2[g] = d[2 * g + 1], w2[g] = w[2 * g + 1];
                    mulmod_step<G / 2>(a2, a2, w2, f);
WV_UNROLL
                    for (int g = 0; g < G / 2; g++) r[2 * g + 1] = a2[g];
WV_UNROLL
                    for (int g = 0; g < G; g++) d[g] = r[g];
                } else if ((k0 & (len - 1)) == 0) {
                    double a3[G - 1], w3[G - 1];
WV_UNROLL
                    for (int g = 1; g < G; g++) a3[g - 1] = d[g], w3[g - 1] = w[g];
                    mulmod_step<G - 1>(a3, a3, w3, f);
WV_UNROLL
                    for (int g = 1; g < G; g++) d[g] = a3[g - 1];
                    d[0] = keep;
                } else {
                    mulmod_step<G>(d, d, w, f);
                }
            }
WV_UNROLL
            for (int g = 0; g < G; g++) {
                const int k = k0 + g, j = k & (len - 1), i = ((k - j) << 1) + j;
                x[i + len] = d[g];
            }
        }
    }
}

// Their inverses times R (decimation in time); rt: powers of the inverse root.
template <int R, int E>
__device__ __forceinline__ void ntt_dit(double (&x)[E], const double *rt, const Fmod &f) {
    constexpr int LR = ilog2(R), G = kNttGroup;
WV_UNROLL
    for (int s = LR - 1; s >= 0; s--) {
        const int len = R >> (s + 1);
WV_UNROLL
        for (int k0 = 0; k0 < E / 2; k0 += G) {
            double d[G], w[G];
WV_UNROLL
            for (int g = 0; g < G; g++) {
                const int k = k0 + g, j = k & (len - 1), i = ((k - j) << 1) + j;
                d[g] = x[i + len];
                w[g] = rt[j * (16 / len)];
            }
            if (len > 1) {
                if (G > len) {
                    double a2[G / 2], w2[G / 2];
WV_UNROLL
                    for (int g = 0; g < G / 2; g++) a2[g] = d[2 * g + 1], w2[g] = w[2 * g + 1];
                    mulmod_step<G / 2>(a2, a2, w2, f);
WV_UNROLL
                    for (int g = 0; g < G / 2; g++) d[2 * g + 1] = a2[g];
                } else if ((k0 & (len - 1)) == 0) {
                    double a3[G - 1], w3[G - 1];
WV_UNROLL
                    for (int g = 1; g < G; g++) a3[g - 1] = d[g], w3[g - 1] = w[g];
                    mulmod_step<G - 1>(a3, a3, w3, f);
WV_UNROLL
                    for (int g = 1; g < G; g++) d[g] = a3[g - 1];
                } else {
                    mulmod_step<G>(d, d, w, f);
                }
            }
WV_UNROLL
            for (int g = 0; g < G; g++) {
                const int k = k0 + g, j = k & (len - 1), i = ((k - j) << 1) + j;
                const double a = x[i];
                x[i] = a + d[g];
                x[i + len] = a - d[g];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Inter-pass twiddles of product 1 (as long as the vector) come from memory,
// register m's at tid + m T; they are the same for every transform of one
// direction, so a kernel that runs several inverse transforms keeps theirs in
// registers.
template <int LOGL>
__device__ __forceinline__ void twiddle1_load(double (&t)[NttShape<LOGL>::E], const VecBuf &tab, int base, int tid) {
    using S = NttShape<LOGL>;
WV_UNROLL
    for (int m = 1; m < S::E; m++) t[m] = vec_load(tab, tid, base + m * S::T);
    __builtin_amdgcn_sched_barrier(0);
}

template <bool NEG, int E>
__device__ __forceinline__ void twiddle1_mul(double (&x)[E], const double (&t)[E], const Fmod &f) {
    constexpr int G = kNttGroup;
    if constexpr (NEG) {
        mulmod_range<G, 0, E>(x, t, f);
        return;
    }
    double a[G - 1], b[G - 1];
    x[0] = f_reduce(x[0], f);   // its twiddle is 1
WV_UNROLL
    for (int k = 1; k < G; k++) a[k - 1] = x[k], b[k - 1] = t[k];
    mulmod_step<G - 1>(a, a, b, f);
WV_UNROLL
    for (int k = 1; k < G; k++) x[k] = a[k - 1];
    mulmod_range<G, G, E>(x, t, f);
}

// NEG: transforms modulo X^L + 1, the cyclic ones of x[n] psi^n, psi of order 2 L.
// n = tid + T e, so psi^n = psi^tid theta^e with theta = psi^T of order 2 E: with E = 16
// theta is the 32nd root of kNttRt, and psi^tid goes into the twiddles of product
// 1 (then not 1 for register 0 either).
template <int E>
__device__ __forceinline__ void theta_mul(double (&x)[E], const double *rt, const Fmod &f) {
    static_assert(E == 16, "theta is the 32nd root");
    double t[E];
WV_UNROLL
    for (int e = 0; e < E; e++) t[e] = rt[e];
    double a[3], b[3];
WV_UNROLL
    for (int e = 1; e < 4; e++) a[e - 1] = x[e], b[e - 1] = t[e];
    mulmod_step<3>(a, a, b, f);
WV_UNROLL
    for (int e = 1; e < 4; e++) x[e] = a[e - 1];
    mulmod_range<4, 4, E>(x, t, f);
}

// product 1's twiddles modulo X^L + 1: both moduli's, forward then inverse, L each
template <int LOGL>
__device__ __forceinline__ void neg_twiddle1_load(double (&t)[NttShape<LOGL>::E], const double *tab, int at, int tid) {
    using S = NttShape<LOGL>;
    const VecBuf b = vec_buf(tab + (size_t)at * S::L, S::L);
WV_UNROLL
    for (int m = 0; m < S::E; m++) t[m] = vec_load(b, tid, m * S::T);
    __builtin_amdgcn_sched_barrier(0);
}

// Those of the later products are short (1088 values at L = 2^14): both
// directions' tables of one modulus are kept in LDS, where one group is read
// while the group before it is multiplied.
template <int E>
__device__ __forceinline__ void twiddle_mul(double (&x)[E], const double *t, int stride, const Fmod &f) {
    constexpr int G = kNttGroup;
    double a[2][G];
WV_UNROLL
    for (int k = 0; k < G; k++) a[0][k] = t[k * stride];
    const double x0 = x[0];
WV_UNROLL
    for (int m = 0; m < E; m += G) {
        const int cur = (m / G) & 1;
        if (m + G < E) {
WV_UNROLL
            for (int k = 0; k < G; k++) a[cur ^ 1][k] = t[(m + G + k) * stride];
        }
        __builtin_amdgcn_sched_barrier(0);
        double b[G];
WV_UNROLL
        for (int k = 0; k < G; k++) b[k] = x[m + k];
        mulmod_step<G>(b, b, a[cur], f);
WV_UNROLL
        for (int k = 0; k < G; k++) x[m + k] = b[k];
    }
    x[0] = f_reduce(x0, f);
}

// The LDS of one workgroup's transforms.
template <int LOGL>
struct NttLds {
    using S = NttShape<LOGL>;
    double v[S::LDS];
    double tw[2 * (S::DIR - S::L) + 2];   // products 2 .. NT, forward then inverse
};

// Loads the tables of modulus q (the caller's next transform starts with a
// barrier that orders these writes before their first use, and the previous
// one's last use lies before a barrier too).
template <int LOGL>
__device__ __forceinline__ void ntt_lds_tables(NttLds<LOGL> &lds, const VecBuf &tab, int q, int tid) {
    using S = NttShape<LOGL>;
    constexpr int n = S::DIR - S::L;
    for (int i = tid; i < n; i += S::T) {
        lds.tw[i] = vec_load(tab, i, q * S::STRIDE + S::L);
        lds.tw[n + i] = vec_load(tab, i, q * S::STRIDE + S::DIR + S::L);
    }
}

// One pad per E doubles (NttShape::at) keeps the exchanges below free of bank
// conflicts at E = 16, and since N(k) is a multiple of E or divides it, the
// pads of each pattern add up per thread and per register: a pattern is one
// address plus constants.
//
// After pass K the thread tid = s N(K) + t holds the values (s, slot i, t), i <
// E, of sub-vector s of length N(K-1): element s N(K-1) + i N(K) + t.  For
// pass K + 1 it holds sub-vector s' = tid / N(K+1) of length N(K), elements t'
// + N(K+1) e; for the last pass, of radix R < E, the E consecutive elements
// tid E + m.  The values of one s stay with its N(K) threads: within a wave
// when N(K) <= 64.
template <int LOGL, int K>
struct NttStep {
    using S = NttShape<LOGL>;
    static constexpr bool WAVE = S::N(K) <= 64;
    static __device__ __forceinline__ double *out_ptr(double *lds, int tid) {
        return lds + (tid / S::N(K)) * S::at(S::N(K - 1)) + S::at(tid % S::N(K));
    }
    static __device__ __forceinline__ double *in_ptr(double *lds, int tid) {
        if constexpr (K < S::P) return lds + (tid / S::N(K + 1)) * S::at(S::N(K)) + S::at(tid % S::N(K + 1));
        else return lds + S::at(tid * S::E);
    }
    static constexpr int out_at(int i) { return S::at(i * S::N(K)); }
    static constexpr int in_at(int e) { return K < S::P ? S::at(e * S::N(K < S::P ? K + 1 : K)) : e; }
};

template <int LOGL, int K, bool NEG = false>
__device__ __forceinline__ void ntt_fwd_from(double (&x)[NttShape<LOGL>::E], NttLds<LOGL> &lds, const VecBuf &tab, int q,
                                             const double *rt, const Fmod &f, int tid, const double *neg = nullptr) {
    using S = NttShape<LOGL>;
    constexpr int E = S::E;
    if constexpr (K == 1) {
        double t[E];
        if constexpr (NEG) {
            theta_mul(x, rt, f);
            neg_twiddle1_load<LOGL>(t, neg, 2 * q, tid);
        } else {
            twiddle1_load<LOGL>(t, tab, q * S::STRIDE, tid);
        }
        ntt_dif<E, E>(x, rt, f);
        twiddle1_mul<NEG>(x, t, f);
    } else {
        ntt_dif<E, E>(x, rt, f);
        if constexpr (K <= S::NT) twiddle_mul(x, lds.tw + (S::table(K) - S::L) + tid % S::N(K), S::N(K), f);
    }
    if constexpr (K <= S::NT) {
        using X = NttStep<LOGL, K>;
        if constexpr (X::WAVE && K > 1) wave_lds_sync();
        else __syncthreads();   // K = 1: LDS still read by other waves
        double *o = X::out_ptr(lds.v, tid), *n = X::in_ptr(lds.v, tid);
WV_UNROLL
        for (int i = 0; i < E; i++) o[X::out_at(i)] = x[i];
        if constexpr (X::WAVE) wave_lds_sync();
        else __syncthreads();
WV_UNROLL
        for (int i = 0; i < E; i++) x[i] = n[X::in_at(i)];
        if constexpr (K < S::P) ntt_fwd_from<LOGL, K + 1>(x, lds, tab, q, rt, f, tid);
        else ntt_dif<S::R, E>(x, rt, f);
    }
}

// x[e] = value tid + T e on entry; the transform in the (register, thread)
// layout on return, unreduced (< 10.3 q).  Two workgroup barriers, the first
// before LDS is written.
template <int LOGL>
__device__ __forceinline__ void ntt_forward(double (&x)[NttShape<LOGL>::E], NttLds<LOGL> &lds, const VecBuf &tab, int q,
                                            const Fmod &f, int tid) {
    ntt_fwd_from<LOGL, 1>(x, lds, tab, q, kNttRt[2 * q], f, tid);
}

// The same modulo X^L + 1; neg: its tables of product 1 (neg_twiddle1_load).
template <int LOGL>
__device__ __forceinline__ void ntt_forward_neg(double (&x)[NttShape<LOGL>::E], NttLds<LOGL> &lds, const VecBuf &tab,
                                                const double *neg, int q, const Fmod &f, int tid) {
    ntt_fwd_from<LOGL, 1, true>(x, lds, tab, q, kNttRt[2 * q], f, tid, neg);
}

// base of the inverse's product 1 for twiddle1_load
template <int LOGL>
__device__ __forceinline__ int ntt_inverse_tw1(int q) {
    return q * NttShape<LOGL>::STRIDE + NttShape<LOGL>::DIR;
}

template <int LOGL, int K, bool NEG = false>
__device__ __forceinline__ void ntt_inv_from(double (&x)[NttShape<LOGL>::E], const double (&t1)[NttShape<LOGL>::E],
                                             NttLds<LOGL> &lds, const double *rt, const Fmod &f, int tid) {
    using S = NttShape<LOGL>;
    constexpr int E = S::E;
    if constexpr (K >= 1) {
        using X = NttStep<LOGL, K>;
        if constexpr (K == S::NT) __syncthreads();   // LDS still read by other waves
        else wave_lds_sync();
        double *o = X::out_ptr(lds.v, tid), *n = X::in_ptr(lds.v, tid);
WV_UNROLL
        for (int i = 0; i < E; i++) n[X::in_at(i)] = x[i];
        if constexpr (X::WAVE) wave_lds_sync();
        else __syncthreads();
WV_UNROLL
        for (int i = 0; i < E; i++) x[i] = o[X::out_at(i)];
        if constexpr (K == 1) twiddle1_mul<NEG>(x, t1, f);
        else twiddle_mul(x, lds.tw + (S::DIR - S::L) + (S::table(K) - S::L) + tid % S::N(K), S::N(K), f);
        ntt_dit<E, E>(x, rt, f);
        if constexpr (K == 1 && NEG) theta_mul(x, rt, f);
        ntt_inv_from<LOGL, K - 1, NEG>(x, t1, lds, rt, f, tid);
    }
}

// The inverse times L: transform layout in, x[e] = value tid + T e out
// (unreduced, < 10.3 q for |x| < 0.7 q in).  Two workgroup barriers, the first
// before LDS is written.
// NEG: modulo X^L + 1, t1 from neg_twiddle1_load.
template <int LOGL, bool NEG = false>
__device__ __forceinline__ void ntt_inverse(double (&x)[NttShape<LOGL>::E], const double (&t1)[NttShape<LOGL>::E],
                                            NttLds<LOGL> &lds, int q, const Fmod &f, int tid) {
    using S = NttShape<LOGL>;
    const double *rt = kNttRt[2 * q + 1];
    if constexpr (S::R > 1) ntt_dit<S::R, S::E>(x, rt, f);
    else ntt_dit<S::E, S::E>(x, rt, f);
    ntt_inv_from<LOGL, S::NT, NEG>(x, t1, lds, rt, f, tid);
}

// A vector of length L, every load requested before the first is used.
template <int LOGL>
__device__ __forceinline__ void load_vec(double (&x)[NttShape<LOGL>::E], const double *base, int tid) {
    using S = NttShape<LOGL>;
    const VecBuf b = vec_buf(base, S::L);
WV_UNROLL
    for (int e = 0; e < S::E; e++) x[e] = vec_load(b, tid, e * S::T);
    __builtin_amdgcn_sched_barrier(0);
}

#endif

// fn(integral_constant<int, logl>) for a compiled length
template <class F>
inline int with_shape(int logl, F &&fn) {
    switch (logl) {
    case 9: return fn(std::integral_constant<int, 9>{});
    case 10: return fn(std::integral_constant<int, 10>{});
    case 11: return fn(std::integral_constant<int, 11>{});
    case 12: return fn(std::integral_constant<int, 12>{});
    case 13: return fn(std::integral_constant<int, 13>{});
    case 14: return fn(std::integral_constant<int, 14>{});
    default: return -1   /* WV_EINVAL */;
    }
}

// The residue mod p (< 0.51 p) of the integer c, |c| <= q1 q2 / 4, given r1 ==
// c (mod q1), |r1| <= 0.51 q1, and r2 == c (mod q2), |r2| <= 10.3 q2: c = r1 +
// q1 t with t = (r2 - r1) / q1 mod q2.  f_mulmod gives |t| < 0.65 q2, and the
// true |t| is below 0.26 q2, so they are equal; t q1 mod p (|t| < 2^46.2, q1
// mod p < 0.51 p: inside f_mulmod's range) plus r1 stays below 2^47.
// q1p = q1 mod p, balanced; q1i = 1 / q1 mod q2, balanced.
__host__ __device__ __forceinline__ double ntt_crt(double r1, double r2, double q1i, double q1p, const Fmod &f2,
                                                   const Fmod &fp) {
    const double t = f_mulmod(r2 - r1, q1i, f2);
    return f_reduce(f_mulmod(t, q1p, fp) + r1, fp);
}

}  // namespace wv
