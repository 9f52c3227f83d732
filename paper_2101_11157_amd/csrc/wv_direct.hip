// wv_direct.hip -- the residues of a batch whose term sums are little work: one
// launch takes the primes to their residues, instead of the plan, chunk
// layout, sums, reduction and finish over (prime, sum) slots, whose launches and
// records cost more than the sums (a call of 16 primes near 2e7 0.46 ms, now
// 0.12; the search of the primes below 1e5 0.62 ms, now 0.18, k_direct 72 us of it
// for 4e7 terms and 9590 stagings and inverses).
//
// The sums of a side, sum_j coef_j sum_s s^-3 or s^-2, are kept as one
// fraction c1 / c0 per lane, coefficients in: a group of four consecutive s, with
// u = s (s + 3) and v = u (u + 2) = s (s+1) (s+2) (s+3), adds
//   s^-2 + ... + (s+3)^-2 = (v (4 u + 14) + 16 u + 36) / v^2,
//   s^-3 + ... + (s+3)^-3 = (2 s + 3) (v (2 v + 10 u + 38) + 40 u + 72) / v^3
// (the pairs s, s + 3 and s + 1, s + 2 of one sum 2 s + 3 each).  Below 2^27 a
// product of two residues in (-p/2, p/2) is exact in double precision and a
// reduction three more operations: 9 operations per s^-2 term and 11 per s^-3
// term, about those of the blocked difference tables of the term-sum kernel; from
// there on 13.5 and 18.5 (f_mulmod).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "sum_core.hpp"
#include "wave_ops.hpp"
#include "wv_ctx.hpp"

namespace wv {
namespace {

constexpr int kDirectSums = 64;    // sums per side a workgroup stages

// Arithmetic mod p: SMALL (p < 2^27): every product below is an integer below
// 2^53, reduced to within p/2 (1 + 2^-24); else f_mulmod.
template <bool SMALL>
struct Dir {
    Fmod f;
    __device__ __forceinline__ double red(double x) const { return fma(-rint(x * f.pinv), f.p, x); }
    __device__ __forceinline__ double mul(double a, double b) const { return SMALL ? red(a * b) : f_mulmod(a, b, f); }
    // a b + y, |y| below 41 p
    __device__ __forceinline__ double mul_add(double a, double b, double y) const {
        if constexpr (SMALL) return red(fma(a, b, y));
        else return f_mulmod(a, b, f) + y;
    }
    // a b + c d, all within p/2
    __device__ __forceinline__ double dot(double a, double b, double c, double d) const {
        if constexpr (SMALL) return red(fma(a, b, c * d));
        else return f_mulmod(a, b, f) + f_mulmod(c, d, f);
    }
    // a small multiple of a residue, before it enters a product
    __device__ __forceinline__ double fit(double a) const { return SMALL ? red(a) : a; }
};

// (c1 / c0) += coef (s^-d + ... + (s+3)^-d), d = 3 or 2
template <int DEG, bool SMALL>
__device__ __forceinline__ void add_four(double s, double coef, double &c0, double &c1, const Dir<SMALL> &m) {
    const double u = m.mul(s, s + 3.0), v = m.mul(u, u + 2.0);
    double N, D;
    if constexpr (DEG == 2) {
        N = m.mul_add(v, m.fit(fma(4.0, u, 14.0)), fma(16.0, u, 36.0));
        D = m.mul(v, v);
    } else {
        const double t = m.mul_add(v, m.fit(fma(2.0, v, fma(10.0, u, 38.0))), fma(40.0, u, 72.0));
        N = m.mul(t, fma(2.0, s, 3.0));
        D = m.mul(m.mul(v, v), v);
    }
    c1 = m.dot(c1, D, m.mul(coef, N), c0);
    c0 = m.mul(c0, D);
}

template <int DEG, bool SMALL>
__device__ __forceinline__ void add_one(double s, double coef, double &c0, double &c1, const Dir<SMALL> &m) {
    double D = m.mul(s, s);
    if constexpr (DEG == 3) D = m.mul(D, s);
    c1 = m.dot(c1, D, coef, c0);
    c0 = m.mul(c0, D);
}

// One side's sums of a prime: first s, number of s, coefficient within p/2, and
// the prefix of the groups of four.
struct Side {
    double lo[kDirectSums], coef[kDirectSums];
    uint64_t base[kDirectSums + 1];
    uint32_t odd[kDirectSums];     // s beyond the groups
    uint64_t terms, lhs;
    int n;
};

// by the lanes of one wave
__device__ __forceinline__ void stage(Side &S, const TableStore &ts, int table, uint64_t p, int lane) {
    const TableHead h = ts.head[table];
    uint64_t len = 0;
    if (lane < h.n) {
        const TableTerm d = ts.term[h.term_off + lane];
        const uint64_t lo = floor_mul_div(d.xa, p, d.xb) + 1, hi = floor_mul_minus1_div(d.ya, p, d.yb);
        len = hi >= lo ? hi - lo + 1 : 0;
        const uint64_t c = limbs_mod(ts.limb, d.limb_off, d.nlimb, d.neg != 0, p);
        S.lo[lane] = (double)lo;
        S.coef[lane] = c > p / 2 ? -(double)(p - c) : (double)c;
        S.odd[lane] = (uint32_t)(len & 3);
    }
    uint64_t inc = len >> 2, all = len;
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t v = __shfl_up((unsigned long long)inc, o, 64);
        if (lane >= o) inc += v;
        all += __shfl_xor((unsigned long long)all, o, 64);
    }
    if (lane < h.n) S.base[lane + 1] = inc;
    if (lane == 0) {
        S.base[0] = 0;
        S.terms = all;
        S.lhs = limbs_mod(ts.limb, h.lhs_off, h.lhs_nlimb, h.lhs_neg != 0, p);
        S.n = h.n;
    }
}

// this lane's share (number t of all) of a side, as c1 / c0
template <int DEG, bool SMALL>
__device__ __forceinline__ void side_part(const Side &S, uint64_t t, uint64_t all, double &c0, double &c1,
                                          const Dir<SMALL> &m) {
    c0 = 1.0;
    c1 = 0.0;
    const int n = S.n;
    using Idx = typename std::conditional<SMALL, uint32_t, uint64_t>::type;
    const Idx groups = (Idx)S.base[n], step = (Idx)all;
    if (groups < 2 * (uint64_t)n * all) {
        // short sums: group after group whatever its sum, so that no lane waits for
        // a sum that others have a part in (primes below 1e5: 72 us, 105 the
        // other way)
        int j = 0;
        Idx end = (Idx)S.base[1];
        double s0 = S.lo[0], coef = S.coef[0];
        for (Idx g = (Idx)t; g < groups; g += step) {
            if (g >= end) {
                do end = (Idx)S.base[++j + 1];
                while (g >= end);
                s0 = fma(-4.0, (double)S.base[j], S.lo[j]);
                coef = S.coef[j];
            }
            add_four<DEG>(fma(4.0, (double)g, s0), coef, c0, c1, m);
        }
    } else {
        const double ds = 4.0 * (double)all;
        Idx g = (Idx)t;
        for (int j = 0; g < groups; j++) {
            const Idx end = (Idx)S.base[j + 1];
            if (g >= end) continue;
            const double coef = S.coef[j];
            double s = fma(4.0, (double)(g - (Idx)S.base[j]), S.lo[j]);
#pragma unroll 2
            for (; g < end; g += step, s += ds) add_four<DEG>(s, coef, c0, c1, m);
        }
    }
    for (uint64_t g = t; g < 3 * (uint64_t)n; g += all) {   // the up to three s beyond each sum's groups
        const int k = (int)(g / 3), r = (int)(g % 3);
        if (r < (int)S.odd[k]) add_one<DEG>(S.lo[k] + 4.0 * (double)(S.base[k + 1] - S.base[k]) + r, S.coef[k], c0, c1, m);
    }
}

// c1 / c0 over the wave, in every lane
template <bool SMALL>
__device__ __forceinline__ void wave_add(double &c0, double &c1, const Dir<SMALL> &m) {
WV_UNROLL
    for (int o = 32; o >= 1; o >>= 1) {
        const double d0 = __shfl_xor(c0, o, 64), d1 = __shfl_xor(c1, o, 64);
        c1 = m.dot(c1, d0, d1, c0);
        c0 = m.mul(c0, d0);
    }
}

// G workgroups per prime (blockIdx.x = prime G + part).  Bound by the vector ALU
// where the batch fills the chip, else by the serial steps: staging, one
// lane's terms, six wave steps and a Fermat inverse.  With G > 1 every
// workgroup leaves its fraction in part and the one that draws the last ticket
// (zeroed before the launch) adds them up.
struct DirectLds {
    Side side[2];
    double red[kDirectWaves][4];
    uint32_t last;
};

template <bool SMALL>
__device__ void direct_prime(DirectLds &lds, const TableStore &ts, const uint64_t *__restrict__ primes, int tb, int te,
                             int fb, int fe, uint32_t i, uint32_t g, uint32_t G, double *part, uint32_t *ticket,
                             uint64_t *__restrict__ terms, wv_result *__restrict__ out) {
    Side(&side)[2] = lds.side;
    double(&red)[kDirectWaves][4] = lds.red;
    uint32_t &last = lds.last;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, W = blockDim.x >> 6;
    const uint64_t p = readfirst_u64(primes[i]);
    if (!(p >= 5 && p < WV_P_MAX && (p & 1))) {
        if (threadIdx.x == 0 && g == 0) {
            out[i] = wv_result{0, 0, 0, 0xFFFFFFFFu, 0};
            if (terms) terms[2 * (size_t)i] = terms[2 * (size_t)i + 1] = 0;
        }
        return;
    }
    const Dir<SMALL> m{fmod_of(p)};
    if (wave == 0) stage(side[0], ts, pick_table(ts, 0, p, tb, fb), p, lane);
    if (wave == W - 1) stage(side[1], ts, pick_table(ts, 1, p, te, fe), p, lane);
    __syncthreads();
    const uint64_t all = (uint64_t)G * blockDim.x, t = (uint64_t)g * blockDim.x + threadIdx.x;
    double b0, b1, e0, e1;
    side_part<3>(side[0], t, all, b0, b1, m);
    side_part<2>(side[1], t, all, e0, e1, m);
    wave_add(b0, b1, m);
    wave_add(e0, e1, m);
    if (W > 1) {
        if (lane == 0) red[wave][0] = b0, red[wave][1] = b1, red[wave][2] = e0, red[wave][3] = e1;
        __syncthreads();
        if (wave != 0) {
            if (G == 1) return;
        } else {
            const bool in = lane < W;
            b0 = in ? red[lane & (kDirectWaves - 1)][0] : 1.0;
            b1 = in ? red[lane & (kDirectWaves - 1)][1] : 0.0;
            e0 = in ? red[lane & (kDirectWaves - 1)][2] : 1.0;
            e1 = in ? red[lane & (kDirectWaves - 1)][3] : 0.0;
            wave_add(b0, b1, m);
            wave_add(e0, e1, m);
        }
    }
    if (G > 1) {
        double *mine = part + 4 * ((size_t)i * G + g);
        if (threadIdx.x == 0) {
            const double v[4] = {b0, b1, e0, e1};
            for (int k = 0; k < 4; k++) __hip_atomic_store(mine + k, v[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __threadfence();
            last = atomicAdd(&ticket[i], 1u) == G - 1;
        }
        __syncthreads();
        if (!last || wave != 0) return;
        __threadfence();
        b0 = e0 = 1.0;
        b1 = e1 = 0.0;
        const double *their = part + 4 * (size_t)i * G;
        for (uint32_t k = lane; k < G; k += 64) {
            double v[4];
            for (int q = 0; q < 4; q++)
                v[q] = __hip_atomic_load(their + 4 * (size_t)k + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            b1 = m.dot(b1, v[0], v[1], b0);
            b0 = m.mul(b0, v[0]);
            e1 = m.dot(e1, v[2], v[3], e0);
            e0 = m.mul(e0, v[2]);
        }
        wave_add(b0, b1, m);
        wave_add(e0, e1, m);
    }
    // c1 / (c0 lhs), the Euler side in the odd lanes
    const Side &S = side[lane & 1];
    const double c0 = (lane & 1) ? e0 : b0, c1 = (lane & 1) ? e1 : b1;
    const double x = f_mulmod(c0, (double)S.lhs, m.f);
    const uint64_t r = f_canon(f_mulmod(c1, f_pow_u(x, p - 2, m.f), m.f), m.f);
    const uint64_t re = __shfl((unsigned long long)r, 1, 64);
    if (lane == 0) {
        out[i] = wv_result{p, r, re, (r == 0 ? WV_FLAG_WOLSTENHOLME : 0u) | (re == 0 ? WV_FLAG_VANDIVER : 0u), 0};
        if (terms) {
            terms[2 * (size_t)i] = side[0].terms;
            terms[2 * (size_t)i + 1] = side[1].terms;
        }
    }
}

template <bool SMALL>
__global__ void __launch_bounds__(64 * kDirectWaves) k_direct(TableStore ts, const uint64_t *__restrict__ primes, int tb,
                                                              int te, int fb, int fe, uint32_t G, double *part,
                                                              uint32_t *ticket, uint64_t *__restrict__ terms,
                                                              wv_result *__restrict__ out) {
    __shared__ DirectLds lds;
    direct_prime<SMALL>(lds, ts, primes, tb, te, fb, fe, blockIdx.x / G, blockIdx.x % G, G, part, ticket, terms, out);
}

// The same where only the device knows the primes: k_direct_pick has decided
// (mode[0]: workgroups per prime, 0: the term sums; mode[1]: every p < 2^27), and a
// fixed grid goes through the primes after the term sums have run, on primes
// that were left out of them if they come this way.
__global__ void __launch_bounds__(64 * kDirectWaves) k_direct_device(TableStore ts, const uint64_t *__restrict__ primes,
                                                                     uint32_t n, int tb, int te, int fb, int fe,
                                                                     const uint32_t *__restrict__ mode, double *part,
                                                                     uint32_t *ticket, wv_result *__restrict__ out) {
    __shared__ DirectLds lds;
    const uint32_t G = __builtin_amdgcn_readfirstlane(mode[0]), small = __builtin_amdgcn_readfirstlane(mode[1]);
    for (uint32_t w = blockIdx.x; w < n * G; w += gridDim.x) {
        if (small) direct_prime<true>(lds, ts, primes, tb, te, fb, fe, w / G, w % G, G, part, ticket, nullptr, out);
        else direct_prime<false>(lds, ts, primes, tb, te, fb, fe, w / G, w % G, G, part, ticket, nullptr, out);
        __syncthreads();   // LDS free
    }
}

// One workgroup: the batch's terms and largest prime, the choice of the path by
// direct_rule, the primes for the term sums (all 0, which the
// plan rejects, if they go the other way), cleared scalars and tickets.
__global__ void __launch_bounds__(1024) k_direct_pick(const uint64_t *__restrict__ primes, uint32_t n, double cost,
                                                      uint32_t threads, uint64_t *__restrict__ gated,
                                                      uint64_t *__restrict__ scal, uint32_t *__restrict__ mode,
                                                      uint32_t *__restrict__ ticket) {
    __shared__ double sum[16];
    __shared__ uint64_t top[16];
    __shared__ uint32_t pick;
    double s = 0.0;
    uint64_t m = 0;
    for (uint32_t i = threadIdx.x; i < n; i += 1024) {
        const uint64_t p = primes[i];
        if (p < WV_P_MAX) {
            s += (double)p;
            m = max(m, p);
        }
        ticket[i] = 0;
    }
    for (int o = 32; o >= 1; o >>= 1) {
        s += __shfl_xor(s, o, 64);
        m = max(m, (uint64_t)__shfl_xor((unsigned long long)m, o, 64));
    }
    if ((threadIdx.x & 63) == 0) sum[threadIdx.x >> 6] = s, top[threadIdx.x >> 6] = m;
    if (threadIdx.x < 8) scal[threadIdx.x] = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; w++) s += sum[w], m = max(m, top[w]);
        uint32_t G = 0;
        if (direct_rule(n, m, s, cost)) {
            const double lanes = direct_lanes(n, m, cost);
            for (G = 1; 2.0 * G * threads <= lanes && 2 * G * (uint64_t)n <= kDirectParts; G *= 2) {}
        }
        pick = G;
        mode[0] = G;
        mode[1] = m <= kDirectSmallP;
    }
    __syncthreads();
    const bool sums = pick == 0;
    for (uint32_t i = threadIdx.x; i < n; i += 1024) gated[i] = sums ? primes[i] : 0;
}

__global__ void __launch_bounds__(256) k_direct_zero(uint32_t *__restrict__ t, uint32_t n) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) t[i] = 0;
}

// the batch's terms: scal[kScalTerms], scal[kScalTermsB]; no other word stands for anything
__global__ void __launch_bounds__(1024) k_direct_total(const uint64_t *__restrict__ terms, uint32_t n,
                                                       uint64_t *__restrict__ scal) {
    __shared__ uint64_t part[2][16];
    uint64_t b = 0, e = 0;
    for (uint32_t i = threadIdx.x; i < n; i += 1024) {
        b += terms[2 * (size_t)i];
        e += terms[2 * (size_t)i + 1];
    }
    for (int o = 32; o >= 1; o >>= 1) {
        b += __shfl_xor((unsigned long long)b, o, 64);
        e += __shfl_xor((unsigned long long)e, o, 64);
    }
    if ((threadIdx.x & 63) == 0) part[0][threadIdx.x >> 6] = b, part[1][threadIdx.x >> 6] = e;
    __syncthreads();
    if (threadIdx.x < 8) {
        uint64_t v = 0;
        if (threadIdx.x == kScalTerms || threadIdx.x == kScalTermsB)
            for (int w = 0; w < 16; w++) v += part[0][w] + (threadIdx.x == kScalTerms ? part[1][w] : 0);
        scal[threadIdx.x] = v;
    }
}

}  // namespace

bool direct_takes(const wv_ctx *c, uint64_t n, uint64_t pmax, double sum, DirectShape *d) {
    return grid_allowed(c, c->tb, c->te) && direct_shape(n, pmax, sum, side_cost(c, c->tb) + side_cost(c, c->te), d);
}

int direct_reserve(wv_ctx *c, uint32_t n, const DirectShape &d) {
    WV_TRY(ensure(c, c->direct_terms, 2 * (size_t)n * sizeof(uint64_t)));
    WV_TRY(ensure(c, c->scal, 8 * sizeof(uint64_t)));
    if (d.G > 1) {
        WV_TRY(ensure(c, c->direct_part, 4 * (size_t)n * d.G * sizeof(double)));
        WV_TRY(ensure(c, c->direct_ticket, (size_t)n * sizeof(uint32_t)));
    }
    return WV_OK;
}

int direct_enqueue(wv_ctx *c, const DirectShape &d, const uint64_t *d_primes, uint32_t n, wv_result *d_out) {
    hipStream_t st = c->stream;
    if (d.G > 1)
        hipLaunchKernelGGL(k_direct_zero, dim3((n + 255) / 256), dim3(256), 0, st, as<uint32_t>(c->direct_ticket), n);
    const uint32_t most = direct_launch_primes(d);
    for (uint64_t i = 0; i < n; i += most) {
        const uint32_t k = (uint32_t)std::min<uint64_t>(most, n - i);
        hipLaunchKernelGGL(d.small ? k_direct<true> : k_direct<false>, dim3(k * d.G), dim3(d.threads), 0, st,
                           table_store(c), d_primes + i, c->tb, c->te, table_fallback(c, c->tb),
                           table_fallback(c, c->te), d.G, as<double>(c->direct_part) + 4 * i * d.G,
                           as<uint32_t>(c->direct_ticket) + i, as<uint64_t>(c->direct_terms) + 2 * i, d_out + i);
    }
    hipLaunchKernelGGL(k_direct_total, dim3(1), dim3(1024), 0, st, as<uint64_t>(c->direct_terms), n,
                       as<uint64_t>(c->scal));
    WV_HIP(hipGetLastError());
    return WV_OK;
}

static unsigned device_threads(uint32_t n) { return n > 4096 ? 64 : n > 512 ? 128 : 64 * kDirectWaves; }

int direct_device_pick(wv_ctx *c, const uint64_t *d_primes, uint32_t n, const DirectScratch &x, uint64_t *scal,
                       hipStream_t st) {
    hipLaunchKernelGGL(k_direct_pick, dim3(1), dim3(1024), 0, st, d_primes, n, side_cost(c, c->tb) + side_cost(c, c->te),
                       device_threads(n), x.gated, scal, x.mode, x.ticket);
    WV_HIP(hipGetLastError());
    return WV_OK;
}

int direct_device_run(wv_ctx *c, const uint64_t *d_primes, uint32_t n, const DirectScratch &x, wv_result *d_out,
                      hipStream_t st) {
    hipLaunchKernelGGL(k_direct_device, dim3((unsigned)c->num_cus * 8), dim3(device_threads(n)), 0, st, table_store(c),
                       d_primes, n, c->tb, c->te, table_fallback(c, c->tb), table_fallback(c, c->te), x.mode, x.part,
                       x.ticket, d_out);
    WV_HIP(hipGetLastError());
    return WV_OK;
}

int direct_batch_sync(wv_ctx *c, const DirectShape &d, const uint64_t *d_primes, uint32_t n, wv_result *d_out) {
    hipStream_t st = c->stream;
    WV_TRY(direct_reserve(c, n, d));
    WV_HIP(hipEventRecord(c->ev[EV_PLAN0], st));
    WV_TRY(direct_enqueue(c, d, d_primes, n, d_out));
    WV_HIP(hipEventRecord(c->ev[EV_FINAL], st));
    uint64_t host[8];
    WV_HIP(hipMemcpyAsync(host, c->scal.ptr, sizeof(host), hipMemcpyDeviceToHost, st));
    WV_HIP(hipStreamSynchronize(st));
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, c->ev[EV_PLAN0], c->ev[EV_FINAL]);
    c->stats.ms_total += ms;
    c->stats.ms_sum += ms;   // the phases are not timed apart
    direct_stats(c, d, n, host);
    return WV_OK;
}

void direct_stats(wv_ctx *c, const DirectShape &d, uint64_t n, const uint64_t *scal) {
    wv_stats &s = c->stats;
    s.n_primes += n;
    s.n_sums += n * (uint64_t)(side_slots(c, c->tb) + side_slots(c, c->te));
    s.n_terms += scal[kScalTerms];
    s.n_terms_b += scal[kScalTermsB];
    s.chunk_terms = 4;
    s.block_k_b = (uint32_t)sum_variant_kb(c->variant);
    s.block_k_e = (uint32_t)sum_variant_ke(c->variant);
    s.grid = (uint32_t)std::min<uint64_t>(n * d.G, UINT32_MAX);
}

}  // namespace wv
