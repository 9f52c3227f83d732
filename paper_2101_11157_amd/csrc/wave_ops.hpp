// wave_ops.hpp -- device helpers shared by the kernels: Montgomery constants of
// a prime, wave-uniform values, and the pair product across a wave.
#pragma once
#include <hip/hip_runtime.h>

#include "mont.hpp"
#include "sum_core.hpp"
#include "wv_internal.hpp"

namespace wv {

__device__ __forceinline__ Mont mont_of(const PrimeRec &r) {
    Mont m;
    m.p = r.p;
    m.p0 = (uint32_t)r.p;
    m.p1 = (uint32_t)(r.p >> 32);
    m.ninv = r.ninv;
    return m;
}

// Wave-uniform values are moved into scalar registers with readfirstlane /
// readlane, so that every branch and loop exit that depends on them is a
// scalar branch.  A cross-lane read through a vector shuffle inside a loop lets
// the compiler split the loop per lane, and lanes can then read a register of
// a lane that is parked on another path.
__device__ __forceinline__ uint64_t readfirst_u64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int mask) {
    uint32_t lo = __shfl_xor((int)(uint32_t)v, mask, 64);
    uint32_t hi = __shfl_xor((int)(uint32_t)(v >> 32), mask, 64);
    return ((uint64_t)hi << 32) | lo;
}

// v of lane (lane ^ X) within the same 32-lane half (0 < X < 32): ds_swizzle
// in bit-mask mode (offset = and-mask 0x1f | or-mask 0 << 5 | xor-mask X << 10).
// The pattern is an immediate, so unlike ds_bpermute no per-lane address
// register is held; the persistent sum kernel would otherwise keep those
// addresses live across its loop and spill them.
template <int X>
__device__ __forceinline__ uint32_t swz_xor(uint32_t v) {
    static_assert(X > 0 && X < 32, "swizzle reaches within a 32-lane half");
    return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1f | (X << 10));
}

template <int X>
__device__ __forceinline__ uint64_t swz_xor_u64(uint64_t v) {
    return ((uint64_t)swz_xor<X>((uint32_t)(v >> 32)) << 32) | swz_xor<X>((uint32_t)v);
}

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int l) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, l);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

// minimum over the 64 lanes of a fully active wave, as a wave-uniform value
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
    v = min(v, swz_xor<16>(v));
    v = min(v, swz_xor<8>(v));
    v = min(v, swz_xor<4>(v));
    v = min(v, swz_xor<2>(v));
    v = min(v, swz_xor<1>(v));
    // readlane returns int: compare as unsigned (0xffffffff is the largest value)
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0);
    const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)v, 32);
    return a < b ? a : b;
}

// Butterfly of eqnCombinePairs across the 64 lanes of a fully active wave
// (same prime on all lanes): each 32-lane half by swizzles, then the two
// halves through scalar reads; every lane ends with the product of all 64
// pairs.
template <int X>
__device__ __forceinline__ void pair_swz_step(uint64_t &c0, uint64_t &c1, const Mont &m) {
    const uint64_t d0 = swz_xor_u64<X>(c0);
    const uint64_t d1 = swz_xor_u64<X>(c1);
    pair_mul(c0, c1, d0, d1, m);
}

__device__ __forceinline__ void wave_pair_reduce(uint64_t &c0, uint64_t &c1, const Mont &m) {
    pair_swz_step<16>(c0, c1, m);
    pair_swz_step<8>(c0, c1, m);
    pair_swz_step<4>(c0, c1, m);
    pair_swz_step<2>(c0, c1, m);
    pair_swz_step<1>(c0, c1, m);
    const uint64_t d0 = readlane_u64(c0, 32), d1 = readlane_u64(c1, 32);
    c0 = readlane_u64(c0, 0);
    c1 = readlane_u64(c1, 0);
    pair_mul(c0, c1, d0, d1, m);
}

__device__ __forceinline__ Fmod fmod_of(uint64_t p) {
    Fmod f;
    f.p = (double)p;
    f.pinv = 1.0 / f.p;
    return f;
}

// a^e, e >= 1 the same for the whole wave (scalar control flow)
__device__ __forceinline__ double f_pow_u(double a, uint64_t e, const Fmod &f) {
    e = readfirst_u64(e);
    double r = a;
    for (int i = 62 - __builtin_clzll(e); i >= 0; i--) {
        r = f_mulmod(r, r, f);
        if ((e >> i) & 1) r = f_mulmod(r, a, f);
    }
    return r;
}

// A signed integer of any size (limbs of its magnitude, base 2^32, least
// significant first) mod p, canonical.
__device__ inline uint64_t limbs_mod(const uint32_t *__restrict__ limb, uint32_t off, int nlimb, bool neg, uint64_t p) {
    uint64_t r = 0;
    for (int k = nlimb - 1; k >= 0; k--) r = shift_in_limb(r, limb[off + k], p);
    return neg && r ? p - r : r;
}

// Table of one side for prime p: the configured one where it applies, else
// the table it names for the primes it does not serve (a chain of defined
// tables with falling min_p that ends at a compiled table; fb if a chain were
// ever longer than the registry); the root forms for p = 5 and 7 (readings of
// the paper: the specialised tables need p >= 11).
__device__ inline int pick_table(TableStore ts, int side, uint64_t p, int cfg, int fb) {
    if (side == 0 && p == 5) return WV_TABLE_BB1;
    if (side == 0 && p == 7) return WV_TABLE_V12;
    if (side == 1 && p < 11) return WV_TABLE_E1;
    int t = cfg;
    for (int hop = 0; hop <= kMaxTableChain && t >= WV_TABLE_COUNT; hop++) {
        const TableHead h = ts.head[t];
        if (p >= h.min_p && limbs_mod(ts.limb, h.lhs_off, h.lhs_nlimb, false, p) != 0) return t;
        t = h.below;
    }
    return t >= WV_TABLE_COUNT ? fb : t;
}

}  // namespace wv
