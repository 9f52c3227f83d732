// Host checks of the grid path's plan and of its exact arithmetic (plain C++).
#include <cstdio>
#include <cstdlib>

#include "grid_plan.hpp"

using namespace wv;
typedef unsigned __int128 u128;
typedef __int128 i128;

static int fails = 0;
#define CHECK(c)                                                   \
    do {                                                           \
        if (!(c)) {                                                \
            printf("%s:%d: %s\n", __FILE__, __LINE__, #c);         \
            fails++;                                               \
        }                                                          \
    } while (0)

static uint64_t powmod(uint64_t a, uint64_t e, uint64_t m) {
    uint64_t r = 1;
    for (; e; e >>= 1, a = (uint64_t)((u128)a * a % m))
        if (e & 1) r = (uint64_t)((u128)r * a % m);
    return r;
}

static bool is_prime(uint64_t n) {
    for (uint64_t a : {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37}) {
        if (n % a == 0) return n == a;
        uint64_t d = n - 1;
        int s = 0;
        while (!(d & 1)) d >>= 1, s++;
        uint64_t x = powmod(a, d, n);
        if (x == 1 || x == n - 1) continue;
        bool comp = true;
        for (int r = 1; r < s && comp; r++) {
            x = (uint64_t)((u128)x * x % n);
            if (x == n - 1) comp = false;
        }
        if (comp) return false;
    }
    return true;
}

static uint64_t seed = 88172645463325252ull;
static uint64_t rnd() {
    seed ^= seed << 13;
    seed ^= seed >> 7;
    seed ^= seed << 17;
    return seed;
}

static uint64_t umod(i128 c, uint64_t m) {
    const i128 r = c % (i128)m;
    return (uint64_t)(r < 0 ? r + m : r);
}

static void moduli() {
    for (int i = 0; i < 2; i++) {
        CHECK(is_prime(kNttQ[i]));
        CHECK(kNttQ[i] < (1ull << 47) && kNttQ[i] % (1ull << 17) == 1);
        CHECK(powmod(kNttRoot[i], 1ull << 16, kNttQ[i]) == kNttQ[i] - 1);   // order exactly 2^17
    }
    CHECK((u128)umod((i128)(int64_t)kNttQ1Inv, kNttQ[1]) * kNttQ[0] % kNttQ[1] == 1);
}

// ntt_crt gives c mod p for every |c| <= q1 q2 / 4 and every allowed r1, r2
static void crt() {
    const Fmod f1{(double)kNttQ[0], 1.0 / (double)kNttQ[0]}, f2{(double)kNttQ[1], 1.0 / (double)kNttQ[1]};
    const i128 top = (i128)kNttQ[0] * (i128)kNttQ[1] / 4;
    for (uint64_t p : {134217757ull, 1000000007ull, 99999999977ull, 1099511627689ull}) {
        const Fmod fp{(double)p, 1.0 / (double)p};
        const double q1p = f_reduce((double)kNttQ[0], fp);
        for (int k = 0; k < 20000; k++) {
            i128 c = (i128)(((u128)rnd() << 64 | rnd()) >> 36);   // below 2^92
            if (k < 8) c = top - k;
            if (k == 8) c = 0;
            c %= top + 1;
            if (rnd() & 1) c = -c;
            const double r1 = f_reduce((double)umod(c, kNttQ[0]), f1);
            double r2 = (double)umod(c, kNttQ[1]);
            r2 += ((double)(int)(rnd() % 20) - 10.0) * (double)kNttQ[1];   // |r2| < 10.3 q2
            if (r2 > 10.3 * (double)kNttQ[1]) r2 -= (double)kNttQ[1];
            const double g = ntt_crt(r1, r2, kNttQ1Inv, q1p, f2, fp);
            CHECK(g < 0.51 * (double)p && g > -0.51 * (double)p);
            CHECK(umod((i128)(int64_t)g, p) == umod(c, p));
        }
    }
}

// classes: valid lengths and tables, and the bound on the shifts holds for the
// exact interval lengths
static void classes() {
    for (int k = 0; k < 4000; k++) {
        const double e = 20.0 + 20.0 * (double)(rnd() >> 11) / 9007199254740992.0;
        uint64_t p = (uint64_t)std::exp2(e) | 1;
        if (k == 0) p = (1ull << 40) - 1;
        const GridClass c = grid_class(p);
        if (c.logl == 0) {
            CHECK(p < (4ull << (2 * kGridMinLog)));
            continue;
        }
        CHECK(c.logl >= kGridMinLog && c.logl <= kGridMaxLog && p >= (4ull << (2 * c.logl)));
        CHECK(c.tb >= WV_TABLE_BB1 && c.tb <= WV_TABLE_BB30 && c.te >= WV_TABLE_EE3 && c.te <= WV_TABLE_EE33);
        const uint64_t K = grid_k(c.logl), W = grid_w(c.logl);
        CHECK(W == K + 1);
        for (int t : {c.tb, c.te}) {
            // a run's sums follow one another; its blocks need at most the bound
            const GridRuns &g = grid_runs(t);
            uint64_t shifts = 0, covered = 0;
            auto ends = [&](int i, uint64_t &lo, uint64_t &len) {
                const TermDef &d = kTables[t].t[i];
                lo = (uint64_t)((u128)d.xa * p / d.xb) + 1;
                len = (uint64_t)(((u128)d.ya * p - 1) / d.yb) - lo + 1;
                CHECK(2 * (u128)d.ya <= d.yb);   // up to p / 2
            };
            uint64_t lo, len, sums = 0;
            for (int i = 0; i < kTables[t].n; i++) {
                ends(i, lo, len);
                sums += len;
                CHECK(g.run[i] < g.n);
            }
            for (int r = 0; r < g.n; r++) {
                uint64_t a, b, la, lb;
                ends(g.first[r], a, la);
                ends(g.last[r], b, lb);
                len = b + lb - a;
                covered += len;
                const uint64_t m = (len / K + W - 1) / W;
                shifts += m;
                // every denominator of the inverse list, 0 <= n < (m + 1) W, lies in (0, p)
                CHECK(m == 0 || a + K * ((m + 1) * W - 1) < p);
            }
            CHECK(covered == sums || p % 3 == 0 || p % 5 == 0);   // (p prime: no endpoint is an integer)
            CHECK(shifts <= grid_shifts(t, (double)p, c.logl));
        }
    }
}

int main() {
    moduli();
    crt();
    classes();
    if (fails) return printf("%d failed\n", fails), 1;
    printf("ok\n");
    return 0;
}
