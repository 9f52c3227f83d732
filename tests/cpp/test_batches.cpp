// Host checks of the batches that lists and ranges of primes form on the grid
// path: no prime meets a length that it cannot take, whatever their sizes.
#include <cstdio>
#include <cstdlib>

#include "grid_plan.hpp"

using namespace wv;
typedef unsigned __int128 u128;

static int fails = 0;
#define CHECK(c)                                           \
    do {                                                   \
        if (!(c)) {                                        \
            printf("%s:%d: %s\n", __FILE__, __LINE__, #c); \
            fails++;                                       \
        }                                                  \
    } while (0)

constexpr uint64_t kMinP = 9ull << 23;   // the path's start

static uint64_t seed = 88172645463325252ull;
static uint64_t rnd() {
    seed ^= seed << 13;
    seed ^= seed >> 7;
    seed ^= seed << 17;
    return seed;
}

// every denominator lo + K n, n < (shifts + 1) W, of every run lies in (0, p)
static bool denominators(uint64_t p, const GridClass &g) {
    const uint64_t K = grid_k(g.logl), W = grid_w(g.logl);
    for (int t : {g.tb, g.te}) {
        const GridRuns &r = grid_runs(t);
        for (int k = 0; k < r.n; k++) {
            const TermDef &a = kTables[t].t[r.first[k]], &b = kTables[t].t[r.last[k]];
            const uint64_t lo = (uint64_t)((u128)a.xa * p / a.xb) + 1;
            const uint64_t len = (uint64_t)(((u128)b.ya * p - 1) / b.yb) - lo + 1, m = (len / K + W - 1) / W;
            if (m && lo + K * ((m + 1) * W - 1) >= p) return false;
        }
    }
    return true;
}

// the batches of items: each item in one of them, every prime between an item's
// ends fit for the length its batch runs in
static void check(std::vector<GridItem> items) {
    size_t n = 0, m = 0, next = 0;
    for (const GridItem &t : items) n += t.n;
    for (const GridBatch &b : grid_batches(items)) {
        CHECK(b.begin == next && b.end > b.begin);
        next = b.end;
        uint32_t k = 0;
        for (size_t i = b.begin; i < b.end; i++) {
            const GridItem &t = items[i];
            k += t.n;
            CHECK(b.lo <= t.lo && t.hi <= b.hi);
            CHECK(i == 0 || items[i - 1].hi >= t.hi);
        }
        CHECK(k == b.n);
        m += b.n;
        const GridClass run = grid_batch_class(b.g, b.n, b.hi);
        for (const GridClass &g : {b.g, run}) {
            CHECK(grid_fits(b.lo, g.logl) && g.logl >= kGridMinLog);
            CHECK(g.logl <= kNttMaxLog || b.hi <= kGridSplitMaxP);
            CHECK(denominators(b.lo, g) && denominators(b.hi, g));
        }
    }
    CHECK(next == items.size() && m == n);
}

static void check_list(std::vector<uint64_t> p) {
    std::sort(p.begin(), p.end());
    std::vector<GridItem> items;
    grid_items(p.data(), p.size(), 7, items);
    size_t at = 7;
    for (const GridItem &t : items) {
        CHECK(t.at == at && t.lo == p[at - 7] && t.hi == p[at - 7 + t.n - 1]);
        at += t.n;
    }
    check(items);
}

int main() {
    // sizes of lists whose least primes read a zero denominator in the class of the largest
    for (uint64_t least : {76007749ull, 75510511ull, 75505151ull})
        for (uint64_t most : {50000000000ull, 90000000000ull, (1ull << 39) - 1, (1ull << 40) - 1})
            for (int n : {1, 7, 50, 1000}) {
                std::vector<uint64_t> p(1, least);
                for (int k = 0; k < n; k++) p.push_back(most - 2 * k);
                check_list(p);
            }
    // a class whose sizes are two ranges: 1.13e9 and 4.4e9, alone and beside larger ones
    check_list({1130000009ull, 4400000009ull});
    check_list({1130000009ull, 4400000009ull, 50000000021ull});
    for (int k = 0; k < 3000; k++) {
        const double a = std::log2((double)kMinP), w = 40.0 - a;
        std::vector<uint64_t> p(1 + rnd() % (k % 3 ? 12 : 300));
        for (uint64_t &x : p) {
            const double u = (double)(rnd() >> 11) / 9007199254740992.0;
            x = std::max<uint64_t>(kMinP, (uint64_t)std::exp2(a + w * u) | 1);
        }
        check_list(p);
        // ranges of up to 2^26 integers among them
        std::vector<GridItem> items;
        grid_items(p.data(), 0, 0, items);
        CHECK(items.empty());
        for (uint64_t x : p) {
            const uint64_t hi = std::min<uint64_t>(1ull << 40, x + (rnd() >> (38 + rnd() % 26)));
            items.push_back(GridItem{x, hi, 1 + (uint32_t)(rnd() % 1000), 0, 0.0});
        }
        check(items);
        // a range of any width
        check({GridItem{p[0], std::max(p[0], p.back()), 5, 0, 0.0}});
    }
    if (fails) return printf("%d failed\n", fails), 1;
    printf("ok\n");
    return 0;
}
