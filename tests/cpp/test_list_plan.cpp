// Host checks of how a list of primes of any sizes is shared between the paths.
#include <cstdio>

#include "list_plan.hpp"

using namespace wv;

static int fails = 0;
#define CHECK(c)                                           \
    do {                                                   \
        if (!(c)) {                                        \
            printf("%s:%d: %s\n", __FILE__, __LINE__, #c); \
            fails++;                                       \
        }                                                  \
    } while (0)

constexpr uint64_t kMinP = 9ull << 23;   // the grid path's start
constexpr double kCost = 0.0878;

static uint64_t seed = 88172645463325252ull;
static uint64_t rnd() {
    seed ^= seed << 13;
    seed ^= seed >> 7;
    seed ^= seed << 17;
    return seed;
}

// every entry in one part, each part one that its path takes
static std::vector<ListPart> check(std::vector<uint64_t> p) {
    std::sort(p.begin(), p.end());
    const std::vector<ListPart> parts = list_parts(p.data(), p.size(), kMinP, kCost);
    std::vector<int> held(p.size(), 0);
    for (const ListPart &t : parts) {
        CHECK(t.n > 0 && t.at + t.n <= p.size() && t.lo == p[t.at] && t.hi == p[t.at + t.n - 1]);
        double s = 0;
        for (size_t i = t.at; i < t.at + t.n; i++) held[i]++, s += (double)p[i];
        if (t.path == kListGrid) CHECK(t.lo >= kMinP && grid_fits(t.lo, t.g.logl));
        DirectShape d;
        if (t.path == kListDirect)
            CHECK(direct_shape(t.n, t.hi, s, kCost, &d) && d.key() == t.d.key() && t.d.small == (t.hi <= kDirectSmallP));
    }
    for (int h : held) CHECK(parts.empty() || h == 1);
    return parts;
}

static std::vector<uint64_t> log_uniform(double a, double b, int n) {
    std::vector<uint64_t> p(n);
    for (uint64_t &x : p)
        x = (uint64_t)std::exp2(a + (b - a) * (double)(rnd() >> 11) / 9007199254740992.0) | 1;
    p[0] = std::max(p[0], kMinP);
    return p;
}

// windows: items of ranges in ascending order, the first `low` below the path's start
static void check_windows(int n) {
    std::vector<GridItem> items;
    uint64_t at = (uint64_t)std::exp2(10.0 + (double)(rnd() % 200) / 10.0);
    size_t low = 0;
    for (int k = 0; k < n && at < (1ull << 39); k++) {
        const uint64_t top = at + rnd() % (1 << 20);
        const uint32_t m = 1 + (uint32_t)(rnd() % 2000);
        if (at < kMinP) low++;
        items.push_back(GridItem{at, top, m, (uint32_t)(2 * k), (double)m * (double)top});
        at = top + (rnd() % 3 ? rnd() % (at / 2) : 0);
    }
    const ListPlan plan = plan_items(items, low, kCost);
    size_t next = 0;
    for (const ListPart &t : plan.parts) {
        CHECK(t.begin == next && t.end > t.begin && t.at == items[t.begin].at);
        CHECK(t.lo == items[t.begin].lo && t.hi == items[t.end - 1].hi);
        uint32_t m = 0;
        for (size_t i = t.begin; i < t.end; i++) m += items[i].n;
        CHECK(m == t.n);
        CHECK(t.begin >= low || (t.begin == 0 && t.end == low && t.path != kListGrid));
        if (t.path == kListGrid) CHECK(grid_fits(t.lo, t.g.logl));
        next = t.end;
    }
    CHECK(next == items.size());
}

int main() {
    for (int k = 0; k < 2000; k++) check_windows(1 + (int)(rnd() % 64));
    for (int k = 0; k < 4000; k++) {
        const double a = 3.0 + (double)(rnd() % 300) / 10.0, b = std::max(a, 27.0) + (double)(rnd() % 120) / 10.0;
        check(log_uniform(a, std::min(b, 40.0), 1 + (int)(rnd() % (k % 4 ? 20 : 500))));
    }
    // one size: the grid path alone
    for (uint64_t at : {1000000007ull, 10000000019ull, 99999999977ull}) {
        const std::vector<ListPart> parts = check(std::vector<uint64_t>(64, at));
        CHECK(parts.size() == 1 && parts[0].path == kListGrid);
    }
    // few small primes beside one that needs the grid path: no batch of term sums for them
    std::vector<uint64_t> p(100, 10007);
    p.push_back(20000000089ull);
    const std::vector<ListPart> parts = check(p);
    CHECK(parts.size() == 2 && parts[0].path == kListGrid && parts[1].path == kListDirect);
    // two sizes with more than the direct path takes of each, neither able to join the other:
    // one batch of term sums is quicker than a chain each
    p.assign(60, 150000001);
    p.push_back(7000000001);
    CHECK(check(p).empty());
    if (fails) return printf("%d failed\n", fails), 1;
    printf("ok\n");
    return 0;
}
