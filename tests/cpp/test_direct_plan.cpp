// Host checks of the direct path's rule: its launches at every length of list.
#include <cmath>
#include <cstdio>

#include "direct_plan.hpp"

using namespace wv;

static int fails = 0;
#define CHECK(c)                                           \
    do {                                                   \
        if (!(c)) {                                        \
            printf("%s:%d: %s\n", __FILE__, __LINE__, #c); \
            fails++;                                       \
        }                                                  \
    } while (0)

int main() {
    int taken = 0;
    for (double e = 0.0; e <= 32.0; e += 0.125)
        for (double q = 2.4; q <= 36.0; q += 0.2) {
            const uint64_t n = std::min<uint64_t>((uint64_t)std::exp2(e), 0xFFFFFFFFull), pmax = (uint64_t)std::exp2(q);
            DirectShape d;
            if (!direct_shape(n, pmax, (double)n * (double)pmax, 0.0878, &d)) continue;
            taken++;
            CHECK(d.G >= 1 && d.G <= 1024 && d.threads >= 64 && d.threads <= 64 * kDirectWaves);
            CHECK(d.small == (pmax <= kDirectSmallP));
            // fewer than 2^32 threads a launch, and every prime in one of them
            const uint64_t most = direct_launch_primes(d);
            CHECK(most >= 1 && most * d.G * d.threads < (1ull << 32));
            uint64_t held = 0, launches = 0;
            for (uint64_t i = 0; i < n; i += most) held += std::min(most, n - i), launches++;
            CHECK(held == n && (launches == 1 || n > most));
        }
    CHECK(taken > 1000);
    // slots for every prime a narrow window may hold, and few without one
    uint64_t last = 0;
    for (uint64_t n = 0; n < 5000; n++) {
        const uint64_t pad = direct_pad(n);
        CHECK(pad >= n && pad >= last && pad <= std::max<uint64_t>(16, n <= 1024 ? 2 * n : n + 1023));
        last = pad;
    }
    if (fails) return printf("%d failed\n", fails), 1;
    printf("ok\n");
    return 0;
}
