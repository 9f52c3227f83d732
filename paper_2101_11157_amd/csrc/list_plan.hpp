// list_plan.hpp -- how a list of primes of any sizes is shared between the direct
// path, the grid path and the term sums: plain host code, unit-tested without a
// GPU.
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

#include "direct_plan.hpp"
#include "grid_plan.hpp"

namespace wv {

enum ListPath { kListDirect, kListGrid, kListSums };

// Primes [at, at + n) of the ascending list, all in [lo, hi].
struct ListPart {
    ListPath path;
    size_t at;
    uint32_t n;
    uint64_t lo, hi;
    DirectShape d;   // kListDirect
    GridClass g;     // kListGrid
};

// Time of one batch by itself, seconds, from the calls measured at the rules of
// the paths (direct_plan.hpp, grid_plan.hpp) and at those of list_parts.
inline double direct_time(const DirectShape &d, double terms, double pmax, double cost) {
    return 7e-5 + std::max(terms / (d.small ? 2.2e12 : 1.6e12), pmax * cost / (d.G * d.threads) * (d.small ? 8e-8 : 4e-8));
}
inline double sums_time(double n, double terms) { return 4.5e-4 + 6e-8 * n + terms / 5.5e12; }
inline double grid_time(const GridBatch &b, const std::vector<GridItem> &items) {
    const GridClass g = grid_batch_class(b.g, b.n, b.hi);
    if (b.n <= kGridFew && g.logl >= kGridFewLog) return 1e-6 * grid_few_us(g, b.n, (double)b.hi);
    double ops = 0;
    for (size_t i = b.begin; i < b.end; i++) ops += (double)items[i].n * grid_ops(items[i].hi, g);
    return kGridBatchS + ops / kGridRate;
}

// The parts of an ascending list whose largest prime the grid path takes and
// which the direct path does not take whole: the grid path's batches and the primes
// below the path's start, direct where that is the quicker way.  Each part has a
// chain of its own, so for a few primes of many sizes the parts together can take
// longer than one batch of term sums: then none are returned and the whole list
// goes that way.  cost: terms per unit of p.  Measured, one batch per class of
// primes and term sums below / this: 4 primes from 8e6 to 6e10 1.28 / 0.79 ms, 8
// from 2e7 to 3e9 1.34 / 0.31, 83 from 8e6 to 7e9 1.84 / 1.15.
inline std::vector<ListPart> list_parts(const uint64_t *p, size_t n, uint64_t grid_min, double cost) {
    std::vector<ListPart> out;
    double time = 0, all = 0;
    auto add = [&](ListPart t, double other) {   // other: time by the path of t
        double s = 0;
        for (size_t i = t.at; i < t.at + t.n; i++) s += (double)p[i];
        all += s;
        if (t.path == kListSums) other = sums_time((double)t.n, s * cost);
        if (direct_shape(t.n, t.hi, s, cost, &t.d)) {
            const double v = direct_time(t.d, s * cost, (double)t.hi, cost);
            if (v < other) other = v, t.path = kListDirect;
        }
        time += other;
        out.push_back(t);
    };
    const size_t low = std::lower_bound(p, p + n, grid_min) - p;
    std::vector<GridItem> items;
    grid_items(p + low, n - low, (uint32_t)low, items);
    for (const GridBatch &b : grid_batches(items))   // descending: a batch's first prime is its last item's
        add(ListPart{kListGrid, items[b.end - 1].at, b.n, b.lo, b.hi, {}, b.g}, grid_time(b, items));
    if (low) add(ListPart{kListSums, 0, (uint32_t)low, p[0], p[low - 1], {}, {}}, 0.0);
    if (time > sums_time((double)n, all * cost)) out.clear();
    return out;
}

}  // namespace wv
