// list_plan.hpp -- how primes of any sizes, a list or those of windows, are shared
// between the direct path, the grid path and the term sums: plain host code,
// unit-tested without a GPU.
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

#include "direct_plan.hpp"
#include "grid_plan.hpp"

namespace wv {

enum ListPath { kListDirect, kListGrid, kListSums };

// Items [begin, end): n primes, all in [lo, hi], the first where the first item is.
struct ListPart {
    ListPath path;
    size_t begin, end;
    uint32_t n, at;
    uint64_t lo, hi;
    DirectShape d;   // kListDirect
    GridClass g;     // kListGrid
};

struct ListPlan {
    std::vector<ListPart> parts;   // ascending
    double time, sums;             // of the parts, and of one batch of term sums for all
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

// The parts of items in ascending order (of lo, and of hi): the first `low`, below
// the grid path's start, as one, the others in the grid path's batches, each
// direct where that is the quicker way.  cost: terms per unit of p.
inline ListPlan plan_items(const std::vector<GridItem> &items, size_t low, double cost) {
    ListPlan plan{{}, 0.0, 0.0};
    double n = 0, all = 0;
    for (const GridItem &t : items) n += t.n, all += t.sum;
    plan.sums = sums_time(n, all * cost);
    auto add = [&](ListPart t, double other) {   // other: time by the path of t
        double s = 0;
        for (size_t i = t.begin; i < t.end; i++) s += items[i].sum;
        if (t.path == kListSums) other = sums_time((double)t.n, s * cost);
        if (direct_shape(t.n, t.hi, s, cost, &t.d)) {
            const double v = direct_time(t.d, s * cost, (double)t.hi, cost);
            if (v < other) other = v, t.path = kListDirect;
        }
        plan.time += other;
        plan.parts.push_back(t);
    };
    if (low) {
        ListPart t{kListSums, 0, low, 0, items[0].at, items[0].lo, items[low - 1].hi, {}, {}};
        for (size_t i = 0; i < low; i++) t.n += items[i].n;
        add(t, 0.0);
    }
    std::vector<GridItem> top(items.rbegin(), items.rend() - low);   // descending
    const std::vector<GridBatch> batches = grid_batches(top);
    for (size_t k = batches.size(); k-- > 0;) {
        const GridBatch &b = batches[k];
        const size_t begin = items.size() - b.end;
        add(ListPart{kListGrid, begin, items.size() - b.begin, b.n, items[begin].at, b.lo, b.hi, {}, b.g}, grid_time(b, top));
    }
    return plan;
}

// The parts of an ascending list whose largest prime the grid path takes and
// which the direct path does not take whole.  Each part has a chain of its own,
// so for a few primes of many sizes the parts together can take longer than one
// batch of term sums: then none are returned and the whole list goes that way.
// Measured, one batch per class of primes and term sums below / this: 4 primes
// from 8e6 to 6e10 1.28 / 0.79 ms, 8 from 2e7 to 3e9 1.34 / 0.31, 83 from 8e6 to
// 7e9 1.84 / 1.15.
inline std::vector<ListPart> list_parts(const uint64_t *p, size_t n, uint64_t grid_min, double cost) {
    const size_t low = std::lower_bound(p, p + n, grid_min) - p;
    std::vector<GridItem> items;
    if (low) {
        items.push_back(GridItem{p[0], p[low - 1], (uint32_t)low, 0, 0.0});
        for (size_t i = 0; i < low; i++) items[0].sum += (double)p[i];
    }
    grid_items(p + low, n - low, (uint32_t)low, items);
    ListPlan plan = plan_items(items, low ? 1 : 0, cost);
    if (plan.time > plan.sums) return {};
    return std::vector<ListPart>(plan.parts.rbegin(), plan.parts.rend());   // the largest primes first
}

}  // namespace wv
