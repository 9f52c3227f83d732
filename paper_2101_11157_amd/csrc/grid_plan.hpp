// grid_plan.hpp -- which congruences and which block length the grid path uses
// for primes of a size: plain host code, unit-tested without a GPU.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

#include "ntt.hpp"
#include "wv_tables.hpp"
#include "wvprime.h"

namespace wv {

struct GridClass {
    int logl = 0;          // transform length 2^logl; blocks of K = 2^(logl - 1) - 1 terms
    int tb = 0, te = 0;    // compiled tables
    double ops = 0;        // modelled operations per prime
    bool operator==(const GridClass &o) const { return logl == o.logl && tb == o.tb && te == o.te; }
};

// The longest transform of one workgroup is 2^kNttMaxLog; one of twice that is
// split into two of them (below 2^39, where its sums of 2^14 products stay
// below a quarter of the moduli's product).
constexpr int kGridMaxLog = kNttMaxLog + 1;
constexpr int kGridMinLog = 11;   // the shortest the path's primes take
constexpr uint64_t kGridSplitMaxP = 1ull << 39;

constexpr uint64_t grid_k(int logl) { return (1ull << (logl - 1)) - 1; }
constexpr uint64_t grid_w(int logl) { return 1ull << (logl - 1); }

// Sums whose intervals touch (one's upper endpoint is the next one's lower, and
// y p is no integer, so their s follow one another) are one run: one
// progression of block starts serves them all, and only the blocks that hold
// an endpoint are summed term by term.  EE33's 33 sums are 6 runs.
constexpr int kMaxRunSums = 34;
struct GridRuns {
    uint8_t n = 0;                       // runs
    uint8_t first[kMaxRunSums] = {};     // first and last sum of each run, ascending in s
    uint8_t last[kMaxRunSums] = {};
    uint8_t run[kMaxRunSums] = {};       // run of each sum
};

inline GridRuns find_runs(const TableDef &d) {
    GridRuns g;
    int ord[kMaxRunSums];
    for (int i = 0; i < d.n; i++) ord[i] = i;
    std::sort(ord, ord + d.n, [&](int a, int b) {
        return (uint64_t)d.t[a].xa * d.t[b].xb < (uint64_t)d.t[b].xa * d.t[a].xb;
    });
    for (int k = 0; k < d.n; k++) {
        const TermDef &t = d.t[ord[k]];
        const bool joins = k > 0 && (uint64_t)d.t[ord[k - 1]].ya * t.xb == (uint64_t)t.xa * d.t[ord[k - 1]].yb;
        if (!joins) g.first[g.n++] = (uint8_t)ord[k];
        g.last[g.n - 1] = (uint8_t)ord[k];
        g.run[ord[k]] = (uint8_t)(g.n - 1);
    }
    return g;
}

// runs of compiled table id (eqnBB1 .. eqnEE33)
inline const GridRuns &grid_runs(int id) {
    struct All {
        GridRuns r[WV_TABLE_EE33 + 1];
        All() {
            for (int i = 0; i <= WV_TABLE_EE33; i++) r[i] = find_runs(kTables[i]);
        }
    };
    static const All all;
    return all.r[id];
}

inline double run_width(int id, int r) {
    const GridRuns &g = grid_runs(id);
    const TermDef &a = kTables[id].t[g.first[r]], &b = kTables[id].t[g.last[r]];
    return (double)b.ya / b.yb - (double)a.xa / a.xb;
}

// Upper bound on the shifts (workgroups of W block starts) of one prime p with
// a table's runs: a run over (x p, y p) holds at most (y - x) p + 1 terms.
inline uint64_t grid_shifts(int id, double p, int logl) {
    const double K = (double)grid_k(logl), W = (double)grid_w(logl);
    uint64_t s = 0;
    for (int r = 0; r < grid_runs(id).n; r++) s += (uint64_t)((run_width(id, r) * p + 1.0) / K / W) + 1;
    return s;
}

// The same as an estimate: ceil of the blocks over W, no block no shift.
inline double grid_shifts_est(int id, double p, int logl) {
    const double K = (double)grid_k(logl), W = (double)grid_w(logl);
    double s = 0;
    for (int r = 0; r < grid_runs(id).n; r++) s += std::ceil(std::floor(run_width(id, r) * p / K) / W);
    return s;
}

// Operations of a pair of transforms (both moduli) of length L: about 50 per
// element and modulus at every length used; a split one, bound by memory, takes
// 1.4 times as long (330 primes, split / whole: 3e10 9.9 / 9.2 ms, 5e10 12.8 /
// 13.5, 1e11 19.7 / 22.2, 4e11 57.6 / 86.0).
inline double grid_pair_ops(int logl) {
    const double L = (double)(1ull << logl);
    return 2.0 * L * (14.0 + 2.6 * logl) * (logl > kNttMaxLog ? 1.4 : 1.0);
}

// One side's operations per prime: each shift transforms its kernel and brings
// back `polys` value vectors, whose values are folded once; every run has an
// inverse list, every endpoint a block's worth of single terms (half of one at
// the end of a run).
inline double grid_side_ops(int id, double p, int logl) {
    const double W = (double)grid_w(logl), K = (double)grid_k(logl);
    const TableDef &d = kTables[id];
    const int polys = d.deg + 1, runs = grid_runs(id).n;
    const double s = grid_shifts_est(id, p, logl);
    const double pair = grid_pair_ops(logl);
    return s * (pair + polys * (pair + 2.0 * W * 20.0) + W * 40.0) + (s + runs) * W * 30.0 +
           (d.n - 0.5 * runs) * K * 30.0 + d.n * 4000.0;
}

// Node values of blocks of K terms, by doubling from blocks of 255.
inline double grid_build_ops(int logl) {
    double ops = 255.0 * 256.0 * 28.0 + 4.0 * grid_pair_ops(logl);
    for (int l = kNttMinLog; l < logl; l++) ops += 19.0 * grid_pair_ops(l) + 600.0 * (double)(1ull << l);
    return ops;
}

// The compiled congruences of least modelled work for primes near p at one
// length.
inline GridClass grid_at_length(uint64_t p, int logl) {
    GridClass c;
    c.logl = logl;
    double b = 1e300, e = 1e300;
    for (int t = WV_TABLE_BB1; t <= WV_TABLE_EE33; t++) {
        const double v = grid_side_ops(t, (double)p, logl);
        if (kTables[t].deg == 3 && v < b) b = v, c.tb = t;
        if (kTables[t].deg == 2 && v < e) e = v, c.te = t;
    }
    c.ops = b + e + grid_build_ops(logl);
    return c;
}

// Whether p can take a length: p >= 4 L^2, so that every difference of two
// points, at most p/2 + 2 K W, is below p and nonzero.
inline bool grid_fits(uint64_t p, int logl) { return p >= (4ull << (2 * logl)); }

// The least modelled work for primes near hi over the lengths, too, that every
// prime from lo on can take.
inline GridClass grid_search(uint64_t lo, uint64_t hi, int max_log) {
    GridClass best;
    best.ops = 1e300;
    for (int logl = kGridMinLog; logl <= max_log; logl++) {
        if (!grid_fits(lo, logl) || (logl > kNttMaxLog && hi >= kGridSplitMaxP)) break;
        const GridClass c = grid_at_length(hi, logl);
        if (c.ops < best.ops) best = c;
    }
    return best;
}

// The grid path's class for p: that of the least prime of its sixteenth of an
// octave (so primes of one size share a class), searched once per process.
inline const GridClass &grid_class(uint64_t p) {
    struct Table {
        GridClass c[2][16 * 41];
        Table() {
            for (int i = 0; i < 16 * 41; i++)
                for (int k = 0; k < 2; k++) {
                    const uint64_t p = (uint64_t)std::ceil(std::exp2(i / 16.0));
                    c[k][i] = grid_search(p, p, kNttMaxLog + k);
                }
        }
    };
    static const Table t;
    int i = std::min((int)(std::log2((double)p) * 16.0), 16 * 41 - 1);
    while (i > 0 && p < (uint64_t)std::ceil(std::exp2(i / 16.0))) i--;   // rounding of the logarithm
    // (the last prime of a sixteenth may lie beyond the split's range when its first does not)
    return t.c[p < kGridSplitMaxP ? 1 : 0][i];
}

// The class a batch of n primes up to pmax, of class own, runs in.  Few primes do
// not fill the chip: their time is the chain of doubling steps, longer with every
// length, and the rounds in which the resident workgroups take the shifts (half
// way between whole rounds and their fraction, the waves of a round finishing
// apart).  Fitted to lists of 1 to 32 primes from 1e9 to 4e11, microseconds; of
// the lengths from 2^12 to the batch's own, measured with the class of many primes
// / this choice: 2 primes at 5e9 482 / 380, 1 at 2e10 488 / 403, 1 at 5e10 508 /
// 467, 32 at 5e9 650 / 580, 7 at 1e11 1280 / 1030 (a split length's own).
constexpr int kGridFewLog = 12;     // the shortest length measured
constexpr uint64_t kGridFew = 256;  // primes at most
inline double grid_few_us(const GridClass &c, uint64_t n, double p) {
    static constexpr double chain[] = {330, 330, 400, 530}, round[] = {100, 112, 128, 360};
    static constexpr double resident[] = {1024, 512, 256, 256};
    static_assert(kGridFewLog + 3 == kGridMaxLog, "an entry per length");
    const int k = c.logl - kGridFewLog;
    const double r = (double)n / resident[k] * (grid_shifts_est(c.tb, p, c.logl) + grid_shifts_est(c.te, p, c.logl));
    return chain[k] + round[k] * 0.5 * (r + std::ceil(r));
}

inline GridClass grid_batch_class(const GridClass &own, uint64_t n, uint64_t pmax) {
    if (own.logl <= kGridFewLog || n > kGridFew) return own;
    GridClass best = own;
    double best_t = grid_few_us(own, n, (double)pmax);
    for (int l = own.logl - 1; l >= kGridFewLog; l--) {
        const GridClass c = grid_at_length(pmax, l);
        const double v = grid_few_us(c, n, (double)pmax);
        if (v < best_t) best_t = v, best = c;
    }
    return best;
}

// Operations per prime near p in class g.
inline double grid_ops(uint64_t p, const GridClass &g) {
    return grid_side_ops(g.tb, (double)p, g.logl) + grid_side_ops(g.te, (double)p, g.logl) +
           grid_build_ops(g.logl);
}

// Whether n primes near p join a batch of class g (of larger primes) instead
// of running in their own: the work that g adds has to stay below what the
// kernels of one more batch take whatever it holds (about 0.35 ms of the GPU,
// measured for one prime; the path runs at about 1.7e13 operations/s).
constexpr double kGridRate = 1.7e13, kGridBatchS = 3.5e-4;
inline bool grid_joins(uint64_t p, double n, const GridClass &g) {
    if (!grid_fits(p, g.logl)) return false;
    const GridClass &own = grid_class(p);
    return own == g || (grid_ops(p, g) - own.ops) * n < kGridBatchS * kGridRate;
}

// n primes of [lo, hi], sum in all (or more), all of the path's sizes; at: where
// the caller has them.
struct GridItem {
    uint64_t lo, hi;
    uint32_t n, at;
    double sum;
};

// Items [begin, end) of one batch: n primes of [lo, hi], evaluated in class g,
// whose length every one of them can take.
struct GridBatch {
    GridClass g;
    uint64_t lo, hi;
    uint32_t n;
    size_t begin, end;
};

// The batches of items, which are put in descending order of hi: an item joins the batch before
// it where that is the cheaper way (grid_joins) and its least prime can take
// the batch's length; else it starts one in its own class, of a length that its
// own least prime can take.
inline std::vector<GridBatch> grid_batches(std::vector<GridItem> &items) {
    std::vector<GridBatch> out;
    std::stable_sort(items.begin(), items.end(), [](const GridItem &a, const GridItem &b) { return a.hi > b.hi; });
    for (size_t i = 0; i < items.size(); i++) {
        const GridItem &t = items[i];
        if (out.empty() || !grid_fits(t.lo, out.back().g.logl) || !grid_joins(t.hi, t.n, out.back().g)) {
            const GridClass &own = grid_class(t.hi);
            out.push_back(GridBatch{grid_fits(t.lo, own.logl) ? own : grid_search(t.lo, t.hi, kNttMaxLog), t.lo, t.hi, 0, i, i});
        }
        GridBatch &b = out.back();
        b.lo = std::min(b.lo, t.lo);
        b.n += t.n;
        b.end = i + 1;
    }
    return out;
}

// Ascending primes p[0 .. n), the first of them at `at`, as items of one class
// each, appended to out.
inline void grid_items(const uint64_t *p, size_t n, uint32_t at, std::vector<GridItem> &out) {
    for (size_t i = 0; i < n;) {
        const GridClass &g = grid_class(p[i]);
        size_t j = i;
        double sum = 0;
        while (j < n && grid_class(p[j]) == g) sum += (double)p[j++];
        out.push_back(GridItem{p[i], p[j - 1], (uint32_t)(j - i), at + (uint32_t)i, sum});
        i = j;
    }
}

}  // namespace wv
