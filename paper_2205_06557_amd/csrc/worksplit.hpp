// worksplit.hpp -- host side: how the symmetric all-pairs sum of one system
// is cut into work items (pair_sym_kernel, pair_sym_batch_kernel).  Kept
// apart from the rest of the host code because, with the kernels, it fixes
// what the pair phase reads and writes.
#pragma once

#include <algorithm>
#include <cmath>
#include <vector>

#include "symitems.hpp"

namespace {

constexpr double kSymItemsTarget = 65536.0;    // work items of the symmetric sum
constexpr double kSymMinGroupedItems = 2048.0; // fewer grouped items: one target row per item
constexpr double kSymMinItems = 1024.0;        // fewer one-tile items: one item per 64-ion sub-tile

// Items of the runs.
inline int sym_count(const odk::SymRuns& s)
{
    odk::SymPlace at{0, 0};
    odk::SymItem it{};
    (void)odk::sym_item_at(s, 1 << 30, at, it);
    return at.before;
}

// Work items of the symmetric sum of one system of T tiles: groups of
// kSymRows target tile rows, each group with runs of at most C source tiles
// from its first row on (rows left over at the end alone), C chosen for about
// kSymItemsTarget items.  Where grouping leaves fewer than kSymMinGroupedItems
// items (small systems, too few to fill the chip), one target row per item
// instead; where even one tile pair per item leaves fewer than kSymMinItems
// (up to 11,500 ions), each tile pair is cut into its four 64-ion source
// sub-tiles, so that a step's pair sum is not one long chain per block (whole
// tiles against sub-tiles: 37 / 32 us at 8,192 ions, 46 / 38 at 10,000, 55 /
// 63 at 12,345).  The
// split depends on T only, so a system's sums are grouped the same way alone
// and in a batch.  one_row: one target row per item at every size; target:
// the number of items aimed at (batch options; both change the FP32 partial
// sums that each item flushes).
inline odk::SymRuns sym_runs(int T, bool one_row = false, double target = kSymItemsTarget)
{
    constexpr int R = odk::kSymRows;
    const double pairs = 0.5 * (double)T * (T + 1);
    const odk::SymRuns groups{T, R, (int)std::max((double)R, std::ceil(pairs / (R * target)))};
    if (!one_row && (double)sym_count(groups) >= kSymMinGroupedItems) return groups;
    return {T, 1, (int)std::max(1.0, std::ceil(pairs / target))};
}

// Whether the runs, one tile each, are to be cut into sub-tiles.
inline bool sym_cut(const odk::SymRuns& s)
{
    return s.rows == 1 && s.C == 1 && 0.5 * (double)s.T * (s.T + 1) < kSymMinItems;
}

std::vector<odk::SymItem> sym_items_of(int T, bool one_row = false, double target = kSymItemsTarget)
{
    const odk::SymRuns runs = sym_runs(T, one_row, target);
    const bool sub = sym_cut(runs);
    std::vector<odk::SymItem> v;
    v.reserve((size_t)sym_count(runs) * (sub ? 4 : 1));
    odk::SymPlace at{0, 0};
    odk::SymItem it{};
    for (int k = 0; odk::sym_item_at(runs, k, at, it); ++k)
        for (int st = 0; st < 4; st += sub ? 1 : 4) v.push_back({it.I, it.J0, it.J1, it.rows, st, sub ? st + 1 : 4});
    return v;
}

// Length of sym_items_of(T).
inline int sym_items_count(int T)
{
    const odk::SymRuns runs = sym_runs(T);
    return sym_count(runs) * (sym_cut(runs) ? 4 : 1);
}

// Work of an item: target rows times 64-ion source sub-tiles.
inline long long sym_item_cost(int rows, int J0, int J1, int st0, int st1)
{
    return (long long)rows * (J1 - J0) * (st1 - st0);
}
inline long long sym_item_cost(const odk::SymItem& a) { return sym_item_cost(a.rows, a.J0, a.J1, a.st0, a.st1); }

// Longest items first, so that the short ones fill the tail; items of one
// length in their order.  By counting, since creating a system waits for it
// (28,000 ions: 0.3 ms with a comparison sort).
std::vector<odk::SymItem> sym_items(int T)
{
    const std::vector<odk::SymItem> v = sym_items_of(T);
    long long most = 0;
    for (const odk::SymItem& q : v) most = std::max(most, sym_item_cost(q));
    std::vector<size_t> at((size_t)most + 2, 0);        // at[k]: items longer than most - k
    for (const odk::SymItem& q : v) ++at[(size_t)(most - sym_item_cost(q)) + 1];
    for (size_t k = 1; k < at.size(); ++k) at[k] += at[k - 1];
    std::vector<odk::SymItem> o(v.size());
    for (const odk::SymItem& q : v) o[at[(size_t)(most - sym_item_cost(q))]++] = q;
    return o;
}

}  // namespace
