// How the hot-column layout's row blocks are chosen and handed to workgroups
// (host only, no HIP).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <functional>
#include <queue>
#include <utility>
#include <vector>

namespace lilac {

// Row blocks: first row and first entry of each, and of the end.
struct HotCut {
    std::vector<int32_t> brow, bent;
    int32_t blocks() const { return (int32_t)brow.size() - 1; }
};

// What a block costs beside its entries, in entries: barriers and first loads
// (2^18 vertices, 4.7M edges, 17,000 entries a workgroup, a second block takes
// some 5 of 22 us), and a quarter for each row (8M vertices, 100M edges into
// 100,000 of them, with a row as one entry: blocks of 1.13 shares and empty rows
// apart 309 us a product, blocks of one share 292).
constexpr int64_t kHotBlockCost = 5000, kHotRowsAnEntry = 4;

// Blocks to workgroups: longest first, each to the least loaded workgroup so
// far (work = entries + rows).  Blocks differ a lot (the densest rows come first
// after relabelling), so taking every grid-th block leaves some workgroups a
// quarter more work than the mean.  Returns the cost of the heaviest workgroup.
inline int64_t hot_assign(const HotCut &cut, int32_t grid, std::vector<int32_t> &owner)
{
    const int32_t n = cut.blocks();
    auto work = [&](int32_t b) {
        return (int64_t)cut.bent[b + 1] - cut.bent[b] + (cut.brow[b + 1] - cut.brow[b]);
    };
    std::vector<int32_t> order((size_t)n);
    for (int32_t b = 0; b < n; ++b)
        order[b] = b;
    std::stable_sort(order.begin(), order.end(),
                     [&](int32_t a, int32_t b) { return work(a) > work(b); });
    typedef std::pair<int64_t, int32_t> Load;   // (work so far, workgroup)
    std::priority_queue<Load, std::vector<Load>, std::greater<Load>> least;
    for (int32_t g = 0; g < grid; ++g)
        least.push(Load(0, g));
    owner.assign((size_t)n, 0);
    std::vector<int64_t> cost((size_t)grid, 0);
    for (int32_t b : order) {
        Load l = least.top();
        least.pop();
        owner[b] = l.second;
        cost[l.second] += cut.bent[b + 1] - cut.bent[b] +
                          (cut.brow[b + 1] - cut.brow[b]) / kHotRowsAnEntry + kHotBlockCost;
        l.first += work(b);
        least.push(l);
    }
    return grid > 0 ? *std::max_element(cost.begin(), cost.end()) : 0;
}

// The blocks of a matrix whose rows take few of them: more entries to a block,
// from `target` up to twice that (few_targets), until no workgroup has two
// (PageRank, 20 iterations, 2^18 vertices, 4.7M edges, 298 and 254 blocks 550 and
// 451 us).  Blocks of empty rows alone end at their rows and do not get fewer (and
// blocks of entries then get too large: 8M vertices, 100,000 of them with 100M
// edges, the heaviest workgroup 3.9 times the mean), so where that is not reached,
// or at the price of a heavier workgroup than another try had, the try whose
// heaviest workgroup costs least is taken.  cut(i) gives the i-th try's blocks.
constexpr double kHotFewPrice = 1.25;

inline std::vector<int64_t> hot_few_targets(int64_t target)
{
    std::vector<int64_t> ts;
    for (int64_t t = target; t <= 2 * target; t += std::max<int64_t>(1, t / 32))
        ts.push_back(t);
    return ts;
}

inline HotCut hot_cut_few(size_t tries, int32_t cu, const std::function<HotCut(size_t)> &cut)
{
    HotCut best;
    int64_t least = -1;
    std::vector<int32_t> owner;
    for (size_t i = 0; i < tries; ++i) {
        HotCut c = cut(i);
        const bool one = c.blocks() <= cu;
        const int64_t cost = hot_assign(c, std::min(c.blocks(), cu), owner);
        const bool first = least < 0;
        if (first || cost < least || (one && (double)cost <= kHotFewPrice * (double)least))
            best = std::move(c);
        if (first || cost < least)
            least = cost;
        if (one)
            break;
    }
    return best;
}

}  // namespace lilac
