// Order and groups of a batch's instances (host only).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <numeric>
#include <vector>

namespace mc {

struct PlanItem {
    int32_t M, kind;
    int64_t dim, tiles;
    bool own;   // has a launch of its own
};

// Sorted positions first .. first + count - 1, all of one orbital count and kind.
struct PlanGroup {
    int32_t M, kind, first, count;
    int64_t tiles;
};

// Sorts the items (sorted[j]: caller index) by orbital count, kind, whether they
// join a group, and decreasing dimension, and makes the groups; prefix[j] is the
// first tile of sorted position j within its group.  A group is addressed as
// consecutive positions, so an instance with a launch of its own must not lie
// between two of its members: it does not suffice to sort by dimension, since
// the kernel that such an instance takes has an upper and a lower limit.
inline std::vector<PlanGroup> plan_groups(const std::vector<PlanItem> &items,
                                          std::vector<int32_t> &sorted,
                                          std::vector<int64_t> &prefix)
{
    sorted.resize(items.size());
    std::iota(sorted.begin(), sorted.end(), 0);
    std::stable_sort(sorted.begin(), sorted.end(), [&](int a, int b) {
        const PlanItem &x = items[a], &y = items[b];
        if (x.M != y.M) return x.M < y.M;
        if (x.kind != y.kind) return x.kind < y.kind;
        if (x.own != y.own) return y.own;
        return x.dim > y.dim;
    });
    prefix.assign(items.size() + 1, 0);
    std::vector<PlanGroup> groups;
    for (size_t j = 0; j < sorted.size(); ++j) {
        const PlanItem &t = items[sorted[j]];
        if (t.own) continue;
        if (groups.empty() || groups.back().M != t.M || groups.back().kind != t.kind)
            groups.push_back(PlanGroup{t.M, t.kind, (int32_t)j, 0, 0});
        PlanGroup &g = groups.back();
        prefix[j] = g.tiles;
        g.tiles += t.tiles;
        ++g.count;
    }
    return groups;
}

}  // namespace mc
