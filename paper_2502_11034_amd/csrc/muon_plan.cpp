#include "muon_plan.h"

#include <algorithm>
#include <functional>
#include <queue>
#include <utility>

namespace adagc {
namespace {

constexpr int kXcds = 8, kDepth = 64;      // dies with an L2 each (workgroup b runs on die b mod 8); k per operand tile

// What a tile takes, in microseconds: per operand tile, and for its first loads and its results.  A 256-tile has a compute unit
// for itself; of 128-tiles a unit holds one, or two that share it.
struct Cost {
    double step, ends;
};
Cost cost_of(MuonProduct product, int side, bool two)
{
    const bool next = product == MuonProduct::next;
    if (side == 256) return {1.25, next ? 14.0 : 10.0};
    return two ? Cost{0.68, next ? 9.5 : 7.5} : Cost{0.30, 5.0};
}
constexpr double kLaunch = 3.0;

struct Shape {
    int group;                             // place in the extents
    int tiles_m, tiles_n, depth;           // depth: operand tiles
    int64_t tiles;
};

Shape shape_of(MuonProduct product, const MuonExtent& e, int group, int side)
{
    Shape s;
    s.group = group;
    s.tiles_n = e.mp / side;
    s.tiles_m = product == MuonProduct::next ? e.np / side : s.tiles_n;
    s.depth = (product == MuonProduct::gram ? e.np : e.mp) / kDepth;
    s.tiles = product == MuonProduct::next ? (int64_t)s.tiles_m * s.tiles_n : (int64_t)s.tiles_n * (s.tiles_n + 1) / 2;
    return s;
}

// The tiles of the groups, deepest first, are dealt to the XCDs in runs of consecutive ones, one for each of an XCD's places, so that
// the whole chip is on one or two matrices at a time; what is left of a group in equal parts, the larger ones to the XCDs that
// have least to do.  Within an XCD every tile goes to the place that is free first.  A launch over all groups so pays one
// partly filled round, and that with its shortest tiles.
PlannedLaunch plan_launch(MuonProduct product, const std::vector<MuonExtent>& extents, const std::vector<int>& groups, int side)
{
    PlannedLaunch plan;
    plan.side = side;
    std::vector<Shape> shapes;
    int64_t all = 0;
    for (int g : groups) {
        shapes.push_back(shape_of(product, extents[(size_t)g], g, side));
        all += shapes.back().tiles * extents[(size_t)g].count;
    }
    std::stable_sort(shapes.begin(), shapes.end(), [](const Shape& a, const Shape& b) { return a.depth > b.depth; });
    const bool two = side == 128 && all > kXcds * 32;                  // two workgroups per compute unit
    const int places = two ? 64 : 32;
    const Cost tile = cost_of(product, side, two);

    std::vector<GemmItem> of_xcd[kXcds];
    double load[kXcds] = {};
    for (size_t s = 0; s < shapes.size(); ++s) {
        const Shape& sh = shapes[s];
        plan.groups.push_back(sh.group);
        const double cost = sh.depth * tile.step + tile.ends;
        const int64_t total = sh.tiles * extents[(size_t)sh.group].count;
        auto deal = [&](int xcd, int64_t from, int64_t to) {
            for (int64_t t = from; t < to; ++t) {
                const int64_t z = t / sh.tiles;
                int m, n;
                if (product == MuonProduct::next) tile_of_matrix<false>((int)(t - z * sh.tiles), sh.tiles_m, sh.tiles_n, &m, &n);
                else tile_of_matrix<true>((int)(t - z * sh.tiles), sh.tiles_m, sh.tiles_n, &m, &n);
                of_xcd[xcd].push_back(GemmItem{(uint16_t)s, (uint16_t)z, (uint16_t)m, (uint16_t)n});
            }
            load[xcd] += cost * (double)(to - from);
        };
        int64_t t = 0;
        for (; t + kXcds * places <= total; t += kXcds * places)
            for (int x = 0; x < kXcds; ++x) deal(x, t + x * places, t + (x + 1) * places);
        int order[kXcds];
        for (int x = 0; x < kXcds; ++x) order[x] = x;
        std::stable_sort(order, order + kXcds, [&](int a, int b) { return load[a] < load[b]; });
        const int64_t left = total - t;
        for (int i = 0; i < kXcds; ++i) {
            const int64_t n = left / kXcds + (i < left % kXcds ? 1 : 0);
            deal(order[i], t, t + n);
            t += n;
        }
    }
    size_t longest = 0;
    for (const auto& items : of_xcd) longest = std::max(longest, items.size());
    const int used = (int)std::min<size_t>((size_t)places, longest);
    plan.workgroups = kXcds * used;

    std::vector<std::vector<GemmItem>> of_workgroup((size_t)plan.workgroups);
    for (int x = 0; x < kXcds; ++x) {
        typedef std::pair<double, int> Free;                               // when, and which place
        std::priority_queue<Free, std::vector<Free>, std::greater<Free>> free;
        for (int p = 0; p < used; ++p) free.push(Free(0.0, p));
        for (const GemmItem& item : of_xcd[x]) {
            const Free f = free.top();
            free.pop();
            of_workgroup[(size_t)(f.second * kXcds + x)].push_back(item);
            const double until = f.first + shapes[item.group].depth * tile.step + tile.ends;
            free.push(Free(until, f.second));
            plan.cost = std::max(plan.cost, until);
        }
    }
    plan.cost += kLaunch;
    for (const auto& items : of_workgroup) {
        plan.first.push_back((int32_t)plan.items.size());
        plan.items.insert(plan.items.end(), items.begin(), items.end());
    }
    plan.first.push_back((int32_t)plan.items.size());
    return plan;
}

}  // namespace

// The size of the tiles is chosen for the launch, by the estimate.  Measured, all on 128-tiles against 256-tiles where they fit, in
// microseconds:
//   24 of 768 x 3072, 12 of 768 x 2304, 12 of 768 x 768    gram 74 / 77        poly 35 / 52        next 194 / 178
//   16 of 1024 x 4096, 8 of 1024 x 3072, 8 of 1024 x 1024  gram 110 / 105      poly 48 / 63        next 272 / 225
//   6 of 2048 x 2560                                       gram 78 / 62        poly 61 / 54        next 129 / 108
//   1 of 1024 x 4096                                       gram 30 / 75        poly 11 / 28        next 15 / 28
//   12 of 4096 x 14336, 8 of 4096 x 4096, 8 of 1024 x 4096 gram 3956 / 2638    poly 1459 / 1184    next 8039 / 5220
// The estimate takes the faster side everywhere but in X X^T of the first list (75 / 73 estimated: 256-tiles, 3 us slower).  It knows
// nothing of operand traffic, and is far too low for large matrices on 128-tiles (a X + B X of the last list 5387).
// A launch for each group instead of one for all: 141 against 77, 85 against 52 and 185 against 178 on the first list (256-tiles),
// 2801 against 2638, 1238 against 1184 and 5080 against 5220 on the last.
std::vector<PlannedLaunch> plan_muon_product(MuonProduct product, const std::vector<MuonExtent>& extents)
{
    std::vector<int> everything, large, rest;
    for (int g = 0; g < (int)extents.size(); ++g) {
        const MuonExtent& e = extents[(size_t)g];
        everything.push_back(g);
        const bool fits = e.mp % 256 == 0 && (product != MuonProduct::next || e.np % 256 == 0);
        (fits ? large : rest).push_back(g);
    }
    std::vector<PlannedLaunch> small(1, plan_launch(product, extents, everything, 128));
    if (large.empty()) return small;
    std::vector<PlannedLaunch> mixed(1, plan_launch(product, extents, large, 256));
    if (!rest.empty()) mixed.push_back(plan_launch(product, extents, rest, 128));
    double cost = 0;
    for (const PlannedLaunch& p : mixed) cost += p.cost;
    return cost < small[0].cost ? mixed : small;
}

}  // namespace adagc
