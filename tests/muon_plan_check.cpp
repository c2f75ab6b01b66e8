// Host-only driver of tests/test_muon_plan.py: plans the products of lists of matrices and checks that every output tile is
// computed exactly once.  Exit code 0 = fine.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <tuple>
#include <vector>

#include "muon_plan.h"

using namespace adagc;

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); std::exit(1); } } while (0)

// Checks the launches of one product; returns the largest number of tiles of a workgroup.
static size_t check(MuonProduct product, const std::vector<MuonExtent>& extents)
{
    const std::vector<PlannedLaunch> launches = plan_muon_product(product, extents);
    std::vector<int> seen(extents.size(), 0);
    size_t most = 0;
    for (const PlannedLaunch& l : launches) {
        CHECK(l.side == 128 || l.side == 256);
        CHECK(l.workgroups > 0 && l.workgroups % 8 == 0 && l.workgroups <= (l.side == 256 ? 256 : 512));
        CHECK(l.first.size() == (size_t)l.workgroups + 1 && l.first[0] == 0 && l.first.back() == (int32_t)l.items.size());
        for (size_t b = 0; b + 1 < l.first.size(); ++b) {
            CHECK(l.first[b] <= l.first[b + 1]);
            most = std::max(most, (size_t)(l.first[b + 1] - l.first[b]));
        }
        std::map<std::tuple<int, int, int, int>, int> tiles;
        for (const GemmItem& i : l.items) ++tiles[std::make_tuple((int)i.group, (int)i.z, (int)i.tile_m, (int)i.tile_n)];
        size_t want = 0;
        for (size_t g = 0; g < l.groups.size(); ++g) {
            const MuonExtent& e = extents[(size_t)l.groups[g]];
            ++seen[(size_t)l.groups[g]];
            const int tn = e.mp / l.side, tm = product == MuonProduct::next ? e.np / l.side : tn;
            CHECK(tn * l.side == e.mp && (product != MuonProduct::next || tm * l.side == e.np));
            for (int z = 0; z < e.count; ++z)
                for (int m = 0; m < tm; ++m)
                    for (int n = 0; n < (product == MuonProduct::next ? tn : m + 1); ++n) {
                        CHECK((tiles[std::make_tuple((int)g, z, m, n)] == 1));
                        ++want;
                    }
        }
        CHECK(want == l.items.size());
    }
    for (int n : seen) CHECK(n == 1);
    return most;
}

// The sizes of the tiles of a product's launches, largest first, and the most tiles that a workgroup has.
static std::vector<int> sides(MuonProduct product, const std::vector<MuonExtent>& extents, size_t* most = nullptr)
{
    std::vector<int> out;
    for (const PlannedLaunch& l : plan_muon_product(product, extents)) out.push_back(l.side);
    if (most) *most = check(product, extents);
    return out;
}

int main()
{
    const MuonProduct products[] = {MuonProduct::gram, MuonProduct::poly, MuonProduct::next};
    std::mt19937 rng(7);
    auto draw = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    for (int round = 0; round < 300; ++round) {
        std::vector<MuonExtent> extents((size_t)draw(1, kMaxGroups));
        for (MuonExtent& e : extents) {
            e.mp = 128 * draw(1, round % 3 ? 6 : 16);
            e.np = e.mp + 128 * draw(0, 12);
            e.count = draw(1, 32);
        }
        for (MuonProduct p : products) check(p, extents);
    }
    // the smallest list; a long one of large matrices, whose work is spread evenly: 12 of 4096 x 14336, 8 of 4096 x 4096, 8 of
    // 1024 x 4096 have 2800 tiles for 256 workgroups in X X^T
    for (MuonProduct p : products) CHECK(check(p, {{128, 128, 1}}) == 1);
    CHECK(check(MuonProduct::gram, {{4096, 14336, 12}, {4096, 4096, 8}, {1024, 4096, 8}}) <= 20);
    // the tiles that the lists of tests/test_gpu_muon.py are there for
    const std::vector<int> small(1, 128), large(1, 256), both{256, 128};
    size_t most = 0;
    for (MuonProduct p : products) {
        CHECK(sides(p, {{768, 2304, 1}}) == small && sides(p, {{768, 2304, 32}}) == large);
        CHECK(sides(p, {{1280, 2560, 16}}) == large);
        CHECK(sides(p, {{128, 256, 1}, {128, 128, 1}, {256, 384, 1}, {384, 512, 1}, {512, 640, 1}}) == small);
        CHECK(sides(p, {{1408, 1536, 1}}) == small && sides(p, {{768, 1024, 1}}) == small && sides(p, {{640, 896, 1}}) == small);
    }
    CHECK(sides(MuonProduct::next, {{640, 1408, 20}}, &most) == small && most == 3);
    CHECK(sides(MuonProduct::next, {{768, 2304, 32}, {640, 1408, 3}}) == both);
    CHECK(sides(MuonProduct::next, {{256, 4096, 32}}) == large);
    CHECK(sides(MuonProduct::next, {{512, 4096, 32}}, &most) == large && most == 4);
    CHECK(sides(MuonProduct::next, {{4096, 14336, 1}}) == small && sides(MuonProduct::next, {{4096, 14336, 2}, {4096, 4096, 1}}) == large);
    std::printf("muon_plan_check: ok\n");
    return 0;
}
