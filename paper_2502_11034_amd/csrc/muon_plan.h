// Which workgroup computes which output tiles of the matrix-core products of Muon's Newton-Schulz steps (muon_gemm.hip).
// Plain C++, without HIP: planned once per context (adagc_muon_attach).
#ifndef ADAGC_MUON_PLAN_H
#define ADAGC_MUON_PLAN_H

#include <cstdint>
#include <vector>

#ifdef __HIP__
#define ADAGC_HOST_DEVICE __attribute__((host, device, always_inline)) inline
#else
#define ADAGC_HOST_DEVICE inline
#endif

namespace adagc {

// Tile b of a matrix, in an order in which tiles that follow one another form a patch a few tiles high and wide, so that the
// workgroups that run at the same time on an XCD share both operands in its L2.  SYM: the lower triangle in panels of kPanel
// tile columns, down the rows of a panel; otherwise panels of kPanelRows tile rows, along the columns.
template <bool SYM>
ADAGC_HOST_DEVICE void tile_of_matrix(int b, int tiles_m, int tiles_n, int* tile_m, int* tile_n)
{
    if constexpr (SYM) {
        constexpr int kPanel = 4;
        for (int c0 = 0;; c0 += kPanel) {
            const int rows = tiles_m - c0, cols = rows < kPanel ? rows : kPanel;
            const int n = cols * rows - cols * (cols - 1) / 2;
            if (b < n) {
                int r = 0;                                 // the panel's first rows have 1, 2, ... cols - 1 tiles
                while (r < cols - 1 && b > r) b -= ++r;
                const int full = r == cols - 1 ? b / cols : 0;
                *tile_m = c0 + r + full;
                *tile_n = c0 + b - full * cols;
                return;
            }
            b -= n;
        }
    } else {
        constexpr int kPanelRows = 8;
        const int per_panel = kPanelRows * tiles_n;
        const int first_m = b / per_panel * kPanelRows;
        const int rows = tiles_m - first_m < kPanelRows ? tiles_m - first_m : kPanelRows;
        const int i = b - first_m * tiles_n;
        *tile_m = first_m + i % rows;
        *tile_n = i / rows;
    }
}

// The three products of a Newton-Schulz step: a <- X X^T;  b <- b A + c A A;  x2 <- a X + B X.
enum class MuonProduct { gram, poly, next };

// count matrices of one padded shape: X is mp x np (mp <= np).
struct MuonExtent {
    int mp, np, count;
};

// An output tile: of matrix z of a group.
struct GemmItem {
    uint16_t group, z, tile_m, tile_n;
};

constexpr int kMaxGroups = 8;              // of one launch

// One launch over the groups whose tiles have this side.  Workgroup b computes items first[b] .. first[b + 1] - 1; `group` of an
// item is a place in `groups`, whose entries are places in the list of extents that was planned.
struct PlannedLaunch {
    int side = 0, workgroups = 0;
    std::vector<int>      groups;
    std::vector<GemmItem> items;
    std::vector<int32_t>  first;
    double                cost = 0;        // estimated, in microseconds
};

// The launches of a product over up to kMaxGroups groups: every tile in exactly one of them.
std::vector<PlannedLaunch> plan_muon_product(MuonProduct product, const std::vector<MuonExtent>& extents);

}  // namespace adagc
#endif
