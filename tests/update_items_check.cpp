// Host-only driver of tests/test_launch_rules.py: update_items (csrc/adagc_internal.h) for lines of optimizer, unroll, update_split, grid_blocks and elements on
// stdin;
// prints the vectors in flight, the work items of a chunk and the most elements in full ones of a list whose rule is in the update kernel.
#include <cstdio>

#include "adagc_internal.h"

int main()
{
    int optimizer, unroll, split, grid;
    long long elems;
    while (std::scanf("%d %d %d %d %lld", &optimizer, &unroll, &split, &grid, &elems) == 5) {
        const adagc::UpdateItems u = adagc::update_items(optimizer, unroll, split, grid, elems);
        std::printf("%d %d %lld\n", u.unroll, u.per_chunk,
                    (long long)(adagc::fused_max_items(optimizer, u.per_chunk, grid) * (adagc::kChunkElems / u.per_chunk)));
    }
    return 0;
}
