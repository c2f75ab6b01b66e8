// Host-only driver of tests/test_launch_rules.py: one_launch_pays (csrc/adagc_internal.h) for lines of numbers on stdin: optimizer, bf16
// gradients, compute units, number of tensors, their elements; prints 0 or 1 for each.
#include <cinttypes>
#include <cstdio>

#include "adagc_internal.h"

using namespace adagc;

int main()
{
    int optimizer, bf16;
    int64_t compute_units, n;
    while (std::scanf("%d %d %" SCNd64 " %" SCNd64, &optimizer, &bf16, &compute_units, &n) == 4) {
        const int unroll = default_unroll(optimizer), items_per_chunk = default_items(unroll);
        LaunchShape s{0, 0, 0, 0, 0, true};
        int64_t numel[4096], elems = 0;
        for (int64_t i = 0; i < n; ++i) {
            if (n > 4096 || std::scanf("%" SCNd64, &numel[i]) != 1) return 1;
            elems += numel[i];
        }
        const int short_items = most_short_items(n, elems, items_per_chunk);
        for (int64_t i = 0; i < n; ++i) {
            const int64_t last = (numel[i] - 1) % kChunkElems + 1, chunks = (numel[i] + kChunkElems - 1) / kChunkElems;
            const ChunkKind kind = chunk_kind(last, items_per_chunk, unroll, short_items);
            s.n_long += chunks - (kind == kLongChunk ? 0 : 1);
            if (kind == kTinyChunk) ++s.n_tiny;
            if (kind == kShortChunk) s.n_short += chunk_items(last, items_per_chunk);
            s.n_full += numel[i] / kChunkElems;
            if (chunks > s.most_chunks) s.most_chunks = chunks;
            if (numel[i] > kChunkElems / items_per_chunk) s.alone = false;
        }
        std::printf("%d\n", one_launch_pays(optimizer, bf16 != 0, s, items_per_chunk, compute_units) ? 1 : 0);
    }
    return 0;
}
