// Host-only driver of tests/test_walk_lines.py: evaluates csrc/walk_lines.h for lines of eight numbers on stdin (optimizer,
// bf16 gradients, copy, tensors, elements, elements of tensors that start off a line, workgroups, work items), printing 0 or 1 for each.
#include <cinttypes>
#include <cstdio>

#include "walk_lines.h"

int main()
{
    int opt, bf16, copy;
    int64_t tensors, elems, off, workgroups, items;
    while (std::scanf("%d %d %d %" SCNd64 " %" SCNd64 " %" SCNd64 " %" SCNd64 " %" SCNd64, &opt, &bf16, &copy, &tensors, &elems, &off,
                      &workgroups, &items) == 8)
        std::printf("%d\n", adagc::walk_lines(opt, bf16 != 0, copy != 0, tensors, elems, off, workgroups, items) ? 1 : 0);
    return 0;
}
