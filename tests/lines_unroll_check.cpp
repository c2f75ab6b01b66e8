// Host-only driver of tests/test_launch_rules.py: the numbers of vectors in flight for which an optimizer's update kernel can walk whole
// lines (lines_with_unroll, csrc/walk_lines.h), AdamW's and then Lion's.
#include <cstdio>

#include "adagc_internal.h"

int main()
{
    for (int optimizer : {ADAGC_OPT_ADAMW, ADAGC_OPT_LION})
        for (int unroll : {1, 2, 4}) std::printf("%d%s", adagc::lines_with_unroll(optimizer, unroll) ? 1 : 0, unroll == 4 ? "\n" : " ");
    return 0;
}
