// Host-only driver of tests/test_launch_rules.py: group_end (csrc/adagc_internal.h) of a full group's elements, a number of tensors and their
// elements on stdin; prints where each group ends.
#include <cstdio>
#include <vector>

#include "adagc_internal.h"

int main()
{
    long long most, n;
    if (std::scanf("%lld %lld", &most, &n) != 2) return 1;
    std::vector<adagc_tensor_desc> descs((size_t)n);
    for (adagc_tensor_desc& d : descs) {
        long long numel;
        if (std::scanf("%lld", &numel) != 1) return 1;
        d.numel = numel;
    }
    for (long long first = 0; first < n;) {
        first = adagc::group_end(descs.data(), n, first, most);
        std::printf("%lld ", first);
    }
    return 0;
}
