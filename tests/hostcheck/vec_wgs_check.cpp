// Host-only check of the projection's vector launches (no device call): up to
// 2^24 cells as many workgroups as the reductions take without folding, beyond
// it one for every 1024 cells, always enough for the grid and within the
// launch limits.  Prints "ok" or the first failure and exits non-zero.
#include <cstdio>

#include "varcoef_launch.hpp"

int main()
{
    using namespace pcx::vc;
    const size_t big = (size_t)1 << 24;
    for (size_t n : {(size_t)8, (size_t)256, (size_t)257, (size_t)1 << 18, ((size_t)1 << 18) + 1, big - 1, big, big + 1, big + 1024,
                     big + 1025, (size_t)134217728, (size_t)2147483647}) {
        const long w = vec_wgs(n);
        const bool ok = n > big ? w > RED_MAX && (size_t)w * 1024 >= n && (size_t)(w - 1) * 1024 < n && w < (1L << 22)
                                : w >= 1 && w <= RED_MAX && (w == RED_MAX || (size_t)w * 256 >= n);
        if (!ok) {
            std::printf("FAIL %zu cells: %ld workgroups\n", n, w);
            return 1;
        }
    }
    std::printf("ok\n");
    return 0;
}
