// Host-only check of the marching passes' chunk rule (no device call): the
// chunk is the cheapest in rounds of workgroups times the planes each takes
// of those allowed; the grids whose times the rule was taken from.  Prints "ok" or the first
// failure and exits non-zero.
#include <cstdio>

#include "pcx_plan.hpp"

int main()
{
    for (int nz = 2; nz <= 1024; nz = nz < 40 ? nz + 1 : nz + 23)
        for (long txy : {1, 2, 7, 32, 100, 255, 256, 257, 511, 512, 513, 1500, 2048, 9000})
            for (int occ : {1, 2})
                for (int most : {64, nz}) {
                    const int c = pcx::march_chunk(nz, txy, occ, most);
                    auto rounds = [&](int k) { return (txy * ((nz + k - 1) / k) + 256 * occ - 1) / (256 * occ); };
                    auto may = [&](int k) { return k <= most || (k == nz && (nz <= 128 || rounds(k) >= 4)); };
                    bool ok = c >= 1 && c <= nz && may(c);
                    for (int n = 1; ok && n <= nz; ++n) {
                        const int k = (nz + n - 1) / n;
                        if (may(k)) ok = rounds(c) * (c + 3) <= rounds(k) * (k + 3);
                    }
                    if (!ok) {
                        std::printf("FAIL %d planes, %ld tiles, %d per CU, chunks up to %d: %d\n", nz, txy, occ, most, c);
                        return 1;
                    }
                }
    const struct { int nz; long txy; int occ, most, want; } at[] = {
        {512, 512, 2, 64, 64}, {512, 256, 1, 512, 512}, {512, 2048, 2, 64, 512}, {100, 512, 2, 64, 100},
        {256, 128, 2, 64, 64}, {384, 768, 2, 64, 64},   {32, 2, 2, 64, 1},       {75, 42, 2, 64, 7},
        {384, 288, 2, 64, 55}};
    for (const auto &q : at) {
        const int c = pcx::march_chunk(q.nz, q.txy, q.occ, q.most);
        if (c != q.want) {
            std::printf("FAIL %d planes, %ld tiles: %d, not %d\n", q.nz, q.txy, c, q.want);
            return 1;
        }
    }
    std::printf("ok\n");
    return 0;
}
