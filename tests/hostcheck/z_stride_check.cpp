// Host-only check of the z-line stride's rule (no device call): the stride
// holds a line, is whole 128-byte lines or nz itself, never takes more than
// half of nz as padding, and is padded wherever that takes at most a quarter.
// Prints "ok" or the first failure and exits non-zero.
#include <cstdio>

#include "pcx_dev.hpp"

int main()
{
    for (int zline : {8, 16})
        for (int nz = 2; nz <= 1024; ++nz) {
            const int zs = pcx::z_stride(nz, zline), up = (nz + zline - 1) / zline * zline;
            const bool ok = (zs == nz || zs == up) && 2 * zs <= 3 * nz && (4 * up > 5 * nz || zs == up);
            if (!ok) {
                std::printf("FAIL nz %d, %d elements a 128-byte line: stride %d\n", nz, zline, zs);
                return 1;
            }
        }
    std::printf("ok\n");
    return 0;
}
