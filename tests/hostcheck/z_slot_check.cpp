// Host-only check of the z solve's LDS slots (no device call): for every
// number of levels and every lane split, a wave's stores to S2 (whole padded
// lines) read slots of its own lines only, slots it staged and wrote, and no
// slot lies past the tile's LDS.  Prints "ok" or the first failure and exits
// non-zero.
#include <cstdio>
#include <vector>

#include "pcx_dev.hpp"

using namespace pcx;

static int check(int nz, int G, int pad)
{
    const int lpw = 64 / G, lines = (NT / 64) * lpw, ls = (nz + G - 1) / G * G, zs = (nz + pad - 1) / pad * pad;
    const int room = lines * ls + lines * ls / 16 + 1; // elements of LDS (lds_z)
    std::vector<int> owner(room, -1);
    for (int line = 0; line < lines; ++line)
        for (int k = 0; k < nz; ++k) {
            const int q = z_slot(line, k, ls);
            if (q < 0 || q >= room || owner[q] >= 0) {
                std::printf("FAIL slot of line %d level %d: nz %d lanes %d\n", line, k, nz, G);
                return 1;
            }
            owner[q] = line;
        }
    for (int line = 0; line < lines; ++line)
        for (int k = 0; k < zs; ++k) {
            const int q = z_out_slot(line, k, ls, nz);
            if (q < 0 || q >= room || owner[q] != line || (k < nz && q != z_slot(line, k, ls))) {
                std::printf("FAIL element %d of line %d (wave %d) stored from a slot of line %d: nz %d lanes %d\n", k, line,
                            line / lpw, q < 0 || q >= room ? -1 : owner[q], nz, G);
                return 1;
            }
        }
    return 0;
}

int main()
{
    for (int nz = 2; nz <= 1024; ++nz)
        for (int G = 1; G <= 64; G *= 2) {
            if ((nz + G - 1) / G > 16 || (G > 1 && 2 * G > nz)) continue;
            for (int pad : {1, 8, 16})
                if (check(nz, G, pad)) return 1;
        }
    std::printf("ok\n");
    return 0;
}
