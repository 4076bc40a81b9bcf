// Host-only check of the lists the autotuner times grouped launches on (no
// device call): they hold every tile of the pass, and no two items of the z
// solve, which works in place, are the same tile of the same copy; the copies
// take 64 MB or are 1024.  Prints "ok" or the first failure and exits
// non-zero.
#include <cstdio>
#include <set>
#include <utility>

#include "pcx_tune.hpp"

int main()
{
    using namespace pcx;
    for (size_t bytes : {(size_t)1024, (size_t)100000, (size_t)1 << 20, (size_t)50 << 20, (size_t)3 << 30}) {
        const int c = tune_z_copies(bytes);
        if (c < 1 || c > 1024 || (c < 1024 && c * bytes < (size_t)64 << 20) || (c > 1 && (c - 1) * bytes >= (size_t)64 << 20)) {
            std::printf("FAIL %zu bytes: %d copies\n", bytes, c);
            return 1;
        }
    }
    for (int kind : {(int)PK_Z, (int)PK_YF, (int)PK_XINV_STORE})
        for (long t : {1, 7, 600, 1023, 1024, 5000})
            for (int copies : {1, 3, 200}) {
                std::set<std::pair<unsigned, unsigned>> seen;
                std::set<unsigned> tiles;
                const std::vector<GItem> v = tune_items(kind, t, copies);
                for (const GItem &i : v) {
                    seen.insert({i.dom, i.tile});
                    tiles.insert(i.tile);
                }
                const bool z = kind == PK_Z;
                const bool ok = (long)tiles.size() == t && *tiles.rbegin() == t - 1 && (long)v.size() % t == 0 &&
                                (z ? seen.size() == v.size() && (long)v.size() == t * copies && (int)seen.rbegin()->first == copies - 1
                                   : (long)v.size() + t > GFILL && seen.rbegin()->first == 0);
                if (!ok) {
                    std::printf("FAIL pass %d of %ld tiles, %d copies: %zu items, %zu different\n", kind, t, copies, v.size(), seen.size());
                    return 1;
                }
            }
    std::printf("ok\n");
    return 0;
}
