// Host-only check of the LDS the fixed-plan passes ask for (no device call):
// at every length and in both precisions and directions, what the tile takes
// and nothing more, so that as many tiles run per CU as there is room for.
// Prints "ok" or the first failure and exits non-zero.
#include <cstdio>

#include "pcx_fplan.hpp"
#include "pcx_plan.hpp"

int main()
{
    for (int n = 2; n <= 2 * pcx::FXMAX; ++n) {
        if (!pcx::fplan(n).n) continue;
        for (int prec : {pcx::PREC_F64, pcx::PREC_F32})
            for (int bc : {pcx::BC_PER, pcx::BC_WALL, pcx::BC_DIR}) {
                const int csz = prec == pcx::PREC_F64 ? 16 : 8;
                pcx::Dom d{};
                d.M = d.ny = n;
                d.xlines = d.ylines = pcx::fft_lines(n, csz);
                d.bcx = d.bcy = bc;
                if ((n <= pcx::FXMAX && pcx::lds_x(d, prec) != pcx::fft_lds(n, csz)) || pcx::lds_y(d, prec) != pcx::fft_lds(n, csz)) {
                    std::printf("FAIL %d points of %d bytes: x %zu, y %zu, the tile takes %zu\n", n, csz, pcx::lds_x(d, prec),
                                pcx::lds_y(d, prec), pcx::fft_lds(n, csz));
                    return 1;
                }
            }
    }
    std::printf("ok\n");
    return 0;
}
