// Host-only check of the tile shapes the library chooses (no device call):
// a lone FP32 domain with walls takes the general passes where it has few
// fixed-plan tiles and the fixed ones where it has many; FP64, periodic
// directions, lengths with a much longer general plan and the domains of a
// batch take the fixed ones at any size.  Prints "ok" or the first failure
// and exits non-zero.
#include <cstdio>
#include <vector>

#include "pcx_fplan.hpp"
#include "pcx_plan.hpp"

static int check(int nx, int ny, int nz, int wall, int prec, bool lone, bool xfix, bool yfix)
{
    std::vector<double> zf(nz + 1);
    for (int k = 0; k <= nz; ++k) zf[k] = k;
    pcx_grid g{};
    g.nx = nx; g.ny = ny; g.nz = nz;
    g.lx = nx; g.ly = ny;
    g.zf = zf.data();
    g.bc_x = g.bc_y = g.bc_z = wall ? PCX_BC_WALL : PCX_BC_PERIODIC;
    pcx::Shapes sh;
    pcx::choose_shapes(g, prec, nullptr, sh, false, lone);
    const int csz = prec == pcx::PREC_F64 ? 16 : 8;
    const bool ok = (sh.xfix != 0) == xfix && (sh.yfix != 0) == yfix &&
                    (!xfix || sh.xth == pcx::fft_threads(nx / 2, csz)) && (!yfix || sh.yth == pcx::fft_threads(ny, csz)) &&
                    (xfix || sh.xth == 512) && (yfix || sh.yth == 256 || sh.yth == 512);
    if (!ok)
        std::printf("FAIL %d x %d x %d walls %d prec %d lone %d: fixed x %d (%d threads), y %d (%d)\n", nx, ny, nz, wall, prec,
                    (int)lone, sh.xfix, sh.xth, sh.yfix, sh.yth);
    return !ok;
}

int main()
{
    using pcx::PREC_F32;
    using pcx::PREC_F64;
    int bad = 0;
    for (bool lone : {false, true}) {
        bad += check(64, 64, 3, 1, PREC_F64, lone, true, true);
        bad += check(64, 64, 3, 0, PREC_F32, lone, true, true);
        bad += check(64, 64, 3, 1, PREC_F32, lone, !lone, !lone);
        bad += check(64, 64, 129, 1, PREC_F32, lone, true, true);
        bad += check(64, 64, 128, 1, PREC_F32, lone, !lone, true);
        bad += check(162, 81, 3, 1, PREC_F32, lone, true, true); // 81: four general stages, two fixed
        bad += check(512, 512, 48, 1, PREC_F32, lone, true, true);
        bad += check(8, 8, 64, 1, PREC_F32, lone, false, false); // no fixed plan
    }
    if (!bad) std::printf("ok\n");
    return bad != 0;
}
