// varcoef_launch.hpp -- host launchers of the variable-coefficient
// projection kernels (varcoef_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "flow_tile.hpp"

namespace pcx {
namespace vc {

// device scalar slots of the conjugate-gradient iteration
// (S_RZN: rz of the direction in use, S_RZ: of the one before it, so that
// the kernel that forms beta reads the one and stores the other)
enum { S_RZ, S_RZN, S_M, S_DRIFT, S_RES, S_BNORM, S_WTOT, S_PMEAN, NSC };

// what red_scal makes of the two reduced sums (S0, S1)
enum {
    MODE_MEAN,  // m = S0 / wtot
    MODE_BNORM, // bnorm = sqrt(S0); res = 1 (S0 itself when it is 0 or not finite); drift = 0
    MODE_RZ,    // rz = S0
    MODE_RES,   // drift = S0 / wtot; res = sqrt(S1 - drift S0) / bnorm
    MODE_PMEAN  // pmean = S0 / wtot
};

// Reductions: a partial-writing kernel stores the two sums of its workgroup
// b at part[b] and part[nb + b], and what needs the total sums them in a fixed
// order: red_scal (one workgroup) into the scalar slots, or every workgroup of
// the next kernel for itself, which costs it about a microsecond and spares
// two launches in the chain.  More than RED_MAX partials are first folded to
// RED_FOLD (launch_fold).
constexpr int RED_MAX = 1024, RED_FOLD = 256;
struct VRed {
    double *part; // 2 nb
    double *sc;   // NSC
    int nb;
    double *fold; // 2 RED_FOLD (nb > RED_MAX)
};

// Workgroups of the vector kernels: 256 cells each and round, RED_MAX at most;
// beyond 2^24 cells a workgroup for every 1024 consecutive cells (VCells).
inline int vec_wgs(size_t cells)
{
    if (cells > (size_t)1 << 24) return (int)((cells + 4 * flow::FT - 1) / (4 * flow::FT));
    const size_t n = (cells + flow::FT - 1) / flow::FT;
    return n < (size_t)RED_MAX ? (int)n : RED_MAX;
}

// Tiles of the operator: MAI x MAJ columns over chunks of ckc planes, each
// workgroup a plane in LDS.  A chunk starts with two extra planes, and 512
// workgroups (two per CU) run at once: the chunk length with the fewest
// planes marched in a row.
constexpr int MAI = 64, MAJ = 8, MAT = MAI * MAJ;
struct ATiles {
    int nti, ntj, ckc, n, wgs; // tiles, workgroups (a multiple of 8)
};
inline ATiles apply_tiles(const flow::FGrid &G)
{
    ATiles t{(G.n[0] + MAI - 1) / MAI, (G.n[1] + MAJ - 1) / MAJ, G.n[2], 0, 0};
    const long txy = (long)t.nti * t.ntj;
    long best = -1;
    for (int n = 1; n <= G.n[2]; ++n) {
        const int c = (G.n[2] + n - 1) / n;
        const long wgs = txy * ((G.n[2] + c - 1) / c), cost = (wgs + 511) / 512 * (c + 2);
        if (best < 0 || cost < best) { best = cost; t.ckc = c; }
    }
    t.n = (int)(txy * ((G.n[2] + t.ckc - 1) / t.ckc));
    t.wgs = t.n < RED_MAX ? (t.n + 7) / 8 * 8 : RED_MAX;
    return t;
}

using flow::FGrid;

using flow::TilePlan;

// out = sign D((1/rho_f) G p); with R (nb = T.wgs) partial sums of dzf p out
hipError_t launch_apply(const FGrid &G, const ATiles &T, const double *rho, const double *p, double *out, double sign,
                        const VRed *R, hipStream_t s);
hipError_t launch_rhs(const FGrid &G, const double *u, const double *v, const double *w, double idt, double *r, const VRed &R, hipStream_t s);
hipError_t launch_center(const FGrid &G, double *r, const VRed &R, hipStream_t s);
hipError_t launch_dinit(const FGrid &G, const double *r, const double *z, double *d, double rho0,
                        const VRed &R, hipStream_t s);
// IN: partials whose sum the kernel takes, R: the ones it writes
hipError_t launch_update(const FGrid &G, double *p, const double *d, double *r, const double *q, const VRed &IN,
                         const VRed &R, hipStream_t s);
hipError_t launch_dot(const FGrid &G, const double *r, const double *z, double rho0, const VRed &R, hipStream_t s);
// nv: the launch's workgroups (vec_wgs)
hipError_t launch_dupd(const FGrid &G, const double *z, double *d, double rho0, const VRed &IN, int nv, hipStream_t s);
hipError_t launch_pmean(const FGrid &G, const double *p, const VRed &R, hipStream_t s);
hipError_t launch_correct(const FGrid &G, const TilePlan &tp, const double *rho, const double *p, const double *u,
                          const double *v, const double *w, double dt, double *uo, double *vo, double *wo,
                          hipStream_t s);
hipError_t launch_pshift(const FGrid &G, double *p, const VRed &R, hipStream_t s);
// R, or its partials folded to RED_FOLD where they are more than RED_MAX
hipError_t launch_fold(const VRed &R, VRed &out, hipStream_t s);
// the sums of the partials and the scalar step `mode`; MODE_RES also stores
// the residual at *host (host memory the device can write)
hipError_t red_scal(const VRed &R, int mode, hipStream_t s, double *host = nullptr);

} // namespace vc
} // namespace pcx
