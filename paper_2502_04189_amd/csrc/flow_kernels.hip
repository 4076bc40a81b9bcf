// flow_kernels.hip -- kernels of the Runge-Kutta substep around the pressure
// correction: normals, regularization flux and curvature, phase-field
// update, momentum predictor, on the tiles of flow_tile.hpp: the flux of the
// interior box and the momentum pass march in z, the others take one thread
// per cell; interior tiles on code without wall rules.
#include <algorithm>

#include "flow_launch.hpp"
#include "flow_tile.hpp"

namespace pcx {
namespace flow {

// every output of these kernels is streamed: written once, read by a later
// kernel only, so it is stored non-temporally (it does not evict the
// neighbour values other workgroups of the same kernel still read)
__device__ __forceinline__ void put(double *p, double v) { __builtin_nontemporal_store(v, p); }
// inputs read at their own cell only (previous right-hand sides, pressures)
__device__ __forceinline__ double own(const double *p) { return __builtin_nontemporal_load(p); }

// psi of every cell (one logarithm per cell), then the normals from it
__global__ __launch_bounds__(FT) void k_flow_psi(FArgs A)
{
    const size_t n = (size_t)A.G.n[0] * A.G.n[1] * A.G.n[2];
    const size_t c = (size_t)blockIdx.x * FT + threadIdx.x;
    if (c < n) put(A.psi + c, psi_of(A.P, A.phi[c]));
}

// the normals on the tiles along the walls (the interior tiles' flux kernel
// evaluates its own)
__global__ __launch_bounds__(FT) void k_flow_normals(BoxList L, FArgs A)
{
    const BoxPick p = box_pick(L);
    const FTile t = btile(A.G, p.b, p.w);
    if (!t.act) return;
    double nx, ny, nz;
    normal_cell(Gen{A.G, t.i, t.j, t.k}, A.psi, nx, ny, nz);
    const size_t c = at(A.G, t.i, t.j, t.k);
    put(A.n[0] + c, nx);
    put(A.n[1] + c, ny);
    put(A.n[2] + c, nz);
}

// Regularization flux and curvature on the tiles along the walls, from the
// stored normals (their own tiles' by k_flow_normals, an interior
// neighbour's by k_flow_flux_in)
__global__ __launch_bounds__(FT) void k_flow_flux_wall(BoxList L, FArgs A)
{
    const BoxPick p = box_pick(L);
    const FTile t = btile(A.G, p.b, p.w);
    if (!t.act) return;
    const size_t c = at(A.G, t.i, t.j, t.k);
    const PVec n{A.n[0], A.n[1], A.n[2]};
    const Gen x{A.G, t.i, t.j, t.k};
    put(A.a[0] + c, flux_face<0>(x, A.P, A.phi, A.psi, A.n[0]));
    put(A.a[1] + c, flux_face<1>(x, A.P, A.phi, A.psi, A.n[1]));
    put(A.a[2] + c, flux_face<2>(x, A.P, A.phi, A.psi, A.n[2]));
    put(A.kap + c, curvature_cell(x, n));
}

// The flux and curvature on the interior box (planes from 2 on with walls in
// z), marching in z: a workgroup takes MFI x MFJ columns over a chunk of
// planes, keeps four planes of psi and three of phi in LDS (tile and halo)
// and evaluates each normal once, one plane ahead of the flux that uses it:
// n of the own cell stays in registers, its x and y components go through
// LDS for the in-plane neighbours, and the cells just outside the tile (144
// of them for 512 threads) are evaluated by the first waves.  Evaluating the
// seven normals a cell reads at every cell took 481 VALU instructions per
// cell and 3.1 ms at 512^3; here 1.61 ms, of which the six fields it moves
// take 1.24 ms at copy rate.  One barrier per plane: a plane of LDS is
// written no earlier than a barrier after its last read.
constexpr int MFI = 64, MFJ = 8, MFT = MFI * MFJ;
constexpr int PSX = MFI + 4, PSY = MFJ + 4, PSN = PSX * PSY; // psi plane: two cells of halo
constexpr int PHX = MFI + 1, PHY = MFJ + 1, PHN = PHX * PHY; // phi plane: one cell up in x and y
constexpr int NXX = MFI + 2, NXN = NXX * MFJ;                // n_x: one cell of halo in x
constexpr int NYN = MFI * (MFJ + 2);                         // n_y: one in y
constexpr int MFR = 2 * (MFI + MFJ);                         // halo cells whose normal is evaluated
static_assert(PSN <= 2 * MFT && PHN <= 2 * MFT && MFR <= MFT, "two items per thread");

// uniform entry of a table no kernel writes, by a scalar load
__device__ __forceinline__ double utab(const double *p, int k)
{
    return ((const __attribute__((address_space(4))) double *)p)[__builtin_amdgcn_readfirstlane(k)];
}

__global__ __launch_bounds__(MFT) void k_flow_flux_in(TileBox b, int ckc, FArgs A)
{
    __shared__ double sps[4][PSN], sph[3][PHN], snx[2][NXN], sny[2][NYN];
    const FGrid &G = A.G;
    const int nx = G.n[0], ny = G.n[1], nz = G.n[2];
    const size_t sz = (size_t)nx * ny;
    // tile of this workgroup, an XCD's workgroups a contiguous range
    const int i1 = min((b.it0 + b.nit) * FTI, nx), j1 = min((b.jt0 + b.njt) * FTJ, ny);
    const int ntj = (j1 - b.jt0 * FTJ + MFJ - 1) / MFJ, nch = (b.nk + ckc - 1) / ckc;
    const int ntile = b.nit * ntj * nch, per = (ntile + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || tile >= ntile) return;
    const int ch = tile / (b.nit * ntj), rem = tile - ch * (b.nit * ntj), jt = rem / b.nit;
    const int i0 = (b.it0 + rem - jt * b.nit) * FTI, j0 = b.jt0 * FTJ + jt * MFJ;
    const int kb = b.k0 + ch * ckc, ke = min(b.k0 + b.nk, kb + ckc);
    const int tid = threadIdx.x, tx = tid & (MFI - 1), ty = tid / MFI;
    const int i = i0 + tx, j = j0 + ty;
    const bool act = i < i1 && j < j1;
    // in-plane offset of cell (i0 + a, j0 + c): wrapped once across a
    // periodic direction; past a partial tile any valid cell
    auto off = [&](int a, int c) {
        int x = i0 + a, y = j0 + c;
        x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
        y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
        return (size_t)min(max(y, 0), ny - 1) * nx + min(max(x, 0), nx - 1);
    };
    auto wrapk = [&](int k) { return k < 0 ? k + nz : (k >= nz ? k - nz : k); };
    // the thread's items of a psi and of a phi plane
    const int q1 = min(tid + MFT, PSN - 1), r1 = min(tid + MFT, PHN - 1);
    const size_t o0 = off(tid % PSX - 2, tid / PSX - 2), o1 = off(q1 % PSX - 2, q1 / PSX - 2);
    const int r0 = min(tid, PHN - 1);
    const size_t h0 = off(r0 % PHX, r0 / PHX), h1 = off(r1 % PHX, r1 / PHX);
    const double hx = 0.5 * G.ih[0], hy = 0.5 * G.ih[1];
    const int me = (ty + 2) * PSX + tx + 2; // own cell in a psi plane
    // the halo cell whose normal this thread evaluates: rows j0 - 1 and j0 +
    // MFJ (its y component), then columns i0 - 1 and i0 + MFI (its x component)
    const bool ring = tid < MFR, ry = tid < 2 * MFI;
    const int rq = tid - 2 * MFI;
    const int rj = ry ? (tid < MFI ? -1 : MFJ) : (rq & (MFJ - 1)), ri = ry ? tx : (rq < MFJ ? -1 : MFI);
    const int rme = ring ? (rj + 2) * PSX + ri + 2 : me;
    const int rdst = ry ? (rj + 1) * MFI + ri : rj * NXX + ri + 1;
    // normal at place c of the plane k (psi planes k - 1, k, k + 1 in LDS)
    auto normal = [&](int c, int k, double iz, double &ux, double &uy, double &uz) {
        const double *p = sps[k & 3];
        unit_normal((p[c + 1] - p[c - 1]) * hx, (p[c + PSX] - p[c - PSX]) * hy,
                    (sps[(k + 1) & 3][c] - sps[(k - 1) & 3][c]) * iz, ux, uy, uz);
    };
    auto halo_normal = [&](int k, double iz) {
        if (!ring) return;
        double ux, uy, uz;
        normal(rme, k, iz, ux, uy, uz);
        if (ry) sny[k & 1][rdst] = uy;
        else snx[k & 1][rdst] = ux;
    };
    auto iz2 = [&](int k) { return utab(G.rz, 6 * wrapk(k) + 4); };
    // prologue: psi of planes kb - 2 .. kb + 1, phi of kb
    {
        double p[4][2];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double *s = A.psi + (size_t)wrapk(kb - 2 + q) * sz;
            p[q][0] = s[o0];
            p[q][1] = s[o1];
        }
        const double *f = A.phi + (size_t)wrapk(kb) * sz;
        const double f0 = f[h0], f1 = f[h1];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            sps[(kb - 2 + q) & 3][tid] = p[q][0];
            if (tid + MFT < PSN) sps[(kb - 2 + q) & 3][tid + MFT] = p[q][1];
        }
        sph[kb % 3][r0] = f0;
        if (tid + MFT < PHN) sph[kb % 3][tid + MFT] = f1;
    }
    __syncthreads();
    double nxc, nyc, nzc, nzm, t0, t1;
    normal(me, kb - 1, iz2(kb - 1), t0, t1, nzm);
    normal(me, kb, iz2(kb), nxc, nyc, nzc);
    halo_normal(kb, iz2(kb));
    snx[kb & 1][ty * NXX + tx + 1] = nxc;
    sny[kb & 1][(ty + 1) * MFI + tx] = nyc;
    // width of planes and the z face below plane kb
    const double dzm = utab(G.dzf, wrapk(kb - 1));
    double dz0 = utab(G.dzf, kb);
    double nfb = (nzm * dz0 + nzc * dzm) * (0.5 * utab(G.rz, 6 * kb + 2));
    __syncthreads(); // plane kb - 2 was read above, its place takes kb + 2
    // planes in flight: psi of k + 2, phi of k + 1
    const double *sp = A.psi + (size_t)wrapk(kb + 2) * sz, *sf = A.phi + (size_t)wrapk(kb + 1) * sz;
    double p0 = sp[o0], p1 = sp[o1], f0 = sf[h0], f1 = sf[h1];
    int phs = kb % 3; // phi plane of k
    for (int k = kb; k < ke; ++k) {
        const int phn = phs == 2 ? 0 : phs + 1;
        sps[(k + 2) & 3][tid] = p0;
        if (tid + MFT < PSN) sps[(k + 2) & 3][tid + MFT] = p1;
        sph[phn][r0] = f0;
        if (tid + MFT < PHN) sph[phn][tid + MFT] = f1;
        // the next planes (the last ones of the chunk are read, not used)
        sp = A.psi + (size_t)wrapk(min(k + 3, ke + 1)) * sz;
        sf = A.phi + (size_t)wrapk(min(k + 2, ke)) * sz;
        p0 = sp[o0];
        p1 = sp[o1];
        f0 = sf[h0];
        f1 = sf[h1];
        __syncthreads();
        double nxp, nyp, nzp;
        normal(me, k + 1, iz2(k + 1), nxp, nyp, nzp);
        halo_normal(k + 1, iz2(k + 1));
        snx[(k + 1) & 1][ty * NXX + tx + 1] = nxp;
        sny[(k + 1) & 1][(ty + 1) * MFI + tx] = nyp;
        const double dzp = utab(G.dzf, wrapk(k + 1)), izc = utab(G.rz, 6 * k + 3), izf = utab(G.rz, 6 * k);
        const double *ps = sps[k & 3] + me;
        const double *ph = sph[phs] + ty * PHX + tx;
        const double *px = snx[k & 1] + ty * NXX + tx + 1, *py = sny[k & 1] + (ty + 1) * MFI + tx;
        const double nfe = 0.5 * (nxc + px[1]), nfw = 0.5 * (px[-1] + nxc);
        const double nfn = 0.5 * (nyc + py[MFI]), nfs = 0.5 * (py[-MFI] + nyc);
        const double nft = (nzc * dzp + nzp * dz0) * (0.5 * izc);
        const double P0 = ps[0], F0 = ph[0];
        auto flux = [&](double psf, double gphi, double nf) {
            // (1 - tanh^2 z) / 4 as in flux_face
            const double y = exp(-2.0 * fabs(psf * A.P.ihe));
            const double w = y / ((1.0 + y) * (1.0 + y));
            return A.P.gamma * (A.P.eps * gphi - w * nf);
        };
        const double ax = flux(0.5 * (P0 + ps[1]), (ph[1] - F0) * G.ih[0], nfe);
        const double ay = flux(0.5 * (P0 + ps[PSX]), (ph[PHX] - F0) * G.ih[1], nfn);
        const double az = flux((P0 * dzp + sps[(k + 1) & 3][me] * dz0) * (0.5 * izc),
                               (sph[phn][ty * PHX + tx] - F0) * izc, nft);
        const double kap = -((nfe - nfw) * G.ih[0] + (nfn - nfs) * G.ih[1] + (nft - nfb) * izf);
        if (act) {
            const size_t c = (size_t)k * sz + (size_t)j * nx + i;
            put(A.a[0] + c, ax);
            put(A.a[1] + c, ay);
            put(A.a[2] + c, az);
            put(A.kap + c, kap);
            // the box's cells next to a wall box: their normal is read there
            if ((!G.per[0] && (i == b.it0 * FTI || i == i1 - 1)) || (!G.per[1] && (j == b.jt0 * FTJ || j == j1 - 1)) ||
                (!G.per[2] && (k == b.k0 || k == b.k0 + b.nk - 1))) {
                put(A.n[0] + c, nxc);
                put(A.n[1] + c, nyc);
                put(A.n[2] + c, nzc);
            }
        }
        nxc = nxp;
        nyc = nyp;
        nzc = nzp;
        nfb = nft;
        dz0 = dzp;
        phs = phn;
    }
}

// order-preserving key of a double for atomicMin
__device__ __forceinline__ unsigned long long fkey(double v)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// the substep's phase update of cell c from its right-hand side r: the new
// phi and density, this substep's right-hand side; key: the density's
// minimum key
__device__ __forceinline__ void phase_put(const FArgs &A, size_t c, double r, double phi_c, double old,
                                          unsigned long long &key)
{
    const double q = phi_c + A.Dt * (A.ga * r + A.ze * old);
    put(A.phi_out + c, q);
    const double rho = A.P.rho2 + (A.P.rho1 - A.P.rho2) * q;
    put(A.rho_new + c, rho);
    key = fkey(rho);
    put(A.hphi + c, r);
}

// the workgroup's minimum key into its slot (every thread of the workgroup
// takes part; one slot per workgroup, reduced by k_flow_min: an atomic per
// workgroup on one address would serialize half a million workgroups)
__device__ __forceinline__ void key_to_slot(unsigned long long key, unsigned long long *slot)
{
    __shared__ unsigned long long red[FT / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long x = __shfl_xor(key, o, 64);
        key = x < key ? x : key;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = key;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < FT / 64; ++i) key = red[i] < key ? red[i] : key;
        key = red[0] < key ? red[0] : key;
        *slot = key;
    }
}

// Phase-field right-hand side only (the phase right-hand side entry point;
// the substep's update runs in the momentum pass)
__global__ __launch_bounds__(FT) void k_flow_phase(BoxList L, FArgs A)
{
    const BoxPick p = box_pick(L);
    const FTile t = btile(A.G, p.b, p.w);
    if (!t.act) return;
    double r = 0.0;
    if (p.fast) {
        // phi, u, v, w, a_x, a_y, a_z from registers, loaded up front
        double rg[7][27];
        const double *const src[7] = {A.phi, A.u, A.v, A.w, A.a[0], A.a[1], A.a[2]};
        stage_regs<7>(A.G, t, src, rg);
        r = acdi_cell(StageAcc<0>(A.G, t.i, t.j, t.k, nullptr, 0, 0, 0, rg), SField<0>{}, SVec<1>{}, SVec<4>{});
    } else {
        const PVel vel{A.u, A.v, A.w};
        const PVec av{A.a[0], A.a[1], A.a[2]};
        r = acdi_cell(Gen{A.G, t.i, t.j, t.k}, A.phi, vel, av);
    }
    put(A.hphi + at(A.G, t.i, t.j, t.k), r);
}

// minimum of n workgroup keys: each workgroup's own into out[its number]
constexpr int MINT = 1024;
__global__ __launch_bounds__(MINT) void k_flow_min(const unsigned long long *part, int n, unsigned long long *out)
{
    __shared__ unsigned long long red[MINT / 64];
    unsigned long long key = ~0ull;
    for (int i = blockIdx.x * MINT + threadIdx.x; i < n; i += gridDim.x * MINT) key = part[i] < key ? part[i] : key;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long x = __shfl_xor(key, o, 64);
        key = x < key ? x : key;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = key;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 0; i < MINT / 64; ++i) key = red[i] < key ? red[i] : key;
        __hip_atomic_store(out + blockIdx.x, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

template <int C, class X, class V, class PH, class KP, class AV>
__device__ __forceinline__ double mom_rhs(const FArgs &A, const X &x, const FTile &t, const V &vel, PH phi, KP kap,
                                          const AV &a)
{
    const int s = C == 0 ? t.i : (C == 1 ? t.j : t.k);
    // a branch, not a select: it keeps the three components apart (merged, one
    // workgroup per tile took 160 registers instead of 126)
    return wallf(A.G, C, s) ? 0.0 : mom_face<C>(x, A.P, phi, kap, vel, a);
}

// this substep's right-hand side m into hc (the previous one read first)
// and, with u*, the predictor (0 on a wall face: the correction ignores it)
// (old: the previous right-hand side, qv: the velocity component at c)
template <int C>
__device__ __forceinline__ void mom_put(const FArgs &A, const FTile &t, size_t c, double m, double old, double qv,
                                        double *hc, double *qs)
{
    const int s = C == 0 ? t.i : (C == 1 ? t.j : t.k);
    if (qs) put(qs + c, wallf(A.G, C, s) ? 0.0 : qv + A.Dt * (A.ga * m + A.ze * old));
    put(hc + c, m);
}
static_assert(SLX == FTI + 2 && SLY == FTJ + 2, "stage shape follows the tile shape");

// Cell s of direction d of a stage, one outside the tile at most: wrapped
// across a periodic direction, the adjacent cell across a wall (and, past
// the end of a partial tile, any valid cell).
__device__ __forceinline__ int stage_idx(const FGrid &G, int d, int s)
{
    const int n = G.n[d];
    const int t = G.per[d] ? (s < 0 ? s + n : (s >= n ? s - n : s)) : s;
    return t < 0 ? 0 : (t < n ? t : n - 1);
}

// The thread's cells of a stage plane: u, v, w and phi over the tile of (i0,
// j0) and its one-cell halo.  FAST: interior tiles, where a halo index leaves
// the grid only across a periodic direction and wraps by one period (the tile
// plan has no interior box when a periodic direction is shorter than the tile
// and halo).  Otherwise the stage takes the values the wall rules give (face
// components 0 on and beyond their own walls, minus the adjacent value across
// another), so the stencils read it as they read an interior tile's.  A
// plane's address is uniform over the workgroup and the offsets in it (32
// bits, in bytes) are the same for every plane and field.
constexpr int SNR2 = (SPL + FT - 1) / FT;
template <bool FAST> struct StagePlane {
    uint32_t off[SNR2];
    bool out[2][SNR2], own[2][SNR2]; // outside a wall direction; on or beyond the walls of the direction's own faces
    __device__ __forceinline__ StagePlane(const FGrid &G, int i0, int j0)
    {
        const int nx = G.n[0], ny = G.n[1];
#pragma unroll
        for (int q = 0; q < SNR2; ++q) {
            int e = threadIdx.x + q * FT;
            e = e < SPL ? e : SPL - 1;
            const int jj = e / SLX, ii = e - jj * SLX;
            int gi = i0 - 1 + ii, gj = j0 - 1 + jj;
            if constexpr (FAST) {
                gi = gi < 0 ? gi + nx : (gi >= nx ? gi - nx : gi);
                gj = gj < 0 ? gj + ny : (gj >= ny ? gj - ny : gj);
            } else {
                out[0][q] = !G.per[0] && (gi < 0 || gi >= nx);
                own[0][q] = !G.per[0] && (gi < 0 || gi >= nx - 1);
                out[1][q] = !G.per[1] && (gj < 0 || gj >= ny);
                own[1][q] = !G.per[1] && (gj < 0 || gj >= ny - 1);
                gi = stage_idx(G, 0, gi);
                gj = stage_idx(G, 1, gj);
            }
            off[q] = ((uint32_t)gj * nx + gi) * 8u;
        }
    }
    // plane k from memory, into the registers v
    __device__ __forceinline__ void load(const FArgs &A, int k, double (&v)[SNF][SNR2]) const
    {
        const FGrid &G = A.G;
        const double *const src[SNF] = {A.u, A.v, A.w, A.phi};
        const size_t o = (size_t)stage_idx(G, 2, k) * ((size_t)G.n[0] * G.n[1]);
#pragma unroll
        for (int f = 0; f < SNF; ++f)
#pragma unroll
            for (int q = 0; q < SNR2; ++q) v[f][q] = ldo(src[f] + o, off[q]);
    }
    // and from there into the stage plane at st
    __device__ __forceinline__ void store(const FGrid &G, int k, const double (&v)[SNF][SNR2], double *st) const
    {
        const bool outz = !FAST && !G.per[2] && (k < 0 || k >= G.n[2]);
        const bool ownz = !FAST && !G.per[2] && (k < 0 || k >= G.n[2] - 1);
#pragma unroll
        for (int f = 0; f < SNF; ++f)
#pragma unroll
            for (int q = 0; q < SNR2; ++q) {
                const int e = threadIdx.x + q * FT;
                double x = v[f][q];
                if constexpr (!FAST) {
                    if (f < 3) {
                        const bool zero = f == 0 ? own[0][q] : (f == 1 ? own[1][q] : ownz);
                        const bool neg = f == 0 ? out[1][q] != outz : (f == 1 ? outz != out[0][q] : out[0][q] != out[1][q]);
                        x = zero ? 0.0 : (neg ? -x : x);
                    }
                }
                if (e < SPL) st[f * SFLD + e] = x;
            }
    }
};

// The register stage of a tile along the walls: a_x, a_y, a_z (0 beyond
// their own walls; on them the flux kernel stored 0) and kappa (the adjacent
// value across a wall) over the thread's 3 x 3 x 3 neighbourhood.
__device__ __forceinline__ void stage_regs_wall(const FArgs &A, const FTile &t, double (&rg)[SNR][27])
{
    const FGrid &G = A.G;
    const int c[3] = {t.i, t.j, t.k};
    int ix[3][3];
    bool low[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        low[d] = !G.per[d] && c[d] == 0;
#pragma unroll
        for (int o = 0; o < 3; ++o) ix[d][o] = stage_idx(G, d, c[d] + o - 1);
    }
    const double *const src[SNR] = {A.a[0], A.a[1], A.a[2], A.kap};
#pragma unroll
    for (int q = 0; q < SNR; ++q)
#pragma unroll
        for (int n = 0; n < 27; ++n) {
            const int o[3] = {n % 3, (n / 3) % 3, n / 9};
            const double v = src[q][at(G, ix[0][o[0]], ix[1][o[1]], ix[2][o[2]])];
            rg[q][n] = q < 3 && o[q < 3 ? q : 0] == 0 && low[q < 3 ? q : 0] ? 0.0 : v;
        }
}

// Momentum right-hand side of the three components (all loads of a plane
// before any store); with u*, the substep's predictor; with p*, the
// extrapolated pressure.  With PH also the phase field's right-hand side and
// update (the substep), whose stencil reads only values the stages already
// hold.
// A workgroup marches its tile through a chunk of planes with three planes of
// u, v, w and phi (tile and halo) in LDS, so a plane is fetched once per
// chunk and not by the three tiles that read it: with one workgroup per tile
// and plane a wave issued 62 vector memory instructions and the substep's
// pass took 7.2 ms at 512^3; 6.1-6.2 here, of which the 24 fields it moves take
// 5.0 at copy rate (taking a fifth of the arithmetic out of the former
// changed nothing).  At 144 x 54 x 50 in a closed box 33 us either way.
// The tiles along the walls run the same code on a stage that holds what the
// wall rules give (26 us against 85 with the rules applied at every access).
template <bool PH, bool FAST>
__device__ __forceinline__ void momentum_march(const FArgs &A, FTile t, int ke, double *st, unsigned long long &key)
{
    const int tx = threadIdx.x % FTI, ty = threadIdx.x / FTI, l = (ty + 1) * SLX + tx + 1;
    const StagePlane<FAST> sp(A.G, t.i - tx, t.j - ty);
    int s0 = 1; // slot of plane k; the planes below and above in the ones before and after it
    {
        double v0[SNF][SNR2], v1[SNF][SNR2];
        sp.load(A, t.k - 1, v0);
        sp.load(A, t.k, v1);
        sp.store(A.G, t.k - 1, v0, st);
        sp.store(A.G, t.k, v1, st + SPL);
    }
#pragma unroll 1
    for (; t.k < ke; ++t.k) {
        // nothing computed from the column is kept from plane to plane (220
        // registers otherwise, two waves per SIMD; 164 so, three)
        asm volatile("" : "+v"(t.i), "+v"(t.j));
        const int sm = s0 == 0 ? 2 : s0 - 1, su = s0 == 2 ? 0 : s0 + 1;
        double v[SNF][SNR2], rg[SNR][27];
        sp.load(A, t.k + 1, v);
        if constexpr (FAST) {
            const double *const rsrc[SNR] = {A.a[0], A.a[1], A.a[2], A.kap};
            stage_regs<SNR>(A.G, t, rsrc, rg);
        } else {
            stage_regs_wall(A, t, rg);
        }
        // the cell's previous right-hand sides and pressures, loaded with
        // the stages (threads past the grid read a clamped cell)
        const size_t cc = at(A.G, t.act ? t.i : A.G.n[0] - 1, t.act ? t.j : A.G.n[1] - 1, t.k);
        double old[3] = {0.0, 0.0, 0.0}, pp1 = 0.0, pp2 = 0.0, oldp = 0.0;
        if (!A.first) {
            if (A.us[0]) old[0] = own(A.hu + cc);
            if (A.us[1]) old[1] = own(A.hv + cc);
            if (A.us[2]) old[2] = own(A.hw + cc);
            if (PH) oldp = own(A.hphi + cc);
        }
        if (A.pstar) {
            pp1 = own(A.p1 + cc);
            pp2 = own(A.p2 + cc);
        }
        sp.store(A.G, t.k + 1, v, st + su * SPL);
        __syncthreads();
        if (t.act) {
            const StageAcc<SNF> x(A.G, t.i, t.j, t.k, st, sm * SPL + l, s0 * SPL + l, su * SPL + l, rg);
            const SVel vel;
            const SVec<4> av;
            const double m0 = mom_rhs<0>(A, x, t, vel, SField<3>{}, SField<7>{}, av);
            const double m1 = mom_rhs<1>(A, x, t, vel, SField<3>{}, SField<7>{}, av);
            const double m2 = mom_rhs<2>(A, x, t, vel, SField<3>{}, SField<7>{}, av);
            mom_put<0>(A, t, cc, m0, old[0], x.cv(SField<0>{}, 0, 0, 0), A.hu, A.us[0]);
            mom_put<1>(A, t, cc, m1, old[1], x.cv(SField<1>{}, 0, 0, 0), A.hv, A.us[1]);
            mom_put<2>(A, t, cc, m2, old[2], x.cv(SField<2>{}, 0, 0, 0), A.hw, A.us[2]);
            if (A.pstar) put(A.pstar + cc, (1.0 + A.r) * pp1 - A.r * pp2);
            if constexpr (PH) {
                unsigned long long q;
                phase_put(A, cc, acdi_cell(x, SField<3>{}, vel, av), x.cv(SField<3>{}, 0, 0, 0), oldp, q);
                key = q < key ? q : key;
            }
        }
        __syncthreads(); // the plane below gives its place to the one after next
        s0 = su;
    }
}

template <bool PH> __device__ __forceinline__ void momentum_body(const BoxList &L, const FArgs &A)
{
    __shared__ double st[SNF * SFLD];
    const BoxPick p = box_pick(L);
    int ke;
    const FTile t = bchunk(A.G, L, p, ke);
    unsigned long long key = ~0ull;
    // hu, hv, hw (and hphi) are read and written in place: each thread
    // reads and writes only its own cells
    if (t.valid) { // uniform over the workgroup, as p.fast
        if (p.fast) momentum_march<PH, true>(A, t, ke, st, key);
        else momentum_march<PH, false>(A, t, ke, st, key);
    }
    if constexpr (PH) key_to_slot(key, A.rho_part + blockIdx.x);
}

__global__ __launch_bounds__(FT) void k_flow_momentum(BoxList L, FArgs A) { momentum_body<false>(L, A); }
// the substep's momentum predictor with the phase update
__global__ __launch_bounds__(FT) void k_flow_mom_phase(BoxList L, FArgs A) { momentum_body<true>(L, A); }

// The normals and the flux take a plan made with zlow = 2 (the flux kernel's
// interior form reads psi two cells away).
hipError_t launch_normals(const FArgs &A, const TilePlan &tp, hipStream_t s)
{
    if (tp.zlow < 2) return hipErrorInvalidValue;
    const size_t n = (size_t)A.G.n[0] * A.G.n[1] * A.G.n[2];
    hipLaunchKernelGGL(k_flow_psi, dim3((unsigned)((n + FT - 1) / FT)), dim3(FT), 0, s, A);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // the tiles along the walls only: the interior box's flux kernel
    // evaluates its normals itself
    const BoxList out = box_list(tp, false, true);
    if (out.n) hipLaunchKernelGGL(k_flow_normals, dim3(out.grid), dim3(FT), 0, s, out, A);
    return hipGetLastError();
}
// Planes per chunk of the marching flux (txy tiles per plane, two workgroups
// per CU): rounds of workgroups times the planes each takes, four of them to
// start, is least.
static int flux_chunk(int nk, int txy)
{
    int best = nk;
    long cost = -1;
    for (int n = 1; n <= nk; ++n) {
        const int c = (nk + n - 1) / n;
        const long wgs = (long)txy * ((nk + c - 1) / c), t = (wgs + 511) / 512 * (c + 4);
        if (cost < 0 || t < cost) { cost = t; best = c; }
    }
    return best;
}
hipError_t launch_flux(const FArgs &A, const TilePlan &tp, hipStream_t s)
{
    if (tp.zlow < 2) return hipErrorInvalidValue;
    const BoxList out = box_list(tp, false, true);
    for (int q = 0; q < tp.n; ++q) {
        if (!tp.fast[q]) continue;
        const TileBox &b = tp.box[q];
        const int j0 = b.jt0 * FTJ, j1 = std::min((b.jt0 + b.njt) * FTJ, A.G.n[1]);
        const int txy = b.nit * ((j1 - j0 + MFJ - 1) / MFJ);
        const int ckc = flux_chunk(b.nk, txy);
        const int tiles = txy * ((b.nk + ckc - 1) / ckc);
        hipLaunchKernelGGL(k_flow_flux_in, dim3((tiles + 7) / 8 * 8), dim3(MFT), 0, s, b, ckc, A);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (out.n) hipLaunchKernelGGL(k_flow_flux_wall, dim3(out.grid), dim3(FT), 0, s, out, A);
    return hipGetLastError();
}
hipError_t launch_phase(const FArgs &A, const TilePlan &tp, hipStream_t s)
{
    return FLOW_LAUNCH_PLAN(tp, k_flow_phase, s, A);
}
hipError_t launch_momentum(const FArgs &A, const TilePlan &tp, hipStream_t s)
{
    const BoxList L = momentum_list(tp);
    hipLaunchKernelGGL(k_flow_momentum, dim3(L.grid), dim3(FT), 0, s, L, A);
    return hipGetLastError();
}
hipError_t launch_momentum_phase(const FArgs &A, const TilePlan &tp, hipStream_t s)
{
    if (!A.phi_out || !A.hphi || !A.rho_new) return hipErrorInvalidValue;
    const BoxList L = momentum_list(tp);
    hipLaunchKernelGGL(k_flow_mom_phase, dim3(L.grid), dim3(FT), 0, s, L, A);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // Up to 16 keys per thread one workgroup takes them all; more (4 million
    // cells and up) in two levels.  The result goes to host memory: clearing
    // a key, minima by atomics and a copy of it took two more steps of the
    // stream's chain and the copy's wait.
    const unsigned long long *part = A.rho_part;
    int n = L.grid; // at most tp.nslots
    if (n > 16 * MINT) {
        hipLaunchKernelGGL(k_flow_min, dim3(MINWG), dim3(MINT), 0, s, part, n, A.rho_part + n);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        part += n;
        n = MINWG;
    }
    hipLaunchKernelGGL(k_flow_min, dim3(1), dim3(MINT), 0, s, part, n, A.rho_min_key);
    return hipGetLastError();
}

double key_to_double(unsigned long long k)
{
    const unsigned long long u = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
    double v;
    __builtin_memcpy(&v, &u, 8);
    return v;
}

} // namespace flow
} // namespace pcx
