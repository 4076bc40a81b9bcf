// flow_tile.hpp -- tiling of the one-thread-per-cell stencil launches of
// the substep and of the variable-coefficient projection: 256-thread
// workgroups of 64 x 4 cells of one plane.
//
// The tiles of a grid are split into boxes (ranges of x tiles, y tiles and
// planes): one interior box whose stencils reach no wall, and up to six
// boxes around it.  A kernel takes all of them in one launch (the flux two:
// its wall tiles read normals the interior ones store) and branches,
// uniformly over the workgroup, to code on the interior accessor or on the
// wall rules.  Within a launch consecutive workgroups go to different XCDs,
// so XCD x gets a contiguous range of a box's tiles in the order below.
#pragma once

#include <vector>

#include "flow_dev.hpp"

namespace pcx {
namespace flow {

constexpr int FT = 256, FTI = 64, FTJ = FT / FTI;

// tiles [it0, it0 + nit) x [jt0, jt0 + njt) x planes [k0, k0 + nk)
struct TileBox {
    int it0, jt0, k0, nit, njt, nk;
};

__host__ __device__ inline long box_tiles(const TileBox &b) { return (long)b.nit * b.njt * b.nk; }

// workgroups of a launch over a box (a multiple of 8, the XCD count)
inline int box_grid(const TileBox &b)
{
    const long n = box_tiles(b);
    return (int)(((n + 7) >> 3) << 3);
}

// The boxes of one grid: box b runs with the interior accessor when fast[b].
// A launch over all of them has at most nslots workgroups (slot0[b] is where
// box b's start), each with a partial-result slot of its own number.
struct TilePlan {
    int n;
    TileBox box[7];
    bool fast[7];
    int slot0[7];
    int nslots;
    int zlow; // first interior plane with walls in z (tile_plan's argument)
};

// Host tables of a grid's z metrics: dzf (nz), dzc (nz, the periodic wrap
// at nz-1), then the 6 nz reciprocals of FGrid::rz, each computed in the
// order and from the values the device accessors would use.
inline std::vector<double> metric_tables(const double *zf, int nz, bool zper)
{
    std::vector<double> t(8 * (size_t)nz);
    double *dzf = t.data(), *dzc = dzf + nz, *rz = dzc + nz;
    for (int k = 0; k < nz; ++k) dzf[k] = zf[k + 1] - zf[k];
    for (int k = 0; k < nz - 1; ++k) dzc[k] = 0.5 * (dzf[k] + dzf[k + 1]);
    dzc[nz - 1] = 0.5 * (dzf[nz - 1] + dzf[0]);
    auto fat = [&](int k) { return k < 0 ? dzf[zper ? nz - 1 : 0] : (k >= nz ? dzf[zper ? 0 : nz - 1] : dzf[k]); };
    auto cat = [&](int k) {
        if (k < 0) return zper ? dzc[nz - 1] : dzf[0];
        if (k >= nz - 1) return zper ? dzc[nz - 1] : dzf[nz - 1];
        return dzc[k];
    };
    for (int k = 0; k < nz; ++k) {
        double *r = rz + 6 * (size_t)k;
        const double f0 = fat(k), fp = fat(k + 1), cm = cat(k - 1), c0 = cat(k);
        r[0] = 1.0 / f0;
        r[1] = 1.0 / fp;
        r[2] = 1.0 / cm;
        r[3] = 1.0 / c0;
        r[4] = 1.0 / (c0 + cm);
        r[5] = 1.0 / (f0 + fp);
    }
    return t;
}

// Tile boxes of a grid.  The stencils reach one cell (and one face) beyond
// their cell, so a wall direction's interior tiles lie within [1, n-3]: x
// tiles it >= 1 with (it + 1) FTI <= nx - 2, likewise y, planes 1 .. nz-3.
// With zlow = 2 the interior planes start at 2 (wall z; x and y tiles are
// at least 4 cells from a wall anyway): the flux kernel's interior form
// evaluates the normals of its neighbours, whose stencils reach two cells.
inline TilePlan tile_plan(const FGrid &G, int zlow = 1)
{
    const int ti = (G.n[0] + FTI - 1) / FTI, tj = (G.n[1] + FTJ - 1) / FTJ, nz = G.n[2];
    const int it0 = G.per[0] ? 0 : 1, it1 = G.per[0] ? ti : (G.n[0] - 2) / FTI;
    const int jt0 = G.per[1] ? 0 : 1, jt1 = G.per[1] ? tj : (G.n[1] - 2) / FTJ;
    const int k0 = G.per[2] ? 0 : zlow, k1 = G.per[2] ? nz : nz - 2;
    TilePlan p{};
    p.zlow = zlow;
    auto add = [&](TileBox b, bool fast) {
        if (b.nit <= 0 || b.njt <= 0 || b.nk <= 0) return;
        p.box[p.n] = b;
        p.fast[p.n] = fast;
        p.slot0[p.n] = p.nslots;
        p.nslots += box_grid(b);
        ++p.n;
    };
    // the interior kernels' stages wrap a halo index by at most one period
    const bool small = (G.per[0] && G.n[0] < FTI + 2) || (G.per[1] && G.n[1] < FTJ + 2) || (G.per[2] && nz < 3);
    if (small || it1 <= it0 || jt1 <= jt0 || k1 <= k0) {
        add(TileBox{0, 0, 0, ti, tj, nz}, false);
        return p;
    }
    add(TileBox{it0, jt0, k0, it1 - it0, jt1 - jt0, k1 - k0}, true);
    add(TileBox{0, 0, 0, ti, tj, k0}, false);                            // planes below
    add(TileBox{0, 0, k1, ti, tj, nz - k1}, false);                      // planes above
    add(TileBox{0, 0, k0, ti, jt0, k1 - k0}, false);                     // rows south
    add(TileBox{0, jt1, k0, ti, tj - jt1, k1 - k0}, false);              // rows north
    add(TileBox{0, jt0, k0, it0, jt1 - jt0, k1 - k0}, false);            // columns west
    add(TileBox{it1, jt0, k0, ti - it1, jt1 - jt0, k1 - k0}, false);     // columns east
    return p;
}

struct FTile {
    int i, j, k;
    bool act;   // the thread's cell is in the grid
    bool valid; // the workgroup has a tile (uniform over the workgroup)
};

// Order of the tiles within a box: chunks of TKC planes; within a chunk, x
// tiles fastest, then planes, then y tiles.  A tile's z neighbours are then
// nit tiles away in the launch order and its y neighbours nit * TKC tiles
// away, inside the window of workgroups an XCD runs at once, so the planes
// and rows a tile re-reads are still in that XCD's L2 (ordered plane by
// plane, the next plane of the same tile came a whole plane of tiles later
// and every z neighbour was fetched again).
constexpr int TKC = 16;

// tile t (0 <= t < box_tiles(b)) of a box in the order above
__host__ __device__ inline void box_tile(const TileBox &b, long t, int &it, int &jt, int &k)
{
    const long chunk = (long)b.nit * b.njt * TKC;
    const int kc = (int)(t / chunk);
    const int rem = (int)(t - (long)kc * chunk);
    const int kb = kc * TKC;
    const int nkc = b.nk - kb < TKC ? b.nk - kb : TKC; // planes in this chunk
    const int ii = rem % b.nit;
    const int q = rem / b.nit;
    it = b.it0 + ii;
    jt = b.jt0 + q / nkc;
    k = b.k0 + kb + q % nkc;
}

// The boxes of one launch: workgroup first[q] + w is workgroup w of box q
// (every box's workgroups are a multiple of 8, so w & 7 is the workgroup's XCD
// as well).
constexpr int MAXBOX = 7;
struct BoxList {
    int n, grid;
    int fast; // box 0 is the interior box
    TileBox box[MAXBOX];
    int first[MAXBOX];
    int ck, kend[MAXBOX]; // a list in chunks of ck planes: box[q].nk counts chunks, kend[q] is the box's last plane + 1
};

// The interior box and / or the boxes along the walls of a plan, as one
// launch: run one after another, the wall boxes of a small grid each took
// the time of one workgroup (45-60 us for the momentum at 144 x 54 x 50) and
// left the device idle.
inline BoxList box_list(const TilePlan &p, bool interior, bool walls)
{
    BoxList L{};
    for (int b = 0; b < p.n; ++b) { // the interior box, if any, is the plan's first
        if (!(p.fast[b] ? interior : walls)) continue;
        if (p.fast[b]) L.fast = 1;
        L.box[L.n] = p.box[b];
        L.first[L.n] = L.grid;
        L.grid += box_grid(p.box[b]);
        ++L.n;
    }
    return L;
}

// The list with a workgroup per chunk of ck planes of a tile, for kernels
// that march in z (no more workgroups than before).
inline BoxList box_chunks(BoxList L, int ck)
{
    L.ck = ck;
    L.grid = 0;
    for (int q = 0; q < L.n; ++q) {
        L.kend[q] = L.box[q].k0 + L.box[q].nk;
        L.box[q].nk = (L.box[q].nk + ck - 1) / ck;
        L.first[q] = L.grid;
        L.grid += box_grid(L.box[q]);
    }
    return L;
}

// The momentum launch: chunks of planes of every box.  Rounds of workgroups
// (three per CU: the kernel takes 164 registers) times the planes each takes,
// three to start, is least; of lengths whose last chunk is rarely a short one
// and whose starts stay aligned.  Kernel times, chunks of 4, 8, 16, 17 and 32
// planes: 512^3 walls in z 6.18 ms (16), 6.12 (17), 6.19 (32), periodic 6.19,
// 6.36, 6.18; 256^3 815, 790, 781, 778, 785 us (10 planes 845); 128^3 106,
// 107, 111, 117, 138 (9 planes 117); 512 x 512 x 64 878, 828, 808, 854, 817 (7
// planes 880); 64^3 24, 41 and 21.6, 18.9 in chunks of 1 and 2; 144 x 54 x 50
// 36, 34, 32 and 38 in 1, 2, 3 and 4.
inline BoxList momentum_list(const TilePlan &tp)
{
    const BoxList L = box_list(tp, true, true);
    int best = 1;
    long cost = -1;
    for (int c : {1, 2, 3, 4, 6, 8, 16, 32}) {
        const long t = (box_chunks(L, c).grid + 767L) / 768 * (c + 3);
        if (cost < 0 || t < cost) { cost = t; best = c; }
    }
    return box_chunks(L, best);
}

// the box of this workgroup and its number in the box
struct BoxPick {
    TileBox b;
    unsigned w;
    bool fast;
    int kend;
};
__device__ __forceinline__ BoxPick box_pick(const BoxList &L)
{
    BoxPick p{L.box[0], blockIdx.x, L.fast != 0, L.kend[0]};
#pragma unroll
    for (int q = 1; q < MAXBOX; ++q)
        if (q < L.n && (int)blockIdx.x >= L.first[q])
            p = BoxPick{L.box[q], blockIdx.x - L.first[q], false, L.kend[q]};
    return p;
}

// The thread's column in a list in chunks and its planes [k, ke): x tiles
// fastest, then y tiles, then chunks, so the tiles an XCD runs at once are
// neighbours in x and y on the same planes.
__device__ __forceinline__ FTile bchunk(const FGrid &G, const BoxList &L, const BoxPick &p, int &ke)
{
    const int nxy = p.b.nit * p.b.njt, n = nxy * p.b.nk, per = (n + 7) >> 3;
    const int t = (int)(p.w & 7) * per + (int)(p.w >> 3);
    FTile c;
    c.act = false;
    c.valid = t < n && (int)(p.w >> 3) < per;
    c.i = c.j = c.k = ke = 0;
    if (!c.valid) return c;
    const int ch = t / nxy, rem = t - ch * nxy, jt = rem / p.b.nit;
    c.k = p.b.k0 + ch * L.ck;
    ke = c.k + L.ck < p.kend ? c.k + L.ck : p.kend;
    c.i = (p.b.it0 + rem - jt * p.b.nit) * FTI + (threadIdx.x % FTI);
    c.j = (p.b.jt0 + jt) * FTJ + (threadIdx.x / FTI);
    c.act = c.i < G.n[0] && c.j < G.n[1];
    return c;
}

// the thread's cell in workgroup w of box b (act false past the box or the grid)
__device__ __forceinline__ FTile btile(const FGrid &G, const TileBox &b, unsigned w)
{
    const long n = box_tiles(b);
    const long per = (n + 7) >> 3;
    const long t = (long)(w & 7) * per + (w >> 3);
    FTile c;
    c.act = false;
    c.valid = t < n;
    c.i = c.j = c.k = 0;
    if (!c.valid) return c;
    int it, jt;
    box_tile(b, t, it, jt, c.k);
    c.i = it * FTI + (threadIdx.x % FTI);
    c.j = jt * FTJ + (threadIdx.x / FTI);
    c.act = c.i < G.n[0] && c.j < G.n[1];
    return c;
}

// the value `off` bytes into a plane whose address is uniform over the wave
__device__ __forceinline__ double ldo(const double *plane, uint32_t off)
{
    return *(const double *)((const char *)plane + off);
}

// register stage of the listed fields: each thread's 3 x 3 x 3 neighbourhood
// (loads whose values no stencil reads are removed by the compiler), all
// issued before the first use; threads past the grid read a clamped cell.
// Plane bases are uniform, offsets in a plane 32 bits.
template <int N>
__device__ __forceinline__ void stage_regs(const FGrid &G, const FTile &t, const double *const (&src)[N],
                                           double (&rg)[N][27])
{
    const int nx = G.n[0], ny = G.n[1], nz = G.n[2];
    const int i = t.act ? t.i : nx - 1, j = t.act ? t.j : ny - 1, k = t.k;
    const int x[3] = {i == 0 ? nx - 1 : i - 1, i, i == nx - 1 ? 0 : i + 1};
    const int y[3] = {j == 0 ? ny - 1 : j - 1, j, j == ny - 1 ? 0 : j + 1};
    const int z[3] = {k == 0 ? nz - 1 : k - 1, k, k == nz - 1 ? 0 : k + 1};
#pragma unroll
    for (int q = 0; q < N; ++q)
#pragma unroll
        for (int n = 0; n < 27; ++n)
            rg[q][n] = ldo(src[q] + (size_t)z[n / 9] * ((size_t)nx * ny),
                           ((uint32_t)y[(n / 3) % 3] * nx + x[n % 3]) * 8u);
}

// Launches a kernel, which takes (box list, args...), on every box of a plan.
#define FLOW_LAUNCH_PLAN(TP, KERNEL, STREAM, ...)                                                          \
    ([&]() -> hipError_t {                                                                                \
        const BoxList l_ = box_list((TP), true, true);                                                    \
        hipLaunchKernelGGL(KERNEL, dim3(l_.grid), dim3(FT), 0, (STREAM), l_, __VA_ARGS__);                \
        return hipGetLastError();                                                                         \
    }())

} // namespace flow
} // namespace pcx
