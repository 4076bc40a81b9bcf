// pcx_fplan.hpp -- the lengths whose x and y passes have a fixed plan
// (pcx_fft.hpp): radices, lines per tile, workgroup size and LDS, shared by
// the kernels and the host.
#pragma once

#include "pcx_dev.hpp"

namespace pcx {

// ------------------------------------------------------------------ plans
// Radices of a length (last 0: unused).  At most 9, so a butterfly's points
// take 36 registers in FP64; the first is small enough that N / R lanes read
// 128 contiguous bytes.  0 radices: no fixed plan.
struct FPlan {
    int n, r[4];
};
__host__ __device__ constexpr FPlan fplan(int n)
{
    switch (n) {
    case 16: return {2, {2, 8}};
    case 18: return {2, {2, 9}};
    case 24: return {2, {3, 8}};
    case 27: return {2, {3, 9}};
    case 32: return {2, {4, 8}};
    case 36: return {2, {4, 9}};
    case 48: return {2, {6, 8}};
    case 54: return {2, {6, 9}};
    case 64: return {2, {8, 8}};
    case 72: return {2, {8, 9}};
    case 81: return {2, {9, 9}};
    case 96: return {3, {6, 4, 4}};
    case 108: return {3, {9, 4, 3}};
    case 128: return {3, {8, 4, 4}};
    case 144: return {3, {6, 6, 4}};
    case 162: return {3, {6, 9, 3}};
    case 192: return {3, {8, 6, 4}};
    case 216: return {3, {6, 6, 6}};
    case 243: return {3, {9, 9, 3}};
    case 256: return {3, {8, 8, 4}};
    case 288: return {3, {8, 6, 6}};
    case 324: return {3, {6, 9, 6}};
    case 384: return {3, {8, 8, 6}};
    case 432: return {3, {8, 9, 6}};
    case 486: return {3, {9, 9, 6}};
    case 512: return {3, {8, 8, 8}};
    case 576: return {3, {8, 9, 8}};
    case 648: return {3, {9, 9, 8}};
    case 729: return {3, {9, 9, 9}};
    case 768: return {4, {8, 4, 4, 6}};
    case 864: return {4, {6, 6, 6, 4}};
    case 972: return {4, {9, 6, 6, 3}};
    case 1024: return {4, {8, 8, 4, 4}};
    }
    return {0, {0, 0, 0, 0}};
}

// Lengths whose passes are compiled together into one kernel (their tiles
// all run in FSMALL_TH threads): one launch then serves the domains of every
// such length in a batch.
constexpr int FSMALL = 128, FSMALL_TH = 256;

// Most points a thread holds in a stage of n points x l lines on th threads.
__host__ __device__ constexpr int fft_points(int n, int l, int th)
{
    const FPlan p = fplan(n);
    int m = 0;
    for (int s = 0; s < p.n; ++s) {
        const int k = (l * n / p.r[s] + th - 1) / th * p.r[s];
        m = k > m ? k : m;
    }
    return m;
}
// Points a thread may hold: at 12 FP64 or 18 FP32 points and four waves per
// SIMD the passes spill.
__host__ __device__ constexpr int fft_points_max(int csz) { return csz == 16 ? 9 : 16; }

// Lines per tile: about 2048 FP64 or 4096 FP32 points, and at least 128
// bytes of a corner-turned segment.  Columns of 648 to 972 take 64-byte
// segments: a tile of 128-byte ones leaves room for one workgroup per CU, and
// only at 1024 do the whole lines outweigh that (128 x 1024 x 512 FP64, y
// forward + inverse: 534 us with 8 lines, 646 with 4; 128 x 768 x 512 with
// walls 508 and 433; FP32 at 1024 279 either way, with walls 306 with 8, 389 with 16).
__host__ __device__ constexpr int fft_lines(int n, int csz)
{
    const int pts = 32768 / csz, least = 128 / csz;
    int l = 128;
    while (l > least && (l * n > pts || (n <= FSMALL && fft_points(n, l, FSMALL_TH) > fft_points_max(csz)))) l >>= 1;
    if (l * n * csz > 72 * 1024 && (n < 1024 || csz == 8)) l >>= 1;
    return l;
}
// Fewest threads (a multiple of 64) that keep within fft_points_max.
__host__ __device__ constexpr int fft_threads(int n, int csz)
{
    if (n <= FSMALL) return FSMALL_TH;
    int th = 64;
    while (fft_points(n, fft_lines(n, csz), th) > fft_points_max(csz)) th += 64;
    return th;
}
// LDS bytes of an x or y tile
__host__ __device__ constexpr size_t fft_lds(int n, int csz)
{
    return ((size_t)fft_lines(n, csz) * lds_line(n) + tw_half(n)) * csz;
}

// Waves per SIMD that as many tiles as LDS has room for make up, between 4
// (128 registers) and 7 (72): a few lengths take some registers more than
// that leaves, and with them a tile per CU less (972 points forward in x:
// 84 instead of 80, one tile instead of two, 142 us instead of 103).  FP64
// tiles that would have to do with 80 registers to run three or more at once
// may take a tile less: 324 points, three tiles, spilled 1 (x inverse) and 3
// (y inverse) registers; with two, 648 x 324 x 320 cells with walls, 518 -> 485
// us y inverse, 311 -> 301 x inverse, periodic 212 -> 207 and 231 -> 230.
__host__ __device__ constexpr int fft_waves(int n, int csz)
{
    const int w = fft_threads(n, csz) / 64, t = (int)(160 * 1024 / fft_lds(n, csz));
    const int all = (t * w + 3) / 4, e = csz == 16 && t >= 3 && all >= 6 ? ((t - 1) * w + 3) / 4 : all;
    return n <= FSMALL || e < 4 ? 4 : (e > 7 ? 7 : e);
}

// longest half length of an x pass (columns: 1024)
constexpr int FXMAX = 512;

} // namespace pcx
