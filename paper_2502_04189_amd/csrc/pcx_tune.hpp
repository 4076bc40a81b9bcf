// pcx_tune.hpp -- autotuner of per-size-class launch shapes (x/y tile sizes,
// FFT radix splits, z lanes per line) and its text cache.
#pragma once

#include <algorithm>
#include <map>
#include <string>
#include <vector>

#include "pcx_launch.hpp"
#include "pcx_plan.hpp"

namespace pcx {

struct TuneCache {
    std::map<std::string, std::pair<TuneParams, RadixChoice>> m;
    static std::string key(const pcx_grid &g, int prec);
    bool load(const char *path);
    bool save(const char *path) const;
    bool lookup(const pcx_grid &g, int prec, TuneParams &tp, RadixChoice &rc) const;
    void store(const pcx_grid &g, int prec, const TuneParams &tp, const RadixChoice &rc);
};

// Items of a timed grouped launch, at least: a small domain's tiles leave
// most of the device idle, and the shape that spreads them best is not the
// one that does the least work per cell, which is what counts when a batch
// fills the device.
constexpr long GFILL = 1024;
// Copies of a domain's S2 the z solve is timed on, 64 MB in all (1024 of the
// smallest ones): it solves
// lines in place, so no two items may have the same ones, and a batch's lines
// come from memory (with the few MB of one domain over and over, out of the
// L2s, 12 and 16 levels per lane looked best, and the tuned batch of 192
// domains took 2928 us against 2891 with the defaults, refined 4865 against
// 4820; now 2888 and 4780).
inline int tune_z_copies(size_t s2_bytes)
{
    return (int)std::min<size_t>(1024, (((size_t)64 << 20) + s2_bytes - 1) / s2_bytes);
}
// The items of a timed grouped launch of a pass of t tiles: of the z solve
// every tile of every copy, last first; of the others the tiles repeated (the
// same values written twice to the same place).
inline std::vector<GItem> tune_items(int kind, long t, int zcopies)
{
    const long reps = kind == PK_Z ? zcopies : std::max(1L, GFILL / t);
    std::vector<GItem> v(t * reps);
    for (long q = 0; q < t * reps; ++q)
        v[q] = kind == PK_Z ? GItem{(uint32_t)(q / t), (uint32_t)(t - 1 - q % t)} : GItem{0u, (uint32_t)(q % t)};
    return v;
}

// Times candidate shapes of each pass on scratch data of this grid and
// returns the fastest per pass.  grouped: time the batch's grouped kernels
// (one-domain item lists), else the single-domain kernels of a plan.
pcx_status autotune_class(const pcx_grid &g, int prec, hipStream_t s, TuneParams &tp, RadixChoice &rc,
                          bool grouped);

} // namespace pcx
