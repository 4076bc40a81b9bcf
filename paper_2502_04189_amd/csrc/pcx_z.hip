// pcx_z.hip -- the z solve, one kernel per number of levels a lane holds,
// for a lone domain and for the items of a batch (as the fixed-plan passes
// of pcx_fft.hpp).
#include "pcx_launch.hpp"
#include "pcx_passes.hpp"

namespace pcx {

template <typename T, int S> __global__ __launch_bounds__(NT) void k_z(FftArgs unused)
{
    extern __shared__ __align__(16) char smem[];
    typedef const __attribute__((address_space(4))) FftArgs *Arg;
    const Arg A = (Arg)__builtin_amdgcn_kernarg_segment_ptr();
    const __attribute__((address_space(4))) Dom *p = &A->d;
    // lines in the reverse of the order the forward y pass wrote them (a
    // batch lists them so), so the first tiles read what the device-side
    // cache still holds
    int tile = A->d.nzt - 1 - (int)blockIdx.x;
    if (A->g.items) {
        p = (const __attribute__((address_space(4))) Dom *)A->g.doms +
            __builtin_amdgcn_readfirstlane((int)A->g.items[blockIdx.x].dom);
        tile = __builtin_amdgcn_readfirstlane((int)A->g.items[blockIdx.x].tile);
    }
    pass_z<T, S>(*(const Dom *)p, tile, smem);
}

template <typename T> static const void *z_fn(int levels)
{
    switch (levels) {
#define PCX_Z(S) case S: return (const void *)k_z<T, S>;
    PCX_Z(2) PCX_Z(3) PCX_Z(4) PCX_Z(5) PCX_Z(6) PCX_Z(7) PCX_Z(8) PCX_Z(10) PCX_Z(12) PCX_Z(14) PCX_Z(16)
#undef PCX_Z
    }
    return nullptr;
}

const void *z_kernel(int prec, int levels) { return prec == PREC_F64 ? z_fn<double>(levels) : z_fn<float>(levels); }

} // namespace pcx
