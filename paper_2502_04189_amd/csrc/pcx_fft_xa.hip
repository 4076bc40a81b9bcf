// pcx_fft_xa.hip -- the inverse x, p accumulated passes of the lengths with a fixed plan
// (pcx_fft.hpp), one kernel per length above FSMALL and one for the rest.
#include "pcx_fft.hpp"

namespace pcx {

const void *fft_xinv_accum_kernel(int prec, int n)
{
    return prec == PREC_F64 ? nullptr : fft_kernel<float, FK_XINV_ACCUM>(n); // only the refined form accumulates
}

} // namespace pcx
