// pcx_fft_xf.hip -- the forward x passes of the lengths with a fixed plan
// (pcx_fft.hpp), one kernel per length above FSMALL and one for the rest.
#include "pcx_fft.hpp"

namespace pcx {

const void *fft_xfwd_kernel(int prec, int n)
{
    return prec == PREC_F64 ? fft_kernel<double, FK_XFWD>(n) : fft_kernel<float, FK_XFWD>(n);
}

} // namespace pcx
