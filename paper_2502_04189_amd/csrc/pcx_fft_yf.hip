// pcx_fft_yf.hip -- the forward y passes of the lengths with a fixed plan
// (pcx_fft.hpp), one kernel per length above FSMALL and one for the rest.
#include "pcx_fft.hpp"

namespace pcx {

const void *fft_yfwd_kernel(int prec, int n)
{
    return prec == PREC_F64 ? fft_kernel<double, FK_YFWD>(n) : fft_kernel<float, FK_YFWD>(n);
}

} // namespace pcx
