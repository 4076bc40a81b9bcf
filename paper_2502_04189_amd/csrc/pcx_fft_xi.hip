// pcx_fft_xi.hip -- the inverse x, p stored passes of the lengths with a fixed plan
// (pcx_fft.hpp), one kernel per length above FSMALL and one for the rest.
#include "pcx_fft.hpp"

namespace pcx {

const void *fft_xinv_store_kernel(int prec, int n)
{
    return prec == PREC_F64 ? fft_kernel<double, FK_XINV_STORE>(n) : fft_kernel<float, FK_XINV_STORE>(n);
}

} // namespace pcx
