// Forward scan kernels of the threshold gate with a constant retention per lane (Sec. 3.2-3.5 of the paper), with the harmonic convolution.
#include "cawn_fwd_kernel.hpp"

namespace cawn {

hipError_t launch_fwd_hconv_plain(const FwdArgs &a, int conv_k, hipStream_t s)
{
    return launch_fwd_family<false, false, false, true>(a, conv_k, s);
}

}  // namespace cawn
