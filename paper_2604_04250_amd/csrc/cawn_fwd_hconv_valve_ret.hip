// Forward scan kernels of the per-head valve with the data-dependent retention (Sec. 3.3 of the paper), with the harmonic convolution.
#include "cawn_fwd_kernel.hpp"

namespace cawn {

hipError_t launch_fwd_hconv_valve_ret(const FwdArgs &a, int conv_k, hipStream_t s)
{
    return launch_fwd_family<false, true, true, true>(a, conv_k, s);
}

}  // namespace cawn
