// Forward scan kernels on short tiles of the data-dependent retention (Sec. 3.3 item 4 of the paper), threshold gate.
#include "cawn_fwd_kernel.hpp"

namespace cawn {

hipError_t launch_fwd_short_ret(const FwdArgs &a, int conv_k, hipStream_t s)
{
    return a.hconv ? launch_fwd_family<true, false, true, true>(a, conv_k, s) : launch_fwd_family<true, false, true, false>(a, conv_k, s);
}

}  // namespace cawn
