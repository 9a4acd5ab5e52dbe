// Forward scan kernels on short tiles of the per-head valve with the data-dependent retention (Sec. 3.3 of the paper).
#include "cawn_fwd_kernel.hpp"

namespace cawn {

hipError_t launch_fwd_short_valve_ret(const FwdArgs &a, int conv_k, hipStream_t s)
{
    return a.hconv ? launch_fwd_family<true, true, true, true>(a, conv_k, s) : launch_fwd_family<true, true, true, false>(a, conv_k, s);
}

}  // namespace cawn
