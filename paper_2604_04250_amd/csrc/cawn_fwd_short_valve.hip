// Forward scan kernels on short tiles of the per-head input valve (Sec. 3.3 of the paper) with a constant retention per lane.
#include "cawn_fwd_kernel.hpp"

namespace cawn {

hipError_t launch_fwd_short_valve(const FwdArgs &a, int conv_k, hipStream_t s)
{
    return a.hconv ? launch_fwd_family<true, true, false, true>(a, conv_k, s) : launch_fwd_family<true, true, false, false>(a, conv_k, s);
}

}  // namespace cawn
