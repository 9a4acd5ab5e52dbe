// Forward scan kernels on short tiles of the threshold gate with a constant retention per lane (Sec. 3.2-3.5 of the paper).
#include "cawn_fwd_kernel.hpp"

namespace cawn {

hipError_t launch_fwd_short_plain(const FwdArgs &a, int conv_k, hipStream_t s)
{
    return a.hconv ? launch_fwd_family<true, false, false, true>(a, conv_k, s) : launch_fwd_family<true, false, false, false>(a, conv_k, s);
}

}  // namespace cawn
