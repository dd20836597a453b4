// Instances of conv_parts_kernel for fp32 storage, forward with the class layer.
#include "kernels_conv_parts.hpp"
#include "launchers.hpp"

namespace mpcnn {

bool launch_conv_head_f32(const ConvArgs& a, const PartsInstance& in, dim3 grid, size_t lds, hipStream_t st)
{
#define CASE(cb, wo, wp, mo, mp)                                                                       \
    if (in.CB == cb && in.WO == wo && in.WP == wp && in.MO == mo && in.MP == mp) {                     \
        conv_parts_kernel<float, false, cb, wo, wp, mo, mp, true><<<grid, 64 * wo * wp, lds, st>>>(a);   \
        return true;                                                                                   \
    }
    MPCNN_HEAD3(CASE)
#undef CASE
    return false;
}

}  // namespace mpcnn
