// Instances of conv_parts_kernel for bf16 storage, forward.
#include "kernels_conv_parts.hpp"
#include "launchers.hpp"

namespace mpcnn {

bool launch_conv_parts_b16_fwd(const ConvArgs& a, const PartsInstance& in, dim3 grid, size_t lds, hipStream_t st)
{
#define CASE(cb, wo, wp, mo, mp)                                                                       \
    if (in.CB == cb && in.WO == wo && in.WP == wp && in.MO == mo && in.MP == mp) {                     \
        conv_parts_kernel<bf16, false, cb, wo, wp, mo, mp><<<grid, kPartsThreads, lds, st>>>(a);      \
        return true;                                                                                   \
    }
    MPCNN_PARTS1(CASE)
    MPCNN_PARTS1_WIDE(CASE)
    MPCNN_PARTS1_ALL(CASE)
#undef CASE
    return false;
}

hipError_t conv_parts_attrs_b16_fwd()
{
    hipError_t e = hipSuccess;
#define ATTR(cb, wo, wp, mo, mp)                                                                                       \
    if (e == hipSuccess)                                                                                               \
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_parts_kernel<bf16, false, cb, wo, wp, mo, mp>),   \
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    MPCNN_PARTS1(ATTR)
    MPCNN_PARTS1_WIDE(ATTR)
    MPCNN_PARTS1_ALL(ATTR)
#undef ATTR
    return e;
}

}  // namespace mpcnn
