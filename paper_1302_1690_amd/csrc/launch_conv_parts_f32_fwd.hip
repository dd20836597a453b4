// Instances of conv_parts_kernel for fp32 storage, forward.
#include "kernels_conv_parts.hpp"
#include "launchers.hpp"

namespace mpcnn {
namespace {
typedef float T;
#define INSTANCES(X) \
    X(1, 4, 1, 1) X(1, 4, 1, 2) X(2, 2, 1, 1) X(2, 2, 1, 2) X(1, 4, 2, 2) X(4, 1, 1, 2) X(4, 1, 1, 4) X(2, 2, 2, 2)
}  // namespace

bool launch_conv_parts_f32_fwd(const ConvArgs& a, int CB, const PartsInstance& in, dim3 grid, size_t lds, hipStream_t st)
{
#define CASE(o, p, mo, mp)                                                                                          \
    if (in.WO == o && in.WP == p && in.MO == mo && in.MP == mp) {                                                   \
        if (CB == 16) conv_parts_kernel<T, false, 16, o, p, mo, mp><<<grid, kPartsThreads, lds, st>>>(a);          \
        else conv_parts_kernel<T, false, 32, o, p, mo, mp><<<grid, kPartsThreads, lds, st>>>(a);                   \
        return true;                                                                                                \
    }
    INSTANCES(CASE)
#undef CASE
    return false;
}

hipError_t conv_parts_attrs_f32_fwd()
{
    hipError_t e = hipSuccess;
#define ATTR(...)                                                                            \
    if (e == hipSuccess)                                                                     \
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&__VA_ARGS__),                 \
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)
#define BOTH(o, p, mo, mp) ATTR(conv_parts_kernel<T, false, 16, o, p, mo, mp>); ATTR(conv_parts_kernel<T, false, 32, o, p, mo, mp>);
    INSTANCES(BOTH)
#undef BOTH
#undef ATTR
    return e;
}

}  // namespace mpcnn
