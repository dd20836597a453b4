// Instances of wgrad_parts_kernel: row tiles per wave.
#include "kernels_wgrad_parts.hpp"
#include "launchers.hpp"

namespace mpcnn {
namespace {
#define INSTANCES(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9)
}  // namespace

template <typename T>
bool launch_wgrad_parts(const WgradPartsArgs& a, int PM, dim3 grid, size_t lds, hipStream_t st)
{
#define CASE(n) if (PM == n) { wgrad_parts_kernel<n, T><<<grid, kWpThreads, lds, st>>>(a); return true; }
    INSTANCES(CASE)
#undef CASE
    return false;
}
template bool launch_wgrad_parts<float>(const WgradPartsArgs&, int, dim3, size_t, hipStream_t);
template bool launch_wgrad_parts<bf16>(const WgradPartsArgs&, int, dim3, size_t, hipStream_t);

template <typename T>
hipError_t wgrad_parts_attrs()
{
    hipError_t e = hipSuccess;
#define ATTR(n)                                                                              \
    if (e == hipSuccess)                                                                     \
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&wgrad_parts_kernel<n, T>),    \
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    INSTANCES(ATTR)
#undef ATTR
    return e;
}
template hipError_t wgrad_parts_attrs<float>();
template hipError_t wgrad_parts_attrs<bf16>();

}  // namespace mpcnn
