// Host-side launch functions of the matrix-core kernel families.  Each family's template
// instances are compiled in a translation unit of its own (launch_*.hip), so that the library
// builds in parallel; mpcnn.hip picks the instance through these plain functions.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels_mfma.hpp"
#include "kernels_wgrad.hpp"
#include "kernels_wgrad_parts.hpp"

namespace mpcnn {

// Forward / data gradient: conv_parts_kernel (kernels_conv_parts.hpp): CB channels per block, WO x WP waves, MO x MP result tiles per wave.  The
// instances that are built (wide blocks only where a tile is small enough for them: 64 channels, 192 halo positions
// with fp32 storage and 384 with bf16; 128 channels, 192):
struct PartsInstance { int CB, WO, WP, MO, MP; };
#define MPCNN_PARTS3(X) /* fp32 storage (two accumulators per tile: no room for four tiles) */                         \
    X(16, 1, 4, 1, 1) X(16, 1, 4, 1, 2) X(16, 2, 2, 1, 1) X(16, 2, 2, 1, 2) X(16, 4, 1, 1, 2)                           \
    X(32, 1, 4, 1, 1) X(32, 1, 4, 1, 2) X(32, 2, 2, 1, 1) X(32, 2, 2, 1, 2) X(32, 4, 1, 1, 2)                           \
    X(64, 1, 4, 1, 1) X(64, 2, 2, 1, 1) X(64, 2, 2, 1, 2) X(64, 4, 1, 1, 2)
#define MPCNN_PARTS1(X) /* bf16 storage (two channel tiles: 2 x 2 per wave where there is a choice, 4 operands per 4 instructions, not 5) */ \
    X(16, 1, 4, 1, 2) X(16, 1, 4, 1, 4) X(16, 2, 2, 1, 2) X(16, 1, 4, 2, 2) X(16, 4, 1, 1, 4)                           \
    X(32, 1, 4, 1, 2) X(32, 1, 4, 1, 4) X(32, 2, 2, 1, 2) X(32, 1, 4, 2, 2)                                             \
    X(32, 4, 1, 1, 2) X(32, 4, 1, 1, 4) X(32, 2, 2, 2, 2)                                                               \
    X(64, 1, 4, 1, 2) X(64, 2, 2, 1, 2) X(64, 1, 4, 2, 2) X(64, 4, 1, 1, 2) X(64, 4, 1, 1, 4) X(64, 2, 2, 2, 2)          \
    X(128, 2, 2, 1, 2) X(128, 4, 1, 1, 2) X(128, 4, 1, 1, 4) X(128, 2, 2, 2, 2)
// bf16 storage, eight tiles per wave: large maps (two workgroups per compute unit instead of three; never by a tiling hint)
#define MPCNN_PARTS1_WIDE(X) X(32, 1, 4, 2, 4) X(64, 1, 4, 2, 4) X(32, 2, 2, 2, 4) X(64, 2, 2, 2, 4) X(128, 2, 2, 2, 4)
// bf16 storage, forward, 161 .. 256 channels in one workgroup instead of two groups that bring the same halo and write halves of the same lines
// (128 -> 200, 2 x 2, 2 x 2048 x 2048: 3020 -> 2706 us; 2 x 200 x 300 no slower).  Five tiles keep three of the four waves busy: whole training
// steps of 64 -> 132, 3 x 3, 2 x 1400 x 1407 4295 -> 4466, 128 -> 132, 2 x 2 5036 -> 5139, 64 -> 160 4344 -> 4386, 128 -> 160 5003 -> 4986.
#define MPCNN_PARTS1_ALL(X) X(64, 4, 1, 2, 4) X(128, 4, 1, 2, 4)
// Forward with the class layer behind it, nothing kept: all channels in one workgroup (a hidden layer of 65 .. 128, 129 .. 256 units; eight waves
// where four of fp32 storage's tiles do not hold them)
#define MPCNN_HEAD3(X) X(16, 4, 1, 1, 2) X(32, 4, 1, 1, 2) X(64, 4, 1, 1, 2) X(32, 8, 1, 1, 2) X(64, 8, 1, 1, 2)
#define MPCNN_HEAD1(X) X(32, 2, 2, 2, 2) X(64, 2, 2, 2, 2) X(64, 2, 2, 2, 4) X(32, 4, 1, 2, 2) X(64, 4, 1, 2, 2) X(64, 4, 1, 2, 4)
#define MPCNN_PARTS_ROW(cb, wo, wp, mo, mp) {cb, wo, wp, mo, mp},
constexpr PartsInstance kParts3[] = {MPCNN_PARTS3(MPCNN_PARTS_ROW)};
constexpr PartsInstance kParts1[] = {MPCNN_PARTS1(MPCNN_PARTS_ROW) MPCNN_PARTS1_WIDE(MPCNN_PARTS_ROW)};
constexpr PartsInstance kParts1Fwd[] = {MPCNN_PARTS1(MPCNN_PARTS_ROW) MPCNN_PARTS1_WIDE(MPCNN_PARTS_ROW) MPCNN_PARTS1_ALL(MPCNN_PARTS_ROW)};
constexpr PartsInstance kHead3[] = {MPCNN_HEAD3(MPCNN_PARTS_ROW)};
constexpr PartsInstance kHead1[] = {MPCNN_HEAD1(MPCNN_PARTS_ROW)};
#undef MPCNN_PARTS_ROW
bool launch_conv_head_f32(const ConvArgs& a, const PartsInstance& in, dim3 grid, size_t lds, hipStream_t st);
bool launch_conv_head_b16(const ConvArgs& a, const PartsInstance& in, dim3 grid, size_t lds, hipStream_t st);
bool launch_conv_parts_f32_fwd(const ConvArgs& a, const PartsInstance& in, dim3 grid, size_t lds, hipStream_t st);
bool launch_conv_parts_f32_back(const ConvArgs& a, const PartsInstance& in, dim3 grid, size_t lds, hipStream_t st);
bool launch_conv_parts_b16_fwd(const ConvArgs& a, const PartsInstance& in, dim3 grid, size_t lds, hipStream_t st);
bool launch_conv_parts_b16_back(const ConvArgs& a, const PartsInstance& in, dim3 grid, size_t lds, hipStream_t st);
hipError_t conv_parts_attrs_f32_fwd();
hipError_t conv_parts_attrs_f32_back();
hipError_t conv_parts_attrs_b16_fwd();
hipError_t conv_parts_attrs_b16_back();

// Weight gradient (kernels_wgrad.hpp, kernels_wgrad_bf16.hpp); a.mw selects the instance.  fp32 storage comes here for channel counts
// that are no multiple of 4 and for little work (below 4e7 operations), else launch_wgrad_parts serves it.
bool launch_wgrad_f32(const WgradArgs& a, int hl, dim3 grid, size_t lds, hipStream_t st);
bool launch_wgrad_b16(const WgradArgs& a, int hl, dim3 grid, size_t lds, hipStream_t st);
bool launch_wgrad_bm(const WgradArgs& a, int nch, dim3 grid, size_t lds, hipStream_t st);
bool launch_wgrad_tr(const WgradArgs& a, int nch, dim3 grid, size_t lds, hipStream_t st);   // kernels_wgrad_tr.hpp
template <typename T> bool launch_wgrad_parts(const WgradPartsArgs& a, int PM, dim3 grid, size_t lds, hipStream_t st);   // kernels_wgrad_parts.hpp
template <typename T> hipError_t wgrad_parts_attrs();

// Kernels that may ask for more than 64 KiB of dynamic LDS must say so once per device.
hipError_t wgrad_attrs_f32();
hipError_t wgrad_attrs_b16();

}  // namespace mpcnn
