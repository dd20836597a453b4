// Powers of two that bring numbers into the range of fp16, for kernels that work on fp16 parts of fp32 numbers (2^-24 to 2^16).
//
// Activations of squashing functions are at most 1 in size: 2^14 times as large, or as they are (kernels_conv_parts.hpp).  tanh's are
// multiples of some 2^-24 (storage.hpp, squash); logistic ones keep their precision however small they are. Weights: a layer's largest
// magnitude is found when its weights are packed (kernels_pack.hpp). Deltas may have any size.  Whoever writes a tensor of them notes the
// largest magnitude it has written, as the bits of |x| (which as unsigned numbers have the same order): each workgroup stores one word into
// the caller's workspace, a reader takes the largest of the words.  Every word is stored in every pass: nothing to clear, and no atomics
// (2048 waves that end together take 20 us to meet in one word).  A word at or above kNoPeak, as an infinity leaves it or a writer whose
// weights may put maps too far below each other, says that the tensor does not suit fp16 parts of one power of two.  In logistic nets
// the weight gradient looks at the maps as well (kernels_wgrad_parts.hpp).  NaN is passed over: it is one in any number of parts, and so is
// every sum it belongs to.
#pragma once
#include <hip/hip_runtime.h>

namespace mpcnn {

constexpr unsigned kNoPeak = 0x7f800000u;      // infinity
constexpr int kActRaise = 14;
// Second parts are raised by 2^11 more, to the size of the first: numbers down to 2^-28 of the tensor's largest then keep all bits that two
// parts hold, smaller ones lose those below 2^-51 of it (2^-16 and 2^-40 without).  Their products go to an accumulator of their own
// (kernels_conv_parts.hpp) or have a partner that much smaller (kernels_wgrad_parts.hpp: deltas; its inputs' second parts stay as they are).
constexpr float kLowUp = 0x1p11f, kLowDown = 0x1p-11f;
constexpr int kSmallOctaves = 26;              // weights that far below the largest are counted as small (weights_wide)
constexpr int kDeltaWords = 2048;              // of a tensor, at most

__device__ __forceinline__ unsigned bits_of(float x) { return __builtin_bit_cast(unsigned, x); }
__device__ __forceinline__ float larger(float peak, float x) { return fmaxf(peak, fabsf(x)); }   // (not a NaN)

// The largest of the wave's values (all lanes active)
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned larger_moved(unsigned m)
{
    const unsigned o = (unsigned)__builtin_amdgcn_update_dpp((int)m, (int)m, CTRL, ROWS, 0xf, false);
    return o > m ? o : m;
}
__device__ __forceinline__ unsigned wave_largest(unsigned m)
{
    m = larger_moved<0x128, 0xf>(m);   // row_ror:8, 4, 2, 1
    m = larger_moved<0x124, 0xf>(m);
    m = larger_moved<0x122, 0xf>(m);
    m = larger_moved<0x121, 0xf>(m);
    m = larger_moved<0x142, 0xa>(m);   // row_bcast:15 into rows 1 and 3,
    m = larger_moved<0x143, 0xc>(m);   // row_bcast:31 into rows 2 and 3
    return (unsigned)__builtin_amdgcn_readlane((int)m, 63);
}
// The largest of a tensor's words (called by whole waves; one trip for 512 words)
__device__ __forceinline__ unsigned peak_of(const unsigned* words, int n)
{
    unsigned m = 0;
    for (int i = 0; i < n; i += 512) {
        unsigned v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int at = i + 64 * j + (threadIdx.x & 63);
            v[j] = words[at < n ? at : 0];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) m = v[j] > m ? v[j] : m;
    }
    return wave_largest(m);
}
// The exponent that takes numbers of at most `peak` * 2^margin below 2^15
__device__ __forceinline__ int raise_of(unsigned peak, int margin)
{
    const int r = 14 - ((int)(peak >> 23) - 127 + margin);
    return r < -126 ? -126 : r > 127 ? 127 : r;
}
__device__ __forceinline__ float power_of_two(int e) { return __builtin_bit_cast(float, (unsigned)(e + 127) << 23); }   // e = -126 .. 127

// Factors first and second with first * second = 2^-up, up = -252 .. 254 (to the last, 2^-126 twice: there is nothing left of a sum)
struct Lower { float first, second; };
__device__ __forceinline__ Lower lower_by(int up)
{
    const int a = up < -126 ? -126 : up > 126 ? 126 : up;
    return {power_of_two(-a), power_of_two(a - up < -126 ? -126 : a - up)};
}

}  // namespace mpcnn
