// Repacking of a layer's parameters into the operand order of the matrix-core convolution
// kernels (forward and data gradient; Method, forward and backward of layer C).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "storage.hpp"

namespace mpcnn {

// The packs of conv_parts_kernel, P parts per number: in step order, 16-channel chunks and the taps of each,
//   Q[ch*k*k2 + tap][part][g][o][s] = part of W[..][16*ch + 8*g + s][..], s < 8.
// One thread: one (step, g, o), 8 numbers and P 128-bit stores.
template <int P>
__global__ void pack_parts_kernel(const float* __restrict__ W, bf16* __restrict__ Q, int kk, int Ci, int Co,
                                  int RPad, int OPad, int dgrad)
{
    const long total = (long)kk * (RPad / 16) * 2 * OPad;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (long)gridDim.x * blockDim.x) {
        const int oo = (int)(e % OPad);
        const int g = (int)((e / OPad) & 1), step = (int)(e / (2 * OPad));
        const int ch = step / kk, tap = step - ch * kk;
        bf16 parts[P][8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int c = 16 * ch + 8 * g + s;   // index along the reduced dimension
            float v = 0.f;
            if (!dgrad) {
                if (c < Ci && oo < Co) v = W[((long)tap * Ci + c) * Co + oo];
            } else {
                if (c < Co && oo < Ci) v = W[((long)(kk - 1 - tap) * Ci + oo) * Co + c];
            }
#pragma unroll
            for (int i = 0; i < P; ++i) {        // v = the sum of its parts, exactly
                parts[i][s] = (bf16)v;
                v -= (float)parts[i][s];
            }
        }
#pragma unroll
        for (int i = 0; i < P; ++i) {
            typedef bf16 bf16x8_t __attribute__((ext_vector_type(8)));
            bf16x8_t o;
#pragma unroll
            for (int s = 0; s < 8; ++s) o[s] = parts[i][s];
            *reinterpret_cast<bf16x8_t*>(Q + ((((long)step * P + i) * 2 + g) * OPad + oo) * 8) = o;
        }
    }
}

}  // namespace mpcnn
