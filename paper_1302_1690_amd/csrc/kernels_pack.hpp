// Repacking of a layer's parameters into the operand order of the matrix-core convolution
// kernels (forward and data gradient; Method, forward and backward of layer C).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels_conv_parts.hpp"   // the order of its steps
#include "storage.hpp"

namespace mpcnn {

// Repack W[tap][c][o] (+ bias row) into the operand order of conv_mfma_kernel, G lane groups:
//   forward : reduce over c, outputs o:  P[tap*nch + ch][g][o][s]  = W[tap][4G*ch+4g+s][o]
//   dgrad   : reduce over o, outputs c:  P[tap'*nch + ch][g][c][s] = W[k*k-1-tap'][c][4G*ch+4g+s]
// (taps reversed: the data gradient at x collects deltas at x - u*d).  Padding is zero.
__global__ void pack_weights_kernel(const float* __restrict__ W, float* __restrict__ P, int kk,
                                    int Ci, int Co, int RPad, int OPad, int G, int dgrad)
{
    const int nch = RPad / (4 * G);
    long total = (long)kk * nch * G * OPad * 4;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (long)gridDim.x * blockDim.x) {
        int s = (int)(e & 3);
        long q = e >> 2;
        int oo = (int)(q % OPad); q /= OPad;
        int g = (int)(q % G); q /= G;
        int ch = (int)(q % nch);
        int tap = (int)(q / nch);
        int r = 4 * G * ch + 4 * g + s;  // index along the reduced dimension
        float v = 0.f;
        if (!dgrad) {
            if (r < Ci && oo < Co) v = W[((long)tap * Ci + r) * Co + oo];
        } else {
            if (r < Co && oo < Ci) v = W[((long)(kk - 1 - tap) * Ci + oo) * Co + r];
        }
        P[e] = v;
    }
}

// The same packs for the bf16 matrix instruction (v_mfma_f32_32x32x16_bf16: lane l supplies
// 8 consecutive reduction indices, 8*(l/32) .. +7, of row / column l%32): 8 channels per item,
//   P[tap*nch + ch][g][o][s] = W[..][16*ch + 8*g + s][..], s < 8, as bf16.
__global__ void pack_weights_bf16_kernel(const float* __restrict__ W, bf16* __restrict__ P, int kk,
                                         int Ci, int Co, int RPad, int OPad, int dgrad)
{
    const int nch = RPad / 16;
    long total = (long)kk * nch * 2 * OPad * 8;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (long)gridDim.x * blockDim.x) {
        int s = (int)(e & 7);
        long q = e >> 3;
        int oo = (int)(q % OPad); q /= OPad;
        int g = (int)(q & 1); q >>= 1;
        int ch = (int)(q % nch);
        int tap = (int)(q / nch);
        int r = 16 * ch + 8 * g + s;  // index along the reduced dimension
        float v = 0.f;
        if (!dgrad) {
            if (r < Ci && oo < Co) v = W[((long)tap * Ci + r) * Co + oo];
        } else {
            if (r < Co && oo < Ci) v = W[((long)(kk - 1 - tap) * Ci + oo) * Co + r];
        }
        P[e] = (bf16)v;
    }
}

// The packs of conv_parts_kernel, P parts per number: steps in the order that kernel takes them - channel
// blocks of CB, in a block the taps, in a tap its 16-channel chunks -
//   Q[step][part][g][o][s] = part of W[..][16*ch + 8*g + s][..], s < 8.
// One thread: one (step, g, o), 8 numbers and P 128-bit stores.
template <int P>
__global__ void pack_parts_kernel(const float* __restrict__ W, bf16* __restrict__ Q, int kk, int Ci, int Co,
                                  int RPad, int OPad, int CB, int dgrad)
{
    const int nsub_full = CB / 16, blk_steps = parts_block_steps(P, kk, nsub_full);
    const long total = (long)parts_steps(P, CB, kk, RPad) * 2 * OPad;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (long)gridDim.x * blockDim.x) {
        const int oo = (int)(e % OPad);
        const int g = (int)((e / OPad) & 1), step = (int)(e / (2 * OPad));
        const int blk = step / blk_steps, r = step - blk * blk_steps;
        const int left = RPad / 16 - blk * nsub_full, nsub = left < nsub_full ? left : nsub_full;
        const int tap = r / nsub, ch = blk * nsub_full + (r - tap * nsub);   // (tap == kk: the step of zeros that fills a unit)
        bf16 parts[P][8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int c = 16 * ch + 8 * g + s;   // index along the reduced dimension
            float v = 0.f;
            if (tap >= kk) v = 0.f;
            else if (!dgrad) {
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
