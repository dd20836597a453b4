// Repacking of a layer's parameters into the operand order of the matrix-core convolution
// kernels (forward and data gradient; Method, forward and backward of layer C).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels_conv_parts.hpp"

namespace mpcnn {

// The packs of conv_parts_kernel, P parts per number: in step order, 16-channel chunks and the taps of each,
//   Q[ch*k*k2 + tap][part][g][o][s] = part of W[..][16*ch + 8*g + s][..], s < 8.
// One thread: one (step, g, o), 8 numbers and P 128-bit stores.  All layers and both directions in one launch: a
// training step packs after every update, and each of a net's 6 or 8 packs by itself took a launch's
// 4-7 us for well under 1 us of work.
constexpr int kMaxPackSegs = 64;
struct PackSeg {
    long w_off, q_off;    // first number of the layer's parameters; first float of the pack
    int kk, Ci, Co, RPad, OPad, dgrad, block0;
};
struct PackArgs {
    const float* W;
    float* Q;
    int n_seg, total_blocks;
    PackSeg seg[kMaxPackSegs];
};
template <int P>
__global__ __launch_bounds__(256) void pack_parts_kernel(PackArgs a)
{
    int si = 0;
    while (si + 1 < a.n_seg && (int)blockIdx.x >= a.seg[si + 1].block0) ++si;
    const PackSeg& sg = a.seg[si];
    const float* __restrict__ W = a.W + sg.w_off;
    bf16* __restrict__ Q = reinterpret_cast<bf16*>(a.Q + sg.q_off);
    const int kk = sg.kk, Ci = sg.Ci, Co = sg.Co, OPad = sg.OPad, dgrad = sg.dgrad;
    const int steps = kk * (sg.RPad / 16);
    const long total = (long)steps * 2 * OPad, e = (long)((int)blockIdx.x - sg.block0) * 256 + threadIdx.x;
    if (e < total) {
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
            if constexpr (P == 3) v *= kPartsUp;
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
            for (int again = step + steps; again < steps + parts_ahead(P); again += steps)   // the ring's lead past the last step
                *reinterpret_cast<bf16x8_t*>(Q + ((((long)again * P + i) * 2 + g) * OPad + oo) * 8) = o;
        }
    }
}

// Parameters or gradients between the device order (layer by layer W[tap][c][o], b[o]) and the host order
// (W[o][c][tap], b[o]).  `host` is pinned host memory, accessed in order; the scattered side is the device's, which
// its L2 holds.  blockIdx.y picks the layer, so that its place and sizes are uniform (looked up per number they are
// loads of the argument segment, one after the other).  On the host the same permutation of 90 K numbers took about 60 us, the copy through pageable
// memory another 20.
constexpr int kMaxParamSegs = 48;
struct ParamOrder {
    long off[kMaxParamSegs + 1];          // first number of every layer with parameters; the total behind the last
    int ci[kMaxParamSegs], co[kMaxParamSegs], kk[kMaxParamSegs];
    int n_seg;
};
__global__ void params_order_kernel(float* __restrict__ dev, float* __restrict__ host, ParamOrder a, int to_host)
{
    const int s = blockIdx.y;
    const long off = a.off[s], n = a.off[s + 1] - off;
    const int ci = a.ci[s], co = a.co[s], kk = a.kk[s];
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
        long j = i;                       // biases keep their place
        if (i < (long)co * ci * kk) {
            const int q = (int)(i / kk), t = (int)(i - (long)q * kk), o = q / ci, c = q - o * ci;
            j = ((long)t * ci + c) * co + o;
        }
        if (to_host) host[off + i] = dev[off + j];
        else dev[off + j] = host[off + i];
    }
}

// A few numbers that travel with the launch, written in place
constexpr int kCarried = 960;
struct CarriedNumbers { int n; float v[kCarried]; };
__global__ void write_numbers_kernel(float* __restrict__ dst, CarriedNumbers c)
{
    for (int i = threadIdx.x; i < c.n; i += blockDim.x) dst[i] = c.v[i];
}

}  // namespace mpcnn
