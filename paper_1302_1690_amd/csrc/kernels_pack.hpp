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
// Two parts (fp16) are of numbers raised by the layer's own power of two, which weight_peaks_kernel prepares: it leaves the largest
// magnitudes of kPeakParts stretches of every layer's weights, pack_weights_kernel takes the largest of those, leaves it in the layer's words
// (conv_parts_kernel reads them) and counts there the numbers whose last bits two parts do not hold.
constexpr int kMaxPackSegs = 64, kPeakParts = 16, kPeakWords = kPeakParts + 2;   // a layer's words: peak, small numbers, the stretches' peaks
struct PackSeg {
    long w_off, q_off;    // first number of the layer's parameters; first float of the pack
    unsigned* words;      // the layer's peak words; null where nothing has two parts
    int kk, Ci, Co, RPad, OPad, dgrad, block0, parts, first;   // first: this segment notes peak and small numbers for its layer
};
struct PackArgs {
    const float* W;
    float* Q;
    int n_seg, total_blocks;
    PackSeg seg[kMaxPackSegs];
};

// blockIdx.y: segment (its layer, if it is the first of it), blockIdx.x: stretch
__global__ __launch_bounds__(256) void weight_peaks_kernel(PackArgs a)
{
    const PackSeg& sg = a.seg[blockIdx.y];
    if (!sg.first) return;
    const float* __restrict__ W = a.W + sg.w_off;
    const int n = sg.kk * sg.Ci * sg.Co;                       // (below 2^31 bytes: wider layers have no packs)
    float m = 0.f;
#pragma unroll 4
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += kPeakParts * 256) m = larger(m, W[i]);
    __shared__ unsigned most;
    if (threadIdx.x == 0) most = 0;
    __syncthreads();
    atomicMax(&most, bits_of(m));
    __syncthreads();
    if (threadIdx.x == 0) {
        sg.words[2 + blockIdx.x] = most;
        if (blockIdx.x == 0) sg.words[1] = 0;
    }
}

template <int P>
__device__ __forceinline__ void pack_segment(const PackArgs& a, const PackSeg& sg)
{
    typedef typename std::conditional<P == 2, _Float16, bf16>::type Part;
    typedef Part Part8 __attribute__((ext_vector_type(8)));
    const float* __restrict__ W = a.W + sg.w_off;
    Part* __restrict__ Q = reinterpret_cast<Part*>(a.Q + sg.q_off);
    const int kk = sg.kk, Ci = sg.Ci, Co = sg.Co, OPad = sg.OPad, dgrad = sg.dgrad;
    const int steps = kk * (sg.RPad / 16);
    const long total = (long)steps * 2 * OPad, e = (long)((int)blockIdx.x - sg.block0) * 256 + threadIdx.x;
    float up = P == 3 ? kPartsUp : 1.f;
    unsigned peak = 0;
    if (P == 2 || sg.first) {
        for (int i = 0; i < kPeakParts; ++i) peak = sg.words[2 + i] > peak ? sg.words[2 + i] : peak;
        if (P == 2) up = power_of_two(raise_of(peak, 0));
        if (sg.first && (int)blockIdx.x == sg.block0 && threadIdx.x == 0) sg.words[0] = peak;
    }
    int small = 0;
    if (e < total) {
        const int oo = (int)(e % OPad);
        const int g = (int)((e / OPad) & 1), step = (int)(e / (2 * OPad));
        const int ch = step / kk, tap = step - ch * kk;
        Part parts[P][8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int c = 16 * ch + 8 * g + s;   // index along the reduced dimension
            float v = 0.f;
            if (!dgrad) {
                if (c < Ci && oo < Co) v = W[((long)tap * Ci + c) * Co + oo];
            } else {
                if (c < Co && oo < Ci) v = W[((long)(kk - 1 - tap) * Ci + oo) * Co + c];
            }
            if (sg.first && peak < kNoPeak) small += v != 0.f && bits_of(fabsf(v)) < peak && (peak - bits_of(fabsf(v))) >> 23 >= kSmallOctaves;
            if constexpr (P != 1) v *= up;
#pragma unroll
            for (int i = 0; i < P; ++i) {        // three parts: v is their sum, exactly
                parts[i][s] = (Part)v;
                v -= (float)parts[i][s];
                if constexpr (P == 2) v *= kLowUp;
            }
        }
#pragma unroll
        for (int i = 0; i < P; ++i) {
            Part8 o;
#pragma unroll
            for (int s = 0; s < 8; ++s) o[s] = parts[i][s];
            *reinterpret_cast<Part8*>(Q + ((((long)step * P + i) * 2 + g) * OPad + oo) * 8) = o;
            for (int again = step + steps; again < steps + parts_ahead(P); again += steps)   // the ring's lead past the last step
                *reinterpret_cast<Part8*>(Q + ((((long)again * P + i) * 2 + g) * OPad + oo) * 8) = o;
        }
    }
    if (__any(small)) {                          // (numbers of a wave together: of a wide layer nearly all are small)
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) small += __shfl_xor(small, s);
        if ((threadIdx.x & 63) == 0) atomicAdd(sg.words + 1, (unsigned)small);
    }
}
template <bool BF16>
__global__ __launch_bounds__(256) void pack_weights_kernel(PackArgs a)
{
    int si = 0;
    while (si + 1 < a.n_seg && (int)blockIdx.x >= a.seg[si + 1].block0) ++si;
    const PackSeg& sg = a.seg[si];
    if constexpr (BF16) pack_segment<1>(a, sg);
    else if (sg.parts == 2) pack_segment<2>(a, sg);
    else pack_segment<3>(a, sg);
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
