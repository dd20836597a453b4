// Weight gradient of one dilated convolution with fp32 storage on v_mfma_f32_32x32x16_f16, every fp32 number as the sum of two fp16 parts,
// three products each, or, where the numbers do not suit fp16 (ranges.hpp), on v_mfma_f32_32x32x16_bf16 in three bf16 parts, six products
// each (kernels_conv_parts.hpp has the arithmetic of both).  The accumulator's roundings, half as many with two parts, make up for the bits
// that two parts lose once a wave adds some 144 positions; shorter chains take three parts (plan_wgrad_parts has the errors on both sides).
//
// bf16 storage: one part, one product, raw copies, for the layers that wgrad_tr_kernel does not take (input channels no multiple of 32, or
// 32 maps and fewer, which went to the fp32 instruction).  Bound by its operand reads: PM + 1 of a kilobyte for PM products, half of the
// LDS's rate times the matrix pipes'.  3 x 501 x 389, 16 -> 32, 5 x 5: 150 -> 48 us (94 -> 295 TFLOP/s); error in the 2-norm on 1500 x 1400
// 4.1e-8 -> 2.7e-8, 48 -> 64 k4 on 700 x 640 3.9e-8 -> 3.0e-8, smaller maps 2.3e-8 to 3.2e-8 both.
//
// Range of two parts.  One accumulator takes all three products, so y1, a delta's second part, can only be 2^11 times as large (as in
// kernels_conv_parts.hpp) where its partner is 2^-11 as large: x0 2^-11 is made in registers, four multiplications of eight halves for
// three instructions of 32 cycles.  Deltas keep their bits down to 2^-28 of the tensor's largest, so a map of them that far below the
// others is as good as they are.  Maps below that come from weights that far apart, of which their writers tell (ranges.hpp), or from
// slopes: tanh's are 2^-23 at least and off by as much, logistic ones are looked at (logistic_maps_reach).  The inputs' second parts stay
// as they are: tanh leaves multiples of 2^-24, logistic maps are looked at as well.
//
// Accuracy.  All six products go to one accumulator, as there is no room for two, and the instruction's results are a little too low
// whatever their sign: over the slabs of a large map such offsets add up where roundings cancel.  So every other slab has the signs of its
// deltas turned, and its sums' signs turned back.  Error of the gradient in the 2-norm, fp32 instruction / without turns / now: 32 -> 64 k5
// on 1024 x 1024 1.3e-7 / 1.8e-7 / 1.0e-7, with cancelling deltas 1.6e-6 / 2.3e-6 / 1.4e-6; 64 -> 128 k3 2.0e-7 / 2.5e-7 / 1.6e-7 and
// 2.8e-6 / 4.5e-6 / 1.9e-6; 128 -> 200 k2 on 700 x 640 2.9e-7 / 1.7e-7 / 1.1e-7 and 1.1e-6 / 1.2e-6 / 6.3e-7.
//
//   dW[tap][c][o] = sum over positions of in[pos + tap][c] * dY[pos][o]        (Alg. 2)
//
// As in the other weight-gradient kernels the result is tiny and the contraction runs over all positions:
// blockIdx.x = slab of tiles, the workgroup's share of the result stays in accumulators for the whole
// slab, reduce_all_kernel adds the slabs.  The instruction contracts 16 positions, a lane supplying 8 of
// them for ONE gradient row or output channel; the transposing LDS read (ds_read_b64_tr_b16, see
// kernels_wgrad_tr.hpp) gives that from channels-last tiles.
//
// Layout (three parts; two: 64 bytes per position, planes shifted by 32; one: 32 bytes per position, planes by 128 mod 256).  Both tiles
// sit in LDS as planes of 16 channels, [plane][position][part][16 channels] (96 bytes per position: the 16 lanes that read 4 positions
// together meet no bank twice, and with a plane pitch of 128 mod 256 bytes neither do the 32 of two planes; counters, stores included,
// still read 26-42 % of the LDS cycles as conflicts).  Parts, the second half of an operand and successive chunks are immediates.  A
// gradient row tile is two UNITS of 16 rows, a unit being (plane, tap): the two halves of the lanes address their units separately, so
// 16-channel layers fill row tiles with two taps and 100 channels pad to 112, not 128.
//
// Waves.  Eight waves = wm (row tiles) x wn (column tiles) x wk (positions), each with PM x 1 result
// tiles: a chunk of 16 positions is PM + 1 operands of three parts for 6 PM instructions, 70 bytes per cycle of
// LDS reads for PM = 8 with the matrix pipes full.  The operands of row tile p + 1 are fetched while p is multiplied.
// Two LDS buffers: tile t + 1 is split into parts and written while tile t is multiplied, one barrier per tile;
// of the two waves of a SIMD one writes before it multiplies and the other after, so that one's
// conversions lie under the other's instructions.
//
// Measured on the deep net (1 x 1024 x 1024, 32 -> 64 k5, 64 -> 64 k5, 64 -> 128 k3, 128 -> 200 k2), three parts -> two: 522, 1005, 710,
// 1325 us -> 324, 615, 456, 866 (322, 327, 305, 211 TFLOP/s); errors 1.04e-7, 1.61e-7 (k3), 1.09e-7 (k2, 700 x 640) -> 1.01e-7, 1.57e-7,
// 1.01e-7, with cancelling deltas 1.36e-6, 1.93e-6, 6.3e-7 -> 1.28e-6, 1.72e-6, 5.5e-7. Before (fp32 instruction) and in three parts: 985,
// 1780, 1210, 2030 us -> 512, 975, 700, 1293 us (204, 206, 199, 142 TFLOP/s; what the split instruction sustains on random data is 240-260,
// the last layer pads 200 maps to 256 and 59 columns to 64).  Matrix pipes busy 47-67 %. Splitting numbers 2^16 times as large (two
// multiplications per pair more) took 495, 942, 682, 1222 to 506, 980, 699, 1295, in turn on one machine. Little work (below 4e7
// operations) stays on wgrad_mfma_kernel: a launch takes some 6 us more here whatever it computes. The conversions decide the rest: with
// every item's address worked out per tile and numbers converted one by one (480 vector instructions per thread and tile of 32 positions
// instead of 300) it was 575, 1062, 811, 1540.
#pragma once
#include "kernels_conv_parts.hpp"
#include "kernels_wgrad_tr.hpp"

namespace mpcnn {

constexpr int kWpThreads = 512;
constexpr int kWpItems = 4;       // 8-channel items per thread and tile, at most
constexpr int kWpMaxTiles = 9;    // row tiles per wave
__host__ __device__ constexpr int wp_pos(int parts) { return 32 * parts; }   // LDS bytes of a position of one plane

struct WgradPartsArgs {
    const void* in;      // [B][Hi][Wi][Ci]  layer input (fp32, or bf16: the kernel's template parameter T)
    const void* dY;      // [B][Ho][Wo][Co]  delta w.r.t. the layer's pre-activation
    float* partial;      // [slab][group][row tile][column tile][4][64 lanes][4], then [Nt*32] bias sums
    int B, Hi, Wi, Ci, Ho, Wo, Co;
    int k, k2, d, d2;    // filter rows, columns; spacing of rows, columns
    int R, nch;          // tile = R rows x 16*nch columns of one residue class
    int nty, ntx, tiles_total, tiles_per_slab;
    int Nt, RT;          // 32-column tiles of the result; row tiles of a group
    int wm, wn, wk;      // wm * wn * wk = 8
    int ppg, tpg, ntg;   // planes and taps per group; groups along the taps (blockIdx.y = plane group * ntg + tap group)
    const unsigned* dy_peak;             // dY's dy_words words (ranges.hpp), or null: not known, or `in` is no output of a squashing function
    int dy_words, dy_margin;             // dY is at most 2^dy_margin times as large as they say
    const float* out;                    // the layer's outputs if that function is the logistic one, else null
    unsigned mg_nqh, mg_hwp, mg_txp, mg_tpg, mg_k2, mg_ntx, mg_nty, mg_d, mg_d2;   // ceil(2^32 / x)
};

// LDS geometry shared with the host's plan (bytes)
struct WpGeom { int hh, hwp, hplane, dplane, halo_b, buf_b, nh, nd; };   // nh, nd: items of the halo (rounded up to whole waves) and of the delta tile
__host__ __device__ inline WpGeom wp_geom(int R, int nch, int k, int k2, int ppg, int wn, int parts)
{
    WpGeom g;
    g.hh = R + k - 1; g.hwp = 16 * nch + k2 - 1;
    if (parts == 1) {                                                    // positions follow each other by 32 bytes, planes by 128 mod 256
        g.hplane = (g.hh * g.hwp * wp_pos(1) + 127) / 256 * 256 + 128;
        g.dplane = 16 * R * nch * wp_pos(1) + 128;
    } else if (parts == 3) {
        g.hplane = (((g.hh * g.hwp + 3) / 8) * 8 + 4) * wp_pos(3);       // positions = 4 mod 8, at least hh * hwp
        g.dplane = (16 * R * nch + 4) * wp_pos(3);
    } else {                                                             // a plane's 32 bytes fall between another's (and 64 to drop items into)
        g.hplane = g.hh * g.hwp * wp_pos(2) + 96;
        g.dplane = 16 * R * nch * wp_pos(2) + 96;
    }
    g.halo_b = 2 * wn * g.dplane;
    g.buf_b = g.halo_b + ppg * g.hplane;
    g.nh = (g.hh * g.hwp * 2 * ppg + 63) / 64 * 64;
    g.nd = 16 * R * nch * 4 * wn;
    return g;
}

// ---- logistic nets in two parts.  A map of logistic units that are off has outputs, and slopes and so deltas, as small as it likes, with
// all their bits (tanh leaves multiples of 2^-24, and a slope is off by as much).  A sample of positions finds such maps, and three parts are
// taken: input maps that do not reach 2^-12 and maps of the layer's own outputs that do not reach 2^-20.  (Not of deltas: few positions may
// have any.)  3 us of a launch.
constexpr int kWpSamples = 8;
constexpr float kWpLeastIn = 0x1p-12f, kWpLeastOut = 0x1p-20f;
constexpr int kWpSampled = 2048;  // most channels of both: their words lie where the first tiles go

// A sample of a tensor [positions][C]: this thread's quad of the `quads` from channel c0 on (up to 512; C a multiple of 4) at kWpSamples of kWpSamples * (512 /
// quads) positions spread over it
struct Sample { v4f v[kWpSamples]; unsigned quad; bool any; };
__device__ __forceinline__ Sample sample_maps(const float* t, long positions, int C, int c0, int quads)
{
    Sample s;
    const unsigned rows = kWpThreads / quads, row = threadIdx.x / (unsigned)quads;
    s.quad = threadIdx.x - row * quads;
    const int c = c0 + 4 * (int)s.quad;
    s.any = row < rows && c < C;
    const float stretch = (float)positions / (float)(kWpSamples * rows);
#pragma unroll
    for (int j = 0; j < kWpSamples; ++j) {            // (all at once)
        // (inside their stretches the positions are irregular: in step with no map's rows or columns)
        const unsigned n = row + rows * j;
        const long at = (long)(((float)n + (float)(n * 40503u & 0xffffu) * 0x1p-16f) * stretch);
        s.v[j] = s.any ? *reinterpret_cast<const v4f*>(t + (at < positions ? at : positions - 1) * C + c) : (v4f){0.f, 0.f, 0.f, 0.f};
    }
    return s;
}
// Bits of the largest magnitudes, into most[4 quads] (which is clear)
__device__ __forceinline__ void largest_of(const Sample& s, unsigned* most)
{
    if (!s.any) return;
    unsigned m[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < kWpSamples; ++j)
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            const unsigned b = bits_of(s.v[j][z]) & 0x7fffffffu;   // (a NaN is above infinity)
            m[z] = b > m[z] ? b : m[z];
        }
#pragma unroll
    for (int z = 0; z < 4; ++z) atomicMax(most + 4 * s.quad + z, m[z]);
}
// Whether the maps suit two parts (all threads call it; words: LDS)
__device__ __forceinline__ bool logistic_maps_reach(const WgradPartsArgs& a, unsigned* words)
{
    const int c0 = 16 * ((blockIdx.y / a.ntg) * a.ppg), n = a.Ci - c0 < 16 * a.ppg ? a.Ci - c0 : 16 * a.ppg;
    if (n + a.Co > kWpSampled) return false;
    unsigned *const low = words, *const out_most = words + 1, *const in_most = out_most + a.Co;
    for (int i = threadIdx.x; i < 1 + n + a.Co; i += kWpThreads) words[i] = 0;
    __syncthreads();
    for (int q = 0; q < a.Co / 4; q += kWpThreads)
        largest_of(sample_maps(a.out, (long)a.B * a.Ho * a.Wo, a.Co, 4 * q, a.Co / 4 - q < kWpThreads ? a.Co / 4 - q : kWpThreads), out_most + 4 * q);
    for (int q = 0; q < n / 4; q += kWpThreads)
        largest_of(sample_maps(static_cast<const float*>(a.in), (long)a.B * a.Hi * a.Wi, a.Ci, c0 + 4 * q, n / 4 - q < kWpThreads ? n / 4 - q : kWpThreads), in_most + 4 * q);
    __syncthreads();
    bool is = false;
    for (int i = threadIdx.x; i < a.Co; i += kWpThreads) is |= out_most[i] < bits_of(kWpLeastOut);
    for (int i = threadIdx.x; i < n; i += kWpThreads) is |= in_most[i] < bits_of(kWpLeastIn);
    if (is) *low = 1;
    __syncthreads();
    const bool reach = *low == 0;
    __syncthreads();
    return reach;
}

template <int PM, int P, typename T>
__device__ __forceinline__ void wgrad_parts_body(const WgradPartsArgs a, unsigned dy_peak)
{
    constexpr int kWpPos = wp_pos(P);
    constexpr int SI = kWpItems;
    constexpr bool kF32 = sizeof(T) == 4;
    static_assert(kF32 ? P == 2 || P == 3 : P == 1, "parts of the storage type");
    constexpr unsigned ES = sizeof(T);
    const T* const in_t = static_cast<const T*>(a.in);
    const T* const dy_t = static_cast<const T*>(a.dY);
    constexpr unsigned kNone = 0x80000000u;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    char* ldsb = reinterpret_cast<char*>(lds);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = a.wn;
    const int nidx = wave & (wn - 1);
    const int midx = __builtin_amdgcn_readfirstlane((wave / wn) % a.wm);
    const int kidx = __builtin_amdgcn_readfirstlane(wave / (wn * a.wm));
    const WpGeom g = wp_geom(a.R, a.nch, a.k, a.k2, a.ppg, wn, P);
    const int txp = 16 * a.nch;
    const int p0 = (blockIdx.y / a.ntg) * a.ppg, tap0 = (blockIdx.y % a.ntg) * a.tpg;   // first plane, first tap of the group
    const int nt = blockIdx.z * wn + nidx;
    const bool active = midx * PM < a.RT && nt < a.Nt;

    // ---- staging items: it = tid + 512 u; below nh the halo, a whole wave at a time, then the delta tile.  What an item
    // is never changes, so its place is worked out once; a tile inside the tensors (most) takes every load
    // at the item's offset from a scalar base, the others check its coordinates.
    const int nqh = 2 * a.ppg, nqd = 4 * wn;
    const int qd = tid & (nqd - 1);                   // octet of this thread's delta items (512 and nh are multiples of nqd)
    unsigned i_off[SI];                               // bytes from the tile's first element (kNone: no such item)
    unsigned i_yx[SI];                                // row << 16 | column in the halo / the tile; top bit: only the first four channels exist
    unsigned i_dst[SI];                               // bytes in a buffer
    const bool whole = (a.Ci & 7) == 0 && (a.Co & 7) == 0;   // no item has only four channels (uniform)
#pragma unroll
    for (int u = 0; u < SI; ++u) {
        const int first = kWpThreads * u + 64 * wave;  // uniform
        unsigned y, x;
        int left;                                      // channels from the item's first on
        if (first < g.nh) {
            const unsigned it = first + lane;
            const unsigned pos = parts_div(it, a.mg_nqh, nqh), q = it - pos * nqh;
            y = parts_div(pos, a.mg_hwp, g.hwp); x = pos - y * g.hwp;
            left = a.Ci - (16 * p0 + 8 * (int)q);
            const bool ok = y < (unsigned)g.hh && left > 0;
            i_off[u] = ok ? ES * ((y * a.d * a.Wi + x * a.d2) * a.Ci + 16 * p0 + 8 * q) : kNone;
            // (what lies past the halo's last position goes to the padding of the last delta plane)
            i_dst[u] = y < (unsigned)g.hh ? g.halo_b + (q >> 1) * g.hplane + pos * kWpPos + (q & 1) * 16 : g.halo_b - kWpPos;
        } else {
            const unsigned m = (unsigned)(first - g.nh + lane) / (unsigned)nqd;
            y = parts_div(m, a.mg_txp, txp); x = m - y * txp;
            const int oc = 32 * wn * blockIdx.z + 8 * qd;
            left = a.Co - oc;
            const bool ok = y < (unsigned)a.R && left > 0;
            i_off[u] = ok ? ES * ((y * a.d * a.Wo + x * a.d2) * a.Co + oc) : kNone;
            i_dst[u] = (qd >> 1) * g.dplane + m * kWpPos + (qd & 1) * 16;
        }
        i_yx[u] = (left <= 4 ? 0x80000000u : 0u) | (y << 16) | x;
    }
    u32x4 pre[SI][kF32 ? 2 : 1];
    // signs of this slab's deltas (see Accuracy above)
    const float turn = blockIdx.x & 1 ? -1.f : 1.f;
    // what numbers are split after being multiplied by, and what takes their products' sums back
    const int in_raise = P == 2 ? kActRaise : 0, dy_raise = P == 2 ? raise_of(dy_peak, a.dy_margin) : 0;
    const float in_up = P == 2 ? power_of_two(in_raise) : kPartsUp, dy_up = turn * (P == 2 ? power_of_two(dy_raise) : kPartsUp);
    const Lower down = P == 2 ? lower_by(in_raise + dy_raise) : Lower{P == 3 ? kPartsDown : 1.f, 1.f};
    float bsum[8];                                    // this thread's share of the bias gradient: channels 8 qd .. of its delta items
#pragma unroll
    for (int j = 0; j < 8; ++j) bsum[j] = 0.f;
    struct Tile { int b, ry, rx, ty0, tx0, rows, cols; };
    auto decode = [&](int tile) {
        Tile t;
        unsigned bid = tile;
        unsigned qq = parts_div(bid, a.mg_ntx, a.ntx);
        t.tx0 = (int)(bid - qq * a.ntx) * txp; bid = qq;
        qq = parts_div(bid, a.mg_nty, a.nty);
        t.ty0 = (int)(bid - qq * a.nty) * a.R; bid = qq;
        qq = parts_div(bid, a.mg_d2, a.d2);
        t.rx = bid - qq * a.d2; bid = qq;
        qq = parts_div(bid, a.mg_d, a.d);
        t.ry = bid - qq * a.d;
        t.b = qq;
        const int fh = t.ry < a.Ho ? (int)parts_div(a.Ho - t.ry + a.d - 1, a.mg_d, a.d) : 0;
        const int fw = t.rx < a.Wo ? (int)parts_div(a.Wo - t.rx + a.d2 - 1, a.mg_d2, a.d2) : 0;
        t.rows = fh - t.ty0; t.cols = fw - t.tx0;     // of the tile inside its residue class (may be <= 0, or more than the tile's)
        return t;
    };
    // loads of tile `tile` (all issued on every path; what lies outside comes as zeros)
    auto issue = [&](int tile, bool any) {
        const Tile t = decode(tile);
        const int y0 = t.ty0 * a.d + t.ry, x0 = t.tx0 * a.d2 + t.rx;
        const __amdgpu_buffer_rsrc_t in_r = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<T*>(in_t + (((long)t.b * a.Hi + y0) * a.Wi + x0) * a.Ci), 0, 0x7fffffff, 0x00020000);
        const __amdgpu_buffer_rsrc_t dy_r = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<T*>(dy_t + (((long)t.b * a.Ho + y0) * a.Wo + x0) * a.Co), 0, 0x7fffffff, 0x00020000);
        const bool inside = any && t.rows >= a.R && t.cols >= txp && y0 + (g.hh - 1) * a.d < a.Hi && x0 + (g.hwp - 1) * a.d2 < a.Wi;
#pragma unroll
        for (int u = 0; u < SI; ++u) {
            const bool halo = kWpThreads * u + 64 * wave < g.nh;   // uniform
            const __amdgpu_buffer_rsrc_t r = halo ? in_r : dy_r;
            unsigned off = i_off[u];
            if (!inside) {
                const int y = (int)(i_yx[u] >> 16) & 0x7fff, x = (int)(i_yx[u] & 0xffffu);
                const bool ok = any && (halo ? y0 + y * a.d < a.Hi && x0 + x * a.d2 < a.Wi : y < t.rows && x < t.cols);
                off = ok ? off : kNone;
            }
            const unsigned off4 = whole || !(i_yx[u] >> 31) ? off : kNone;
            if constexpr (kF32) {
                pre[u][0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
                pre[u][1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off4, 16, 0));
            } else if (whole)
                pre[u][0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
            else {                                     // (two halves: the second may be another position's)
                const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
                const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off4, 8, 0));
                pre[u][0] = (u32x4){lo[0], lo[1], hi[0], hi[1]};
            }
        }
    };
    auto to_lds = [&](char* buf) {
#pragma unroll
        for (int u = 0; u < SI; ++u) {
            const int first = kWpThreads * u + 64 * wave;   // uniform
            if (first >= g.nh + g.nd) break;
            float x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if constexpr (kF32) x[j] = __builtin_bit_cast(v4f, pre[u][j >> 2])[j & 3];
                else x[j] = (float)__builtin_bit_cast(bf16x8, pre[u][0])[j];
            }
            if (first >= g.nh)
#pragma unroll
                for (int j = 0; j < 8; ++j) bsum[j] += x[j];
            u32x4 p[P];
            const float up = first >= g.nh ? dy_up : in_up;
            if constexpr (P == 2) {
                if (first >= g.nh) split_halves<true>(x, p, {up, up, up, up, up, up, up, up});
                else split_halves<false>(x, p, {up, up, up, up, up, up, up, up});
            } else if constexpr (P == 3) split_parts(x, p, up);
            else p[0] = pre[u][0] ^ (first >= g.nh && blockIdx.x & 1 ? 0x80008000u : 0u);   // (the deltas' turned signs)
            char* dst = buf + i_dst[u];
#pragma unroll
            for (int i = 0; i < P; ++i) *reinterpret_cast<u32x4*>(dst + 32 * i) = p[i];
        }
    };

    // ---- operand addresses: this lane's position and channels inside a plane, and its unit of every row tile
    const unsigned lds_base = (unsigned)reinterpret_cast<size_t>(lds);
    const int grp = lane >> 4, r16 = lane & 15;
    const unsigned lane_b = lds_base + (unsigned)((8 * (grp >> 1) + (r16 >> 2)) * kWpPos + (r16 & 3) * 8);
    const int kk = a.k * a.k2, units = a.ppg * a.tpg;
    unsigned av[PM];
#pragma unroll
    for (int p = 0; p < PM; ++p) {
        const unsigned lu = 2 * (midx * PM + p) + (grp & 1);
        const unsigned pl = parts_div(lu, a.mg_tpg, a.tpg), tap = tap0 + lu - pl * a.tpg;
        const unsigned ta = parts_div(tap, a.mg_k2, a.k2), tb = tap - ta * a.k2;
        const bool ok = lu < (unsigned)units && tap < (unsigned)kk;   // (else: any address inside, never stored)
        av[p] = lane_b + g.halo_b + (ok ? pl * g.hplane + (ta * g.hwp + tb) * kWpPos : 0u);
    }
    const unsigned bv = lane_b + (unsigned)(2 * nidx + (grp & 1)) * (unsigned)g.dplane;

    v16f acc[PM];
#pragma unroll
    for (int p = 0; p < PM; ++p)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[p][r] = 0.f;

    struct Op { tr_bf16x8 part[P]; };
    auto fetch = [&](unsigned addr) {
        typedef tr_bf16x4 __attribute__((address_space(3))) * lds_ptr;
        Op o;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const tr_bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)(uintptr_t)(addr + 32 * i));
            const tr_bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)(uintptr_t)(addr + 32 * i + 4 * kWpPos));
            o.part[i] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
        return o;
    };
    auto mul = [&](const Op& A, const Op& Bo, v16f& c) {
        if constexpr (P == 2) {
            const f16x8 x0 = __builtin_bit_cast(f16x8, A.part[0]), x1 = __builtin_bit_cast(f16x8, A.part[1]);
            const f16x8 y0 = __builtin_bit_cast(f16x8, Bo.part[0]), y1 = __builtin_bit_cast(f16x8, Bo.part[1]);
            c = __builtin_amdgcn_mfma_f32_32x32x16_f16(x1, y0, c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x16_f16(x0 * (_Float16)kLowDown, y1, c, 0, 0, 0);   // (y1: kLowUp times as large)
            c = __builtin_amdgcn_mfma_f32_32x32x16_f16(x0, y0, c, 0, 0, 0);
            return;
        }
#define MPCNN_MUL(i, j) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.part[i], Bo.part[j], c, 0, 0, 0)
        if constexpr (P == 3) { MPCNN_MUL(2, 0); MPCNN_MUL(0, 2); MPCNN_MUL(1, 1); MPCNN_MUL(1, 0); MPCNN_MUL(0, 1); }
        MPCNN_MUL(0, 0);
#undef MPCNN_MUL
    };
    // one tile: the chunks (row, 16 columns) that hold positions, dealt to the wk waves
    auto multiply = [&](int cur, int rows, int cols) {
        rows = rows < a.R ? rows : a.R;
        int nc = (cols + 15) >> 4;
        nc = nc < a.nch ? nc : a.nch;
        if (rows <= 0 || nc <= 0) return;
        const int total = rows * nc;
        int row = 0, cc = kidx;
        while (cc >= nc) { cc -= nc; ++row; }
        const int n = (total - kidx + a.wk - 1) / a.wk;   // this wave's chunks
        if (n <= 0) return;
        unsigned ao = 0, bo = 0;
        auto place = [&]() {
            ao = (unsigned)(cur * g.buf_b + (row * g.hwp + 16 * cc) * kWpPos);
            bo = (unsigned)(cur * g.buf_b + (row * txp + 16 * cc) * kWpPos);
        };
        place();
        Op A[2], Bq[2];
        Bq[0] = fetch(bv + bo);
        A[0] = fetch(av[0] + ao);
        int left = n;
        // two chunks per round: where PM is odd the operand slots change places from one to the next
        for (;;) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                --left;
#pragma unroll
                for (int p = 0; p < PM; ++p) {
                    const int s = (half * PM + p) & 1;
                    if (p + 1 < PM) A[s ^ 1] = fetch(av[p + 1] + ao);
                    else {
                        if (left > 0) {
                            cc += a.wk;
                            while (cc >= nc) { cc -= nc; ++row; }
                            place();
                        }
                        Bq[half ^ 1] = fetch(bv + bo);
                        A[s ^ 1] = fetch(av[0] + ao);
                    }
                    mul(A[s], Bq[half], acc[p]);
                    __builtin_amdgcn_sched_barrier(0);   // (else the reads of many row tiles are moved up, out of registers)
                }
                if (left == 0) return;
            }
        }
    };

    // ---- walk the slab.  Waves 0-3 (one per SIMD) write tile t + 1, loaded a whole tile ahead, before they multiply
    // tile t; waves 4-7 load it before and write it after.
    const int tile_begin = blockIdx.x * a.tiles_per_slab;
    int tile_end = tile_begin + a.tiles_per_slab;
    if (tile_end > a.tiles_total) tile_end = a.tiles_total;
    const bool early = wave < 4;
    if (tile_begin < tile_end) {
        issue(tile_begin, true);
        to_lds(ldsb);
    }
    if (early) issue(tile_begin + 1 < tile_end ? tile_begin + 1 : tile_begin, tile_begin + 1 < tile_end);
    __syncthreads();
    int cur = 0;
    for (int tile = tile_begin; tile < tile_end; ++tile, cur ^= 1) {
        char* other = ldsb + (cur ^ 1) * g.buf_b;
        const bool more = tile + 1 < tile_end;
        if (early) {
            if (more) to_lds(other);
            issue(tile + 2 < tile_end ? tile + 2 : tile, tile + 2 < tile_end);
        } else
            issue(more ? tile + 1 : tile, more);
        if (active) {
            const Tile t = decode(tile);
            multiply(cur, t.rows, t.cols);
        }
        if (!early && more) to_lds(other);
        __syncthreads();
    }

    // ---- partial sums of the waves that shared result tiles (wk > 1) meet in LDS, in a fixed order
    v4f* lds4 = reinterpret_cast<v4f*>(lds);
    for (int s = a.wk >> 1; s >= 1; s >>= 1) {
        if (kidx >= s && kidx < 2 * s) {
            v4f* dst = lds4 + ((((kidx - s) * a.wm + midx) * wn + nidx) * (PM * 4)) * 64 + lane;
#pragma unroll
            for (int p = 0; p < PM; ++p)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4)
                    dst[(p * 4 + r4) * 64] = (v4f){acc[p][4 * r4], acc[p][4 * r4 + 1], acc[p][4 * r4 + 2], acc[p][4 * r4 + 3]};
        }
        __syncthreads();
        if (kidx < s) {
            const v4f* src = lds4 + (((kidx * a.wm + midx) * wn + nidx) * (PM * 4)) * 64 + lane;
#pragma unroll
            for (int p = 0; p < PM; ++p)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const v4f v = src[(p * 4 + r4) * 64];
                    acc[p][4 * r4] += v[0]; acc[p][4 * r4 + 1] += v[1];
                    acc[p][4 * r4 + 2] += v[2]; acc[p][4 * r4 + 3] += v[3];
                }
        }
        __syncthreads();
    }

    // ---- this slab's partial sums, result tiles as the accumulator registers hold them
    const int groups = gridDim.y;
    const long plen = (long)groups * a.RT * a.Nt * 1024 + a.Nt * 32;
    float* out = a.partial + (long)blockIdx.x * plen;
    if (active && kidx == 0) {
        float z = 0.f;                                // NaN as soon as one of the sums is not finite
#pragma unroll
        for (int p = 0; p < PM; ++p)
#pragma unroll
            for (int r = 0; r < 16; ++r) z = fmaf(acc[p][r], 0.f, z);
        const bool odd = P == 3 && __any(z != z);      // (two parts: every number is finite, and no sum overflows)
#pragma unroll
        for (int p = 0; p < PM; ++p)
            if (midx * PM + p < a.RT) {
                v4f* dst = reinterpret_cast<v4f*>(out + (((long)blockIdx.y * a.RT + midx * PM + p) * a.Nt + nt) * 1024) + lane;
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4)
                    dst[r4 * 64] = down.second * (turn * down.first * (v4f){acc[p][4 * r4], acc[p][4 * r4 + 1], acc[p][4 * r4 + 2], acc[p][4 * r4 + 3]});
            }
        if constexpr (P == 3) if (odd) {
            // A sum that is not finite came from infinities, NaN or numbers without parts (or overflows): once more, with fp32
            // multiply-adds over the slab's positions, four gradient rows at a time.  Bound by the trips of its loads, about a tenth
            // of the slab's own time for every four rows that need it; where everything is NaN (a net that diverged) over after one value.
            const int oc = 32 * nt + (lane & 31);
            const bool column = oc < a.Co;
            auto delta = [&](const Tile& t, int y, int x) {
                return dy_t + (((long)t.b * a.Ho + (t.ty0 + y) * a.d + t.ry) * a.Wo + (t.tx0 + x) * a.d2 + t.rx) * a.Co + oc;
            };
            // a NaN among the column's deltas: NaN whatever else, and written already (the slab's first position stands for all)
            bool explained = !column;
            for (int tile = tile_begin; tile < tile_end; ++tile) {
                const Tile t = decode(tile);
                if (t.rows <= 0 || t.cols <= 0) continue;
                if (column) { const float v = load1(delta(t, 0, 0)); explained = v != v; }
                break;
            }
            for (int e = 0; e < PM * 4; ++e) {
                const int p = e >> 2, n = e & 3;
                if (midx * PM + p >= a.RT) break;
                const unsigned lu = 2 * (midx * PM + p) + (n >> 1);
                const unsigned pl = parts_div(lu, a.mg_tpg, a.tpg), tap = tap0 + lu - pl * a.tpg;
                const unsigned ta = parts_div(tap, a.mg_k2, a.k2), tb = tap - ta * a.k2;
                const int c = 16 * (p0 + (int)pl) + 8 * (n & 1) + 4 * (lane >> 5);
                if (lu >= (unsigned)units || tap >= (unsigned)kk) continue;
                v4f* const dst = reinterpret_cast<v4f*>(out + (((long)blockIdx.y * a.RT + midx * PM + p) * a.Nt + nt) * 1024) + lane + 64 * n;
                v4f was = *dst, sum = {0.f, 0.f, 0.f, 0.f};
                unsigned bad = 0;
#pragma unroll
                for (int z = 0; z < 4; ++z) bad |= __builtin_isfinite(was[z]) ? 0u : 1u << z;
                if (explained || c >= a.Ci) bad = 0;
                bool more = __any(bad != 0);          // a sum that is wanted and not NaN yet
                if (!more) continue;
                for (int tile = tile_begin; tile < tile_end && more; ++tile) {
                    const Tile t = decode(tile);
                    const int cols = t.cols < txp ? t.cols : txp;
                    for (int y = 0; y < a.R && y < t.rows && more; ++y) {
                        if (bad) {
                            const T* src = in_t + (((long)t.b * a.Hi + (t.ty0 + y + (int)ta) * a.d + t.ry) * a.Wi + (t.tx0 + (int)tb) * a.d2 + t.rx) * a.Ci + c;
                            const T* dy = delta(t, y, 0);
#pragma unroll 4
                            for (int x = 0; x < cols; ++x) {
                                const v4f v = load4(src + (long)x * a.d2 * a.Ci);
                                const float d = load1(dy + (long)x * a.d2 * a.Co);
#pragma unroll
                                for (int z = 0; z < 4; ++z) sum[z] = fmaf(v[z], d, sum[z]);
                            }
                        }
                        bool open = false;
#pragma unroll
                        for (int z = 0; z < 4; ++z) open |= ((bad >> z) & 1u) && sum[z] == sum[z];
                        more = __any(open);
                    }
                }
#pragma unroll
                for (int z = 0; z < 4; ++z) was[z] = (bad >> z) & 1u ? sum[z] : was[z];
                if (bad) *dst = was;
            }
        }
    }
    // ---- bias gradient = column sums of the delta tiles: the threads of one channel octet in thread order
    if (blockIdx.y == 0) {
        __syncthreads();
        float* sums = lds;
#pragma unroll
        for (int j = 0; j < 8; ++j) sums[tid * 8 + j] = bsum[j];
        __syncthreads();
        if (tid < 32 * wn) {
            const int q = tid >> 3, j = tid & 7, bt = blockIdx.z * wn + (tid >> 5);
            float s = 0.f;
            for (int i = q; i < kWpThreads; i += nqd) s += sums[i * 8 + j];
            if (bt < a.Nt) out[(long)groups * a.RT * a.Nt * 1024 + bt * 32 + (tid & 31)] = s;
        }
    }
}

// fp32 storage: in two parts where both tensors suit them
template <int PM, typename T>
__global__ __launch_bounds__(kWpThreads, 1) void wgrad_parts_kernel(WgradPartsArgs a)
{
    if constexpr (sizeof(T) == 4) {
        extern __shared__ __attribute__((aligned(16))) float lds[];
        unsigned peak = kNoPeak;
        if (a.dy_peak) peak = peak_of(a.dy_peak, a.dy_words);
        if (peak < kNoPeak && a.out && !logistic_maps_reach(a, reinterpret_cast<unsigned*>(lds))) peak = kNoPeak;
        if (peak < kNoPeak) wgrad_parts_body<PM, 2, T>(a, peak);
        else wgrad_parts_body<PM, 3, T>(a, peak);
    } else
        wgrad_parts_body<PM, 1, T>(a, 0);
}

}  // namespace mpcnn
