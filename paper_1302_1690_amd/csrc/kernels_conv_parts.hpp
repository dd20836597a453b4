// Forward / data gradient of one dilated convolution on the 16-bit matrix instructions (v_mfma_f32_32x32x16_f16 and _bf16, 16 times the products
// of the fp32 instruction in the same time), for fp32 storage, whose numbers become sums of two or three 16-bit parts, and for bf16 storage.
//
// THREE bf16 PARTS (fp32 storage).  x = x0 + x1 + x2 exactly (8 + 8 + 8 bits; Henry, Tang, Heinecke: Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations, arXiv 1904.06376), split 2^16 times as large, as below 2^-110 x2 would need bits
// that bf16 does not have. Of the nine products, each exact in fp32, six are taken: x0 y0 in one accumulator, x0 y1 + x1 y0 + (x1 y1 + x0
// y2 + x2 y0) in another.  The three left out are below 2^-24 of |x y| together, 0.36 * 2^-26 in the root mean square.  Two accumulators
// because the instruction rounds its sum twice and before that cuts addends off some ten bits below the largest's last, towards minus
// infinity: with one, 1600 products came out 8e-8 too low on average whatever their sign, which a gradient adds up over all positions while
// its own terms cancel; the second's offset is 2^-8 of that. Infinities, NaN and numbers above 2^-16 of the largest bf16 have no parts and
// leave sums that are not finite, as do sums above 2^96; the epilogue finds those and computes them again with fp32 multiply-adds.
//
// TWO fp16 PARTS (fp32 storage, sums of kHalfLeast products and more).  11 + 11 bits and a sign; three products, x0 y0 in one accumulator and
// x0 y1 + x1 y0 in another: half the instructions.  One number in four loses its last bit and x1 y1 is left out, 7.5e-8 of a sum of random signs
// whatever its length; in exchange there are fewer roundings, as the leading accumulator joins a total after every run of steps (half_run) and starts
// from 0.  Against 64 bits, rms relative, three parts / two without runs / two:
//   K = 64 4.5e-8 / 8.9e-8 / 8.9e-8; 288 8.5e-8 / 1.30e-7 / 1.09e-7; 400 1.01e-7 / 1.47e-7 / 1.12e-7; 576 1.23e-7 / 1.69e-7 / 1.15e-7;
//   800 1.47e-7 / 1.94e-7 / 1.17e-7; 1600 2.18e-7 / 2.64e-7 / 1.25e-7; equal signs 576, 1600: 1.23e-7 / 1.19e-7 / 5.2e-8, 2.22e-7 / 2.21e-7 / 6.4e-8.
// Hence kHalfLeast, where the two are equal.  (The bit that a weight loses is the same at every position: of nets without pools, whose
// gradients show it, these are 1.1 to 1.5 times as far off as with three parts, where few positions carry most of the deltas 2.2 times; 96
// x 110 pixels, five layers, a third.) fp16 reaches from 2^-24 to 2^16, so weights and deltas are raised by powers of two, one per tensor
// (ranges.hpp), and second parts by 2^11 more, their products having an accumulator of their own: numbers below 2^-28 of a tensor's largest
// lose bits below 2^-51 of that.  Activations stay as they are: tanh's are multiples of 2^-24, of logistic ones what is below 2^-36 is
// lost.  The launch takes three parts where this could matter or is not known: a uniform choice at its start (conv_parts_kernel;
// weights_wide, weights_large), so a plan holds for either.
//
// ONE PART (bf16 storage).  One product, one accumulator.
//
// TILING.  A workgroup (4 waves) owns 32*WP*MP positions of ONE residue class (see kernels_mfma.hpp) x 32*WO*MO output channels; a wave
// owns MO x MP result tiles of 32 x 32, one or two with two and three parts, two, four or eight with one.  A step contracts 16 channels of
// one tap: MO + MP operands of P parts each feed 6 (three parts), 3 or 1 instructions per tile.  Weights come through the vector cache,
// activations from LDS, 1 KB per operand and wave. What a product costs in such bytes decides the rate of one part: with 2 x 2 tiles the
// vector cache takes 0.6 of an access per cycle and waits for L2 a third to a half of the time; 2 x 4 tiles take half of that (2 x 2048 x
// 2048, forward 1096, 1745, 1763, 3383 -> 954, 1541, 1519, 3103 us) but need maps that give two workgroups of them to every compute unit. A
// halo is brought in CB channels at a time.  Where the filter is small (2 x 2 taps: 8 steps per 32 channels) blocks are 64 or 128 channels,
// as a block costs two barriers and a wait of its weights behind the halo; where it is large they are 16 channels of kr filter rows.
//
// LATENCY.  Workgroups are persistent and walk (tile, channel block) items.  Two and three parts: the next item's halo is loaded into
// registers before the current one is multiplied and split on its way to LDS after it; two workgroups share a compute unit.  One part: the
// halo goes from memory to LDS without a stop in registers, once every wave has left the last one, in 64-byte pieces of a position per four
// lanes (16 bytes of 64 positions: the last layer's forward 3338 instead of 3040 us), which leaves registers for three workgroups of four
// tiles per wave, or two of eight. Weights run through a ring of parts_ring steps that never drains: the pack is in step order - chunks of
// 16 channels, the taps of each, whatever CB is - and its first steps follow its last once more, so that no fetch looks at the end; behind
// a tile's last step the pointer goes back to its first. The LDS offsets of a block's steps come from a table in LDS, as counting
// taps took more scalar instructions than a step has issue slots for (two parts, 128 -> 200, 2 x 2, 1024 x 1024: 1007 -> 940 us).  Places of a halo's items
// are worked out again only where a tile or the one before it reaches past the tensor. The bias waits in LDS (its loads queued behind the halo's: bf16
// forward 8.8 -> 7.9 ms).
//
// MEASURED, deep net (32 -> 64 k5, 64 -> 64 k5, 64 -> 128 k3, 128 -> 200 k2), microseconds:
//   fp32, 1 x 1024 x 1024, fp32 instruction / three parts / two: forward 838, 1602, 1194, 1956 / 485, 869, 707, 1281 / 319, 555, 480, 889 (326, 362, 290, 207
//     TFLOP/s); data gradient 1060, 1790, 1250, 1880 / 485, 886, 691, 1075 / 311, 568, 453, 745 (335, 355, 307, 247).  A loop of two parts' operands alone
//     sustains 342, of three parts' 221; the clock under these launches is 1.9-2.1 GHz: power bounds the first two layers, waits for halo and stores the others.
//   bf16, 2 x 2048 x 2048: forward 902, 1502, 1518, 2999 (938, 1108, 773, 531 TFLOP/s), data gradient 884, 1480, 1248, 2011 (958, 1124, 940, 791).  The last
//     layer's forward, one image, 1814 whole: without stores 1249, without the next halos 1255, without weights 1616, without the multiplications 1390.
//   Slower than the fp32 instruction's kernel: fp32 launches on one or two thousand positions with at most 16 channels (9 against 7).
//
// THE CLASS LAYER AT THE END (HEAD; forward passes that keep nothing).  The hidden layer's outputs are read once, by the class layer: written and read
// again they were a third of this layer's time with bf16 storage.  Here all channels lie in one workgroup (eight waves for more than 128 with fp32
// storage), a lane multiplies its sixteen of a position by the classes' weights, a half of the wave adds to the other, the waves meet in LDS and a
// thread per position ends with softmax and loss: the sums in class_layer_kernel's order, equal bits.  The halo is then staged once, not once per 128
// channels.  Both launches -> one, microseconds: 128 -> 200, 2 x 2, bf16 2048 x 2048 1756 + 375 -> 1366; fp32 1024 x 1024 1065 + 164 -> 1007 (940 with the steps'
// table); 64 -> 100, 3 x 3, fp32 301 x 293 58.8 + 9.4 -> 59.9.  Where this is taken: make_geom.
//
// Summation order is the step order for every output element, whatever the tiling: equal inputs give bit-equal outputs (exact pooling ties
// stay exact) and a position's value does not depend on how the map is cut.  A data gradient in two parts does depend on the tensor's
// largest delta: by powers of two that change no bit of numbers down to 2^-28 of it, and by the choice of three parts for the whole tensor
// where it is infinite.
#pragma once
#include <stddef.h>

#include <type_traits>

#include "kernels_mfma.hpp"
#include "ranges.hpp"

namespace mpcnn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// Geometry shared with the host's plan.
constexpr int kPartsThreads = 256;   // four waves (a wide class layer's: eight)
__host__ __device__ constexpr int parts_round(int CB, int waves = 4) { return 64 * waves / (CB / 8); }      // halo positions one round of the threads stages
__host__ __device__ constexpr int parts_wgs(int parts, int tiles) { return parts == 1 && tiles <= 4 ? 3 : 2; }   // workgroups that share a compute unit
__host__ __device__ constexpr int parts_items(int parts, int tiles)                                         // rounds, at most: what waits in registers; one part: fits in LDS
{
    return parts > 1 ? 6 : parts_wgs(1, tiles) == 3 ? 12 : 18;
}
// The halo in LDS.  Two and three parts: [position][16 channels][part].  One part: groups of 32 channels (16 where a block has no more), a
// position's octets of a group together - 64 (32) bytes, as the memory holds them.  Octet j of position p sits in place j ^ (p / 4) % 4 (j
// ^ (p / 8) % 2): 16 successive positions meet no bank twice.
__host__ __device__ constexpr int parts_group(int CB) { return CB < 32 ? 2 : 4; }                           // octets of a group
__host__ __device__ constexpr int parts_pitch(int parts, int CB)                                            // bytes of a position, in all groups together
{
    return parts == 1 ? CB * 2 : (CB / 16) * parts * 32 + 16;
}
// steps of weights in registers: 512 cycles of a wave's instructions and more, a trip from L2
__host__ __device__ constexpr int parts_ring(int parts, int tiles) { return parts == 3 ? (tiles > 1 ? 2 : 4) : (parts == 2 || tiles > 2 ? 4 : 8); }

// Numbers are split kPartsUp times as large, and sums of products are brought back by kPartsDown: bf16's last bit lies
// at 2^-133, fp32's at 2^-149.
constexpr float kPartsUp = 0x1p16f, kPartsDown = 0x1p-32f;

// LDS offsets of a block's steps, from a position's, in a table (kernel below), and the entries read past its end
__host__ __device__ constexpr int parts_sets(int parts, int tiles) { return parts == 3 ? 1 : parts == 2 || tiles > 2 ? 2 : 4; }   // activations in registers
constexpr int kPartsTabAhead = 2;
__host__ __device__ inline int parts_table(int CB, int rpad, int taps)
{
    return taps * ((CB < rpad ? CB : rpad) / 16) + 4 + kPartsTabAhead;
}
// With the class layer, behind the table, in floats: the threads' losses (fp64), its weights, one class after the other, the waves' sums of a tile
__host__ __device__ inline int parts_head_at(int CB, int rpad, int taps) { return (parts_table(CB, rpad, taps) + 3) / 4 * 4; }
__host__ __device__ inline int parts_head(int n, int WO, int MO, int positions) { return 2 * positions + n * 32 * WO * MO + WO * n * positions; }
// steps of weights that follow the last in a pack, the first ones again: the ring runs ahead without a look at the end
__host__ __device__ constexpr int parts_ahead(int parts) { return parts == 3 ? 4 : 8; }

// Two fp16 parts of fp32 numbers.  Numbers are first made 2^n times as large (ranges.hpp), the same n for a whole tensor.
// up x = x0 + x1 / LOW_UP but for what x1's 11 bits do not hold: at most one last bit of x, 0 for three numbers of four (8 numbers at once, in pairs:
// two multiplications, two conversions and two subtractions each; two multiplications more where LOW_UP is not 1)
template <bool LOW_UP>
__device__ __forceinline__ void split_halves(const float (&x)[8], u32x4 (&p)[2], const float (&up)[8])
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const f16x2 h = __builtin_convertvector((f32x2){up[2 * j] * x[2 * j], up[2 * j + 1] * x[2 * j + 1]}, f16x2);
        f32x2 rest = {fmaf(up[2 * j], x[2 * j], -(float)h[0]), fmaf(up[2 * j + 1], x[2 * j + 1], -(float)h[1])};
        if constexpr (LOW_UP) rest *= kLowUp;
        const f16x2 l = __builtin_convertvector(rest, f16x2);
        p[0][j] = __builtin_bit_cast(unsigned, h);
        p[1][j] = __builtin_bit_cast(unsigned, l);
    }
}
// Steps between two additions of a tile's leading sums to its total (kernel below): whole chunks of at most 16 taps until they are 8 steps
// (8 to 16), of larger filters whole rows while they are 16 taps at most (12 to 16) or, of those with 8 rows or 9 columns and more, a row
// (4 to k2 steps).  A function of the filter alone.  `period`: steps after which the lengths repeat.
constexpr int kHalfLeast = 512;   // fewest products of a sum that two fp16 parts are taken for
__host__ __device__ inline bool half_filter(int k, int k2) { return k * k2 >= 4 && (k < 8 || k2 >= 4); }   // blocks of four steps at least
struct HalfRun { int period, length; };
__host__ __device__ inline HalfRun half_run(int k, int k2)
{
    const int taps = k * k2;
    if (taps <= 16) { const int whole = taps * ((8 + taps - 1) / taps); return {whole, whole}; }
    return {taps, k < 8 && k2 <= 8 ? k2 * (16 / k2) : k2};
}

// up x = x0 + x1 + x2 exactly (8 numbers at once, in pairs: two multiplications, three conversions, four shifts or masks and four
// subtractions each)
__device__ __forceinline__ void split_parts(const float (&x)[8], u32x4 (&p)[3], float up = kPartsUp)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float lo = up * x[2 * j], hi = up * x[2 * j + 1];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const unsigned two = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
            p[i][j] = two;
            lo -= __builtin_bit_cast(float, two << 16);
            hi -= __builtin_bit_cast(float, two & 0xffff0000u);
        }
    }
}

__device__ __forceinline__ unsigned parts_div(unsigned n, unsigned magic, unsigned x)
{
    return x == 1 ? n : __umulhi(n, magic);   // n / x for n * x < 2^32, magic = ceil(2^32 / x)
}

// Weights that two fp16 parts do not suit: not finite, or with half a sum's number and more, counted over the layer, kSmallOctaves below
// the largest (one output or input map of such weights is enough; a few of them beside larger ones do not matter to any sum)
__device__ __forceinline__ bool weights_wide(const ConvArgs& a)
{
    return a.w_peak && (a.w_peak[0] >= kNoPeak || 2 * a.w_peak[1] >= (unsigned)a.small_limit);
}
// Two parts of activations as they are hold multiples of 2^-24, which tanh leaves, whole; of logistic outputs, however small, they lose
// bits below 2^-36 (rms 2^-37): of no account in a sum that is squashed, known to 2^-24, but under weights that make up for it.  10^4
// products and weights of 16 are off by 2^-26.
__device__ __forceinline__ bool weights_large(const ConvArgs& a) { return a.logistic && a.w_peak[0] >= bits_of(16.f); }

template <typename T, int P, bool BACK, int CB, int WO, int WP, int MO, int MP, bool HEAD>
__device__ __forceinline__ void conv_parts_body(const ConvArgs a, unsigned in_peak)
{
    static_assert(WO * WP == 4 || (HEAD && WO * WP == 8), "four waves");
    constexpr int kThreads = 64 * WO * WP;
    constexpr bool kF32 = sizeof(T) == 4;
    static_assert(kF32 ? P == 2 || P == 3 : P == 1, "parts of the storage type");
    constexpr int QN = CB / 8, NSUB = CB / 16, NS = parts_ring(P, MO * MP);
    constexpr int RP = parts_round(CB, WO * WP), SI = parts_items(P, MO * MP), PITCH = parts_pitch(P, CB);
    constexpr int GO = parts_group(CB), POSB = 16 * GO;   // one part: octets of a group, bytes of a position in it
    constexpr unsigned kNone = 0x80000000u;           // byte offset no buffer reaches: the load returns zeros
    const T* in_t = static_cast<const T*>(a.in);
    const T* act_t = static_cast<const T*>(a.act);
    T* out_t = static_cast<T*>(a.out);
    extern __shared__ __attribute__((aligned(16))) float lds[];
    char* ldsb = reinterpret_cast<char*>(lds);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lt = lane & 31, lg = lane >> 5;
    // channel group turned by the workgroup's index: the waves whose tiles lie past the last channel should not
    // sit on the same SIMDs in both workgroups of a compute unit
    const int wo = (wave + (int)(blockIdx.x % WO)) % WO, wp = wave / WO;

    const int hw = a.Tx + a.k2 - 1, hh = a.Ty + a.kr - 1;
    const int npos = hh * hw;                         // <= SI * RP
    const int GB = (npos + RP - 1) / RP * (RP * POSB);   // one part: bytes of a group (whole kilobytes, as `swapped` wants)
    const int oc0 = 32 * ((blockIdx.y * WO + wo) * MO);   // first channel of this wave's tiles
    const bool live = oc0 < a.Co;                     // uniform for the wave

    // ---- two parts: what numbers are raised by, and their products' sums lowered by
    const int in_raise = P == 2 && BACK ? raise_of(in_peak, a.in_margin) : 0;   // (activations as they are)
    const float in_up = P == 2 ? power_of_two(in_raise) : 1.f;
    const Lower down = P == 2 ? lower_by(in_raise + raise_of(*a.w_peak, 0)) : Lower{1.f, 1.f};

    // ---- staging: thread tid brings 8 channels (octet q of the block) of halo positions tid / QN + RP*u
    const int q = tid % QN, pos0 = tid / QN;
    char* const st_dst = ldsb + pos0 * PITCH + (q >> 1) * (P * 32) + (q & 1) * 16;
    unsigned voff[P == 1 ? 1 : SI];                   // byte offsets from the halo's first element (kNone: outside, or no such position)
    u32x4 pre[P == 1 ? 1 : SI][2];

    struct Tile { int b, ry, rx, ty0, tx0; };
    auto decode = [&](int t) {
        Tile g;
        unsigned bid = t;
        unsigned qd = parts_div(bid, a.mg_ntx, a.ntx);
        g.tx0 = (int)(bid - qd * a.ntx) * a.Tx; bid = qd;
        qd = parts_div(bid, a.mg_nty, a.nty);
        g.ty0 = (int)(bid - qd * a.nty) * a.Ty; bid = qd;
        qd = parts_div(bid, a.mg_d2, a.d2);
        g.rx = bid - qd * a.d2; bid = qd;
        qd = parts_div(bid, a.mg_d, a.d);
        g.ry = bid - qd * a.d;
        g.b = qd;
        return g;
    };
    const T* st_base = in_t;                          // the halo's first element (may lie before the tensor: only valid items are read)
    // (an empty asm keeps what depends on the lane alone from being computed once for all tiles and held in registers
    // beside the accumulators: there are none left)
    auto fresh = [](int v) { asm volatile("" : "+v"(v)); return v; };
    bool inner = false;                               // `voff` is that of a halo inside the tensor, the same for all of them
    auto aim = [&](const Tile& g, bool any, int row0) {   // this thread's items of tile g, filter rows row0 ..
        if (!any) {                                   // (uniform)
#pragma unroll
            for (int u = 0; u < SI; ++u) voff[u] = kNone;
            inner = false;
            return;
        }
        const unsigned row_b = (unsigned)(a.d * a.Wi * a.Cr) * (unsigned)sizeof(T), col_b = (unsigned)(a.d2 * a.Cr) * (unsigned)sizeof(T);
        const int iy0 = (g.ty0 + a.origin + row0) * a.d + g.ry, ix0 = (g.tx0 + a.origin2) * a.d2 + g.rx;
        st_base = in_t + (((long)g.b * a.Hi + iy0) * a.Wi + ix0) * a.Cr;
        const bool was = inner;
        inner = iy0 >= 0 && ix0 >= 0 && iy0 + (hh - 1) * a.d < a.Hi && ix0 + (hw - 1) * a.d2 < a.Wi;   // (uniform)
        if (was && inner) return;
        const int first = fresh(pos0);
#pragma unroll
        for (int u = 0; u < SI; ++u) {
            const unsigned pos = first + RP * u;
            const unsigned ha = parts_div(pos, a.mg_hw, hw), hb = pos - ha * hw;
            const int iy = iy0 + (int)ha * a.d, ix = ix0 + (int)hb * a.d2;
            const bool ok = pos < (unsigned)npos && (unsigned)iy < (unsigned)a.Hi && (unsigned)ix < (unsigned)a.Wi;
            voff[u] = ok ? ha * row_b + hb * col_b + 8u * q * (unsigned)sizeof(T) : kNone;
        }
    };
    // every load is issued on every path (outside: kNone), so that the number in flight is known
    auto issue = [&](int cb) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(st_base), 0, 0x7fffffff, 0x00020000);
        const int c = CB * cb + 8 * q;                // first channel of the item
        const int soff = CB * cb * (int)sizeof(T);
#pragma unroll
        for (int u = 0; u < SI; ++u) {
            if constexpr (kF32) {
                pre[u][0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(c < a.Cr ? voff[u] : kNone), soff, 0));
                pre[u][1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(c + 4 < a.Cr ? voff[u] + 16u : kNone), soff, 0));
            }
        }
    };
    auto to_lds = [&]() {                             // (the LDS holds whole rounds)
#pragma unroll
        for (int u = 0; u < SI; ++u) {
            if (RP * u >= npos) break;                // uniform
            char* dst = st_dst + u * (RP * PITCH);
            if constexpr (kF32) {
                float x[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) x[j] = __builtin_bit_cast(v4f, pre[u][j >> 2])[j & 3];
                u32x4 p[P];
                if constexpr (P == 2) {
                    const float up = BACK ? in_up : 1.f;
                    split_halves<true>(x, p, {up, up, up, up, up, up, up, up});
                }
                else split_parts(x, p);
#pragma unroll
                for (int i = 0; i < P; ++i) *reinterpret_cast<u32x4*>(dst + 32 * i) = p[i];
            }
        }
    };
    // One part needs no conversion: the halo goes from memory to LDS without a stop in registers, 1 KB per instruction - the octets of a group of
    // 16 (32) positions, which lie together in memory too - the waves in turn.  What lies outside comes as zeros.
    constexpr int LP = 64 / GO;                       // positions of an instruction
    auto swapped = [](int at) { return at ^ (at >> 4 & 16 * (GO - 1)); };   // place of an octet, from position * POSB + 16 * octet
    auto bring = [&](const Tile& g, bool any, int row0, int cb) {
        if (!any) return;                             // (uniform; no such tile)
        typedef __attribute__((address_space(3))) void* lds_ptr;
        const unsigned row_b = (unsigned)(a.d * a.Wi * a.Cr) * (unsigned)sizeof(T), col_b = (unsigned)(a.d2 * a.Cr) * (unsigned)sizeof(T);
        const int iy0 = (g.ty0 + a.origin + row0) * a.d + g.ry, ix0 = (g.tx0 + a.origin2) * a.d2 + g.rx;
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<T*>(in_t + (((long)g.b * a.Hi + iy0) * a.Wi + ix0) * a.Cr), 0, 0x7fffffff, 0x00020000);
        const int mine = lane / GO;
        const unsigned oct = (unsigned)(swapped(mine * POSB + lane % GO * 16) >> 4) % GO;   // (LP positions on, an octet's place is the same)
        for (int at = LP * wave; at < npos; at += WO * WP * LP) {
            const unsigned pos = at + mine;
            const unsigned ha = parts_div(pos, a.mg_hw, hw), hb = pos - ha * hw;
            const int iy = iy0 + (int)ha * a.d, ix = ix0 + (int)hb * a.d2;
            const bool ok = pos < (unsigned)npos && (unsigned)iy < (unsigned)a.Hi && (unsigned)ix < (unsigned)a.Wi;
            const unsigned off = ha * row_b + hb * col_b + 16 * oct;
#pragma unroll
            for (int j = 0; j < QN / GO; ++j) {
                const int c = CB * cb + 8 * GO * j;   // the group's first channel
                if (c >= a.CrPad) break;              // (no step reads it)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)(ldsb + j * GB + at * POSB), 16,
                                                         (int)(ok && c + 8 * (int)oct < a.Cr ? off : kNone), c * (int)sizeof(T), 0, 0);
            }
        }
    };
    // The halo is there; with a channel count that is 4 mod 8 the last octet's second half is another position's: zeros
    // (behind an epilogue of whole pieces: without waiting for its stores, which a wave issues after the halo)
    auto brought = [&](int cb, bool stored) {
        constexpr int kStores = 2 * MO * MP;
        if (BACK && stored) __builtin_amdgcn_s_waitcnt(0x0f70 | (kStores & 15) | kStores >> 4 << 14);   // vmcnt(kStores)
        else __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt(0)
        const int oct = (a.Cr >> 3) - cb * QN;
        if ((a.Cr & 7) && oct >= 0 && oct < QN)
            for (int at = LP * wave; at < npos; at += WO * WP * LP)
                if (lane < LP) *reinterpret_cast<u32x2*>(ldsb + oct / GO * GB + swapped((at + lane) * POSB + oct % GO * 16) + 8) = (u32x2){0, 0};
    };

    // ---- the bias of the workgroup's channels, behind the halo's whole rounds
    float* const bias_l = reinterpret_cast<float*>(ldsb + (npos + RP - 1) / RP * (RP * PITCH));
    if constexpr (!BACK)
        if (tid < 32 * WO * MO) {
            const int c = 32 * (int)blockIdx.y * WO * MO + tid;
            bias_l[tid] = c < a.Co ? a.bias[c] : 0.f;
        }

    // ---- the LDS offsets of a block's steps, behind the bias
    int* const table = reinterpret_cast<int*>(bias_l + 32 * WO * MO);
    {
        const int taps = a.kr * a.k2, all = taps * ((CB < a.CrPad ? CB : a.CrPad) / 16);
        const float per_tap = __builtin_amdgcn_rcpf((float)taps), per_row = __builtin_amdgcn_rcpf((float)a.k2);
        for (int i = tid; i < parts_table(CB, a.CrPad, taps); i += kThreads) {
            // (quotients of numbers below 2^20, half a step from the next whole one: exact)
            const int sub = (int)(((float)i + 0.5f) * per_tap), r = i - sub * taps, ta = (int)(((float)r + 0.5f) * per_row), tb = r - ta * a.k2;
            table[i] = i >= all ? 0 : P != 1 ? (ta * hw + tb) * PITCH + sub * (P * 32) : (ta * hw + tb) * POSB + (2 * sub / GO) * GB + (2 * sub % GO) * 16;
        }
    }

    // ---- the class layer's weights, zeros for channels that do not exist; its outputs' sums, [wave's channels][class][position]
    constexpr int kChannels = 32 * WO * MO, kPositions = 32 * WP * MP;
    static_assert(!HEAD || kPositions <= kThreads, "a thread a position");
    float* const head_w = bias_l + kChannels + (HEAD ? parts_head_at(CB, a.CrPad, a.kr * a.k2) : 0);
    // (the arguments are read where they are used, and a thread's loss stays in LDS: there are no registers left in the loop)
    typedef const __attribute__((address_space(4))) HeadArgs* HeadPtr;
    auto head_args = [&] {
        unsigned at = offsetof(ConvArgs, head);
        asm volatile("" : "+s"(at));
        return (HeadPtr)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() + at);
    };
    double* const head_loss = reinterpret_cast<double*>(head_w);
    float* const head_wl = head_w + 2 * kPositions;
    if constexpr (HEAD) {
        const HeadPtr h = head_args();
        const int n = h->n;
        for (int i = tid; i < n * kChannels; i += kThreads) {
            const int o = i / kChannels, c = i % kChannels;
            head_wl[i] = c < a.Co ? h->Wk[c * n + o] : 0.f;
        }
        if (tid < kPositions) head_loss[tid] = 0.0;
    }

    // ---- per lane: LDS address of the positions it feeds as the B operand, at tap 0
    int lbase[MP];
#pragma unroll
    for (int p = 0; p < MP; ++p) {
        const unsigned m = 32 * (wp * MP + p) + lt;
        unsigned ty = parts_div(m, a.mg_tx, a.Tx), tx = m - ty * a.Tx;
        if (ty >= (unsigned)a.Ty) { ty = 0; tx = 0; }   // padding position: any address inside
        lbase[p] = P == 1 ? (int)(ty * hw + tx) * POSB + lg * 16 : (int)(ty * hw + tx) * PITCH + lg * 16;
    }

    // ---- weights: [16-channel chunk][tap][part][lane group][CoPad][8], the step's place a scalar pointer
    const long wpart = 2 * a.CoPad * 16, wstep = P * wpart, wend = (long)a.k * a.k2 * (a.CrPad / 16) * wstep;   // bytes
    const unsigned wlane = (lg * a.CoPad + oc0 + lt) * 16;
    const char* wq = reinterpret_cast<const char*>(P == 2 ? a.wpack2 : a.wpack);   // the next step to fetch
    const int nblk = (a.CrPad + CB - 1) / CB;

    int head[P == 1 ? parts_sets(P, MO * MP) - 1 + kPartsTabAhead : 1];   // the table's first entries
    v16f acc[MO][MP], low[kF32 ? MO : 1][kF32 ? MP : 1];   // low: the smaller products
    v16f tot[P == 2 ? MO : 1][P == 2 ? MP : 1];       // two parts: the runs of leading products before the present one
    int phase = 0;                                    // the ring's slot of the next step (multiply, phased); two parts:
    const HalfRun run = half_run(a.k, a.k2);
    int run_left = 0, period_left = 0;                // the steps left of a run and of a period
    v4f w[NS][MO * P];                                // the ring
    auto fetch_w = [&](int s, int i) {
        if constexpr (P == 1) {
#pragma unroll
            for (int o = 0; o < MO; ++o) w[s][o] = *reinterpret_cast<const v4f*>(wq + wlane + 512 * o);
        } else {                                      // (through a descriptor: the parts' offsets are scalars, no registers beside the lane's)
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(wq), 0, 0x7fffffff, 0x00020000);
#pragma unroll
            for (int o = 0; o < MO; ++o)
                w[s][o * P + i] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(r, (int)wlane + 512 * o, i * (int)wpart, 0));
        }
    };
    auto next_w = [&]() { wq += wstep; };

    // two parts: a run of leading products joins the total
    auto new_run = [&]() {
        run_left = run.length < period_left ? run.length : period_left;
        period_left -= run.length < period_left ? run.length : period_left;
        if (period_left == 0) period_left = run.period;
    };
    auto add_run = [&]() {
#pragma unroll
        for (int o = 0; o < (P == 2 ? MO : 0); ++o)
#pragma unroll
            for (int p = 0; p < MP; ++p)
#pragma unroll
                for (int r = 0; r < 16; ++r) { tot[o][p][r] += acc[o][p][r]; acc[o][p][r] = 0.f; }
        new_run();
    };

    // one tile's share of one channel block: its 16-channel chunks one after the other, the taps of each
    // Phased (two parts; eight tiles per wave): the ring is entered at the slot where the last block left it, and no slot changes its place.
    constexpr bool kPhased = P == 2 || MO * MP > 4;
    auto multiply = [&](int rows, int nsub) {
        const int taps = rows * a.k2, n = taps * nsub;   // steps of this block
        constexpr int XS = parts_sets(P, MO * MP), TS = kPartsTabAhead;
        static_assert(NS % XS == 0 && NS % TS == 0, "a turn of the ring uses each set as often");
        v4f x[XS][P][MP];
        auto fetch_x = [&](int s, int i, int off) {
#pragma unroll
            for (int p = 0; p < MP; ++p)
                if constexpr (P == 1) x[s][i][p] = *reinterpret_cast<const v4f*>(ldsb + swapped(lbase[p] + off));
                else x[s][i][p] = *reinterpret_cast<const v4f*>(ldsb + lbase[p] + off + 32 * i);
        };
        // The steps' places, from the table.  A step is two to twelve instructions of 32 cycles, and a wave alone on its SIMD issues something every four
        // to five cycles: counting cost some 20 scalar instructions per step, with few tiles more than the matrix pipe leaves time for.
        const int* tv = table;
        int at[TS];
        auto product = [&](int s, int t, int i, int j) {   // weight part i, activation part j
#pragma unroll
            for (int o = 0; o < MO; ++o)
#pragma unroll
                for (int p = 0; p < MP; ++p) {
                    v16f& sum = i + j > 0 ? low[o][p] : acc[o][p];
                    if constexpr (P == 2)
                        sum = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, w[s][o * P + i]),
                                                                     __builtin_bit_cast(f16x8, x[t][j][p]), sum, 0, 0, 0);
                    else
                        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[s][o * P + i]),
                                                                      __builtin_bit_cast(bf16x8, x[t][j][p]), sum, 0, 0, 0);
                }
        };
        auto step = [&](int s) {
            if constexpr (P == 3) {
                const int off = at[0];
                at[0] = tv[s + 2];
                // A step's operands are fetched for the next one as soon as they are free: the activations' third part
                // behind the first product, its second behind the third, its first behind the last (three products
                // before it is needed).
                product(s, 0, 0, 2); fetch_x(0, 2, off);
                product(s, 0, 1, 1); product(s, 0, 0, 1); fetch_x(0, 1, off);
                product(s, 0, 2, 0); fetch_w(s, 2);
                product(s, 0, 1, 0); fetch_w(s, 1);
                product(s, 0, 0, 0); fetch_x(0, 0, off); fetch_w(s, 0);
            } else if constexpr (P == 2) {
                // Activations a step ahead.  What is no matrix instruction stands between pairs of those, which cover it: in one place, before the
                // first, it left the matrix pipe empty for as long (64 -> 100, 3 x 3, a wave alone on its SIMD 400 cycles per step, of which 192 are
                // products, now 340; two waves 425, now 385).  The barriers keep it there: reads sink to where they are used, and are waited for.
                product(s, s % XS, 0, 1);
                __builtin_amdgcn_sched_barrier(0);
                const int off = at[s % TS];
                fetch_x((s + 1) % XS, 1, off); at[s % TS] = tv[s + XS - 1 + TS];
                __builtin_amdgcn_sched_barrier(0);
                product(s, s % XS, 1, 0);
                __builtin_amdgcn_sched_barrier(0);
                fetch_x((s + 1) % XS, 0, off); fetch_w(s, 1);
                __builtin_amdgcn_sched_barrier(0);
                product(s, s % XS, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                fetch_w(s, 0);
                if (--run_left == 0) add_run();
            } else {                                  // activations XS - 1 steps ahead, their places TS more
                fetch_x((s + XS - 1) % XS, 0, at[s % TS]);
                at[s % TS] = tv[s + XS - 1 + TS];
                product(s, s % XS, 0, 0); fetch_w(s, 0);
            }
            next_w();
        };
        if constexpr (kPhased) {
            // the rest of a turn, whole turns, and a part of one
#pragma unroll
            for (int t = 0; t < XS; ++t)
                if (phase % XS == t) {
                    static_assert(XS == 2 && TS == 2, "the other set, the other place");
                    if constexpr (P == 2) { at[t] = tv[1]; at[t ^ 1] = tv[2]; fetch_x(t, 1, 0); fetch_x(t, 0, 0); }
                    else { fetch_x(t, 0, head[0]); at[t] = head[1]; at[t ^ 1] = head[2]; }
                }
            tv -= phase;
            // (A block has four steps at least, and nothing branches around a step: on every path into the loop as many loads follow a slot's.)
            static_assert(NS == 4, "slots");
            if (phase < 3) {
                if (phase < 2) {
                    if (phase < 1) step(0);
                    step(1);
                }
                step(2);
            }
            step(3);
            int more = n - (NS - phase);
            for (; more >= NS; more -= NS) {
                tv += NS;
#pragma unroll
                for (int i = 0; i < NS; ++i) step(i);
            }
            tv += NS;
            if (more > 0) {
                step(0);
                if (more > 1) {
                    step(1);
                    if (more > 2) step(2);
                }
            }
            phase = more;
            return;
        }
        if constexpr (P == 3) {
            at[0] = tv[1];
#pragma unroll
            for (int i = P - 1; i >= 0; --i) fetch_x(0, i, 0);
        } else if constexpr (P == 1) {
#pragma unroll
            for (int i = 0; i < XS - 1; ++i) fetch_x(i, 0, head[i]);
#pragma unroll
            for (int i = 0; i < TS; ++i) at[i] = head[XS - 1 + i];
        }
        // Whole turns of the ring.  The first stands before the loop: behind it the next halo's loads are older than
        // every weight in flight, so the loop's waits count weights only.
        int s = 0;
        if (n >= NS) {
#pragma unroll
            for (int i = 0; i < NS; ++i) step(i);
            for (s = NS; s + NS <= n; s += NS) {
                tv += NS;
#pragma unroll
                for (int i = 0; i < NS; ++i) step(i);
            }
            tv += NS;
        }
        // the rest of a turn; the ring's slots then change places, so that the next block starts at slot 0 again
        const int rest = n - s;
#pragma unroll
        for (int i = 0; i < NS - 1; ++i)
            if (i < rest) step(i);
#pragma unroll
        for (int by = 1; by < NS; by *= 2)
            if (rest & by)
#pragma unroll
                for (int j = 0; j < MO * P; ++j) {
                    v4f t[NS];
#pragma unroll
                    for (int r = 0; r < NS; ++r) t[r] = w[(r + by) % NS][j];
#pragma unroll
                    for (int r = 0; r < NS; ++r) w[r][j] = t[r];
                }
    };

    // ---- result of one element: the sum v, and the bias (forward) or the output whose slope multiplies it (data gradient)
    const bool curved = a.mode == kFwdTanh || a.mode == kDgradTanh;   // uniform
    float peak = 0.f;                                 // data gradient: largest magnitude of what this thread has written
    auto finish = [&](float v, float down, float y) {   // (down: a power of two)
        if constexpr (BACK) return curved ? down * v * squash_slope(y, a.logistic) : down * v;
        else return curved ? squash(fmaf(v, down, y), a.logistic) : fmaf(v, down, y);
    };
    // ---- epilogue of tile g: register 4n + z of tile (o, p) is channel oc0 + 32o + 8n + 4lg + z of position
    // 32*(wp*MP + p) + lt.  The bias waits in LDS; what the data gradient reads (the outputs whose slope
    // multiplies it) is fetched one position tile ahead, so that its trip lies under the tile before.
    auto epilogue = [&](const Tile& g, int fh, int fw) {
        const bool vec = (a.Co & 3) == 0;             // uniform
        const int col = fresh(lt);
        const bool reads = BACK && curved;            // uniform
        long pos_off[2];
        bool pos_ok[2];
        typedef T raw4 __attribute__((ext_vector_type(4)));
        raw4 y[2][MO][4];
        auto place = [&](int p) {
            const unsigned m = 32 * (wp * MP + p) + col;
            const int ty = (int)parts_div(m, a.mg_tx, a.Tx), tx = (int)m - ty * a.Tx;
            const int fy = g.ty0 + ty, fx = g.tx0 + tx;
            pos_ok[p & 1] = ty < a.Ty && fy < fh && fx < fw;
            pos_off[p & 1] = (((long)g.b * a.Ho + (fy * a.d + g.ry)) * a.Wo + (fx * a.d2 + g.rx)) * a.Co;
            if (reads)
#pragma unroll
                for (int o = 0; o < MO; ++o)
#pragma unroll
                    for (int n = 0; n < 4; ++n) {
                        const int oc = oc0 + 32 * o + 8 * n + 4 * lg;
                        raw4& v = y[p & 1][o][n];
                        v = (raw4){0, 0, 0, 0};
                        if (!pos_ok[p & 1] || oc >= a.Co) continue;
                        if (vec) v = *reinterpret_cast<const raw4*>(act_t + pos_off[p & 1] + oc);
                        else for (int z = 0; z < 4; ++z) if (oc + z < a.Co) v[z] = act_t[pos_off[p & 1] + oc + z];
                    }
        };
        place(0);
#pragma unroll
        for (int p = 0; p < MP; ++p) {
            if (p + 1 < MP) place(p + 1);
#pragma unroll
            for (int o = 0; o < MO; ++o)
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    const int oc = oc0 + 32 * o + 8 * n + 4 * lg;
                    if (!pos_ok[p & 1] || oc >= a.Co) continue;
                    v4f yv = __builtin_convertvector(y[p & 1][o][n], v4f), r;
                    if constexpr (!BACK) yv = *reinterpret_cast<const v4f*>(bias_l + (oc - 32 * (int)blockIdx.y * WO * MO));
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        float v = acc[o][p][4 * n + z];
                        if constexpr (P == 2) v *= down.first;
                        r[z] = finish(v, P == 2 ? down.second : P == 3 ? kPartsDown : 1.f, yv[z]);
                    }
                    if constexpr (kF32 && BACK)
#pragma unroll
                        for (int z = 0; z < 4; ++z) peak = larger(peak, r[z]);   // (of a channel that does not exist: 0)
                    T* const dst = out_t + pos_off[p & 1] + oc;
                    if (vec) store4(dst, r);
                    else for (int z = 0; z < 4; ++z) if (oc + z < a.Co) store1(dst + z, r[z]);
                }
        }
    };
    // The same with bf16 storage, where an instruction would write 16 bytes of each of 32 positions, and the caches take such pieces one by
    // one.  Lanes change places with each other first, so that four hold 64 successive bytes of a position and an instruction writes 16
    // positions: part h of a tile is positions 16h .. 16h + 15, a lane's piece 8 channels of position 16h + lane % 16.  (2 x 2048 x 2048,
    // forward: 890, 1477, 1496, 3022 -> 873, 1473, 1413, 2954 us; fp32, 32 bytes of 32 positions: no gain.) The bias waits in LDS; what the
    // data gradient reads (the outputs whose slope multiplies it) is fetched a part ahead, so that its trip lies under the part before.
    auto epilogue_pieces = [&](const Tile& g, int fh, int fw) {
      if constexpr (!kF32) {
        constexpr int W = 8;                          // channels of a piece
        typedef T piece __attribute__((ext_vector_type(W)));
        typedef T quad __attribute__((ext_vector_type(4)));
        const bool vec = (a.Co & 3) == 0, whole = a.Co % W == 0;   // uniform
        const int side = fresh(lane);
        const int lch = 16 * (side >> 4 & 1) + 8 * (side >> 5);   // the lane's first channel
        const bool reads = BACK && curved;            // uniform
        // bf16 data gradients issue their stores on every path, and brought waits for the halo without them (2 x 2048 x 2048, us: 2055,
        // 1263, 1481, 881 -> 2041, 1218, 1449, 870; forwards, whose squashing function then runs for channels that do not exist too: 873,
        // 1473, 1413, 2954 -> 896, 1478, 1479, 3073)
        constexpr bool kCounted = BACK;
        long pos_off[2];
        bool pos_ok[2];
        piece y[2][MO];
        unsigned near[2];                             // bytes from the tile's first position
        auto place = [&](int i) {                     // part i & 1 of position tile i / 2
            const unsigned m = 32 * (wp * MP + (i >> 1)) + 16 * (i & 1) + (side & 15);
            const int ty = (int)parts_div(m, a.mg_tx, a.Tx), tx = (int)m - ty * a.Tx;
            const int fy = g.ty0 + ty, fx = g.tx0 + tx;
            pos_ok[i & 1] = ty < a.Ty && fy < fh && fx < fw;
            pos_off[i & 1] = (((long)g.b * a.Ho + (fy * a.d + g.ry)) * a.Wo + (fx * a.d2 + g.rx)) * a.Co;
            near[i & 1] = (unsigned)(ty * a.d * a.Wo + tx * a.d2) * (unsigned)a.Co * (unsigned)sizeof(T);
            if (reads)
#pragma unroll
                for (int o = 0; o < MO; ++o) {
                    const int oc = oc0 + 32 * o + lch;
                    piece& v = y[i & 1][o];
#pragma unroll
                    for (int z = 0; z < W; ++z) v[z] = 0;
                    if (!pos_ok[i & 1] || oc >= a.Co) continue;
                    const T* const src = act_t + pos_off[i & 1] + oc;
                    if (whole) v = *reinterpret_cast<const piece*>(src);
                    else
#pragma unroll
                        for (int q = 0; q < W; q += 4) {
                            if (oc + q >= a.Co) continue;
                            if (vec) {
                                const quad f = *reinterpret_cast<const quad*>(src + q);
#pragma unroll
                                for (int z = 0; z < 4; ++z) v[q + z] = f[z];
                            } else
                                for (int z = 0; z < 4; ++z) if (oc + q + z < a.Co) v[q + z] = src[q + z];
                        }
                }
        };
        auto swap = [](auto op, v16f& t, int i, int j) {
            const auto r = op(__builtin_bit_cast(unsigned, (float)t[i]), __builtin_bit_cast(unsigned, (float)t[j]));
            t[i] = __builtin_bit_cast(float, (unsigned)r[0]); t[j] = __builtin_bit_cast(float, (unsigned)r[1]);
        };
        auto half = [](unsigned u, unsigned v) { return __builtin_amdgcn_permlane32_swap(u, v, false, false); };   // lanes 32.. of u with 0.. of v
        auto row = [](unsigned u, unsigned v) { return __builtin_amdgcn_permlane16_swap(u, v, false, false); };    // odd rows of u with even rows of v
        const __amdgpu_buffer_rsrc_t out_r = __builtin_amdgcn_make_buffer_rsrc(
            out_t + (((long)g.b * a.Ho + (g.ty0 * a.d + g.ry)) * a.Wo + (g.tx0 * a.d2 + g.rx)) * a.Co, 0, 0x7fffffff, 0x00020000);
        place(0);
#pragma unroll
        for (int i = 0; i < 2 * MP; ++i) {
            if (i + 1 < 2 * MP) place(i + 1);
            const int p = i >> 1, h = i & 1;
            if (h == 0)
#pragma unroll
                for (int o = 0; o < MO; ++o) {
#pragma unroll
                    for (int z = 0; z < 4; ++z) { swap(half, acc[o][p], z, 4 + z); swap(half, acc[o][p], 8 + z, 12 + z); }
#pragma unroll
                    for (int z = 0; z < 8; ++z) swap(row, acc[o][p], z, z + 8);
                }
#pragma unroll
            for (int o = 0; o < MO; ++o) {
                const int oc = oc0 + 32 * o + lch;
                const bool exists = pos_ok[h] && oc < a.Co;
                if (!kCounted && !exists) continue;
                float r[W];
                const int own = fresh(oc - 32 * (int)blockIdx.y * WO * MO);
#pragma unroll
                for (int z = 0; z < W; ++z) {
                    float yv;
                    if constexpr (BACK) yv = (float)y[h][o][z];
                    else yv = bias_l[own + z];
                    r[z] = finish(acc[o][p][8 * h + z], 1.f, yv);
                }
                piece v;
#pragma unroll
                for (int z = 0; z < W; ++z) v[z] = (T)r[z];
                T* const dst = out_t + pos_off[h] + oc;
                if (kCounted && whole) {
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), out_r, (int)(exists ? near[h] + 2u * (unsigned)oc : kNone), 0, 0);
                    __builtin_amdgcn_sched_barrier(0);   // (else the pieces are worked on side by side, out of registers)
                } else if (whole)
                    *reinterpret_cast<piece*>(dst) = v;
                else if (exists)
#pragma unroll
                    for (int q = 0; q < W; q += 4) {
                        if (oc + q >= a.Co) continue;
                        if (vec) store4(dst + q, (v4f){r[q], r[q + 1], r[q + 2], r[q + 3]});
                        else for (int z = 0; z < 4; ++z) if (oc + q + z < a.Co) store1(dst + q + z, r[q + z]);
                    }
            }
        }
      }
    };
    // A sum that is not finite came from infinities, NaN or numbers without parts (or is one that overflows): once more, with
    // fp32 multiply-adds over the taps and channels in step order, four channels of one position tile at a time (more would take
    // registers from the loop above).  Bound by the trips of its loads, about the tile's own time for every four channels that need it;
    // where everything is NaN (a net that diverged) over after one value.
    auto repair = [&](const Tile& g, int fh, int fw, const unsigned (&bad)[MO][MP]) {
        const int ci = BACK ? a.Co : a.Cr, co = BACK ? a.Cr : a.Co;   // the raw weights are [tap][layer input][layer output]
#pragma unroll
        for (int p = 0; p < MP; ++p) {
            const unsigned m = 32 * (wp * MP + p) + lt;
            const int ty = (int)parts_div(m, a.mg_tx, a.Tx), tx = (int)m - ty * a.Tx;
            const int fy = g.ty0 + ty, fx = g.tx0 + tx;
            const bool exists = ty < a.Ty && fy < fh && fx < fw;
            const int iy0 = (fy + a.origin) * a.d + g.ry, ix0 = (fx + a.origin2) * a.d2 + g.rx;
            const long off = (((long)g.b * a.Ho + (fy * a.d + g.ry)) * a.Wo + (fx * a.d2 + g.rx)) * a.Co;
            const T* const img = in_t + (long)g.b * a.Hi * a.Wi * a.Cr;
            // a NaN among the values: NaN whatever else, and written already (the first tap inside the map stands for all)
            bool explained = !exists;
            if (exists) {
                const int y = iy0 < 0 ? iy0 + (-iy0 + a.d - 1) / a.d * a.d : iy0, x = ix0 < 0 ? ix0 + (-ix0 + a.d2 - 1) / a.d2 * a.d2 : ix0;
                if (y < a.Hi && x < a.Wi) {           // (a map smaller than the spacing has positions no tap reaches)
                    const float v = load1(img + ((long)y * a.Wi + x) * a.Cr);
                    explained = v != v;
                }
            }
            for (int on = 0; on < 4 * MO; ++on) {
                unsigned mask = 0;
#pragma unroll
                for (int o = 0; o < MO; ++o) mask = on >> 2 == o ? bad[o][p] >> (4 * (on & 3)) & 15u : mask;
                const int oc = oc0 + 32 * (on >> 2) + 8 * (on & 3) + 4 * lg, left = a.Co - oc;   // the lane's four channels, those that exist
                if (explained || left <= 0) mask = 0;
                if (!__any(mask != 0)) continue;
                v4f sum = {0.f, 0.f, 0.f, 0.f};
                bool more = true;                     // a sum that is wanted and not NaN yet
                for (int tap = 0; tap < a.k * a.k2 && more; ++tap) {
                    const int ta = tap / a.k2, tb = tap - ta * a.k2;
                    const int iy = iy0 + ta * a.d, ix = ix0 + tb * a.d2;
                    const bool here = mask && iy >= 0 && ix >= 0 && iy < a.Hi && ix < a.Wi;
                    if (here) {
                        const T* src = img + ((long)iy * a.Wi + ix) * a.Cr;
                        const float* wr = BACK ? a.wraw + ((long)(a.k * a.k2 - 1 - tap) * ci + oc) * co : a.wraw + (long)tap * ci * co + oc;
#pragma unroll 1
                        for (int c = 0; c < a.Cr; c += 4) {
                            const v4f v = load4(src + c);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
#pragma unroll
                                for (int z = 0; z < 4; ++z)           // (a channel that does not exist: the first one's weight again)
                                    sum[z] = fmaf(v[e], wr[(z < left ? z : 0) * (BACK ? co : 1)], sum[z]);
                                wr += BACK ? 1 : co;
                            }
                        }
                    }
                    bool open = false;
#pragma unroll
                    for (int z = 0; z < 4; ++z) open |= ((mask >> z) & 1u) && sum[z] == sum[z];
                    more = __any(open);
                }
#pragma unroll
                for (int z = 0; z < 4; ++z)
                    if (((mask >> z) & 1u) && z < left) {
                        const float y = BACK ? (curved ? load1(act_t + off + oc + z) : 0.f) : a.bias[oc + z];
                        const float v = finish(sum[z], 1.f, y);
                        peak = larger(peak, v);
                        store1(out_t + off + oc + z, v);
                    }
            }
        }
    };

    // ---- the class layer, on the outputs as they would be stored: sums over each tile's channels in the order of class_layer_kernel, so that
    // the probabilities are the same bits.  `kept`: the outputs of this tile are in memory (sums that were not finite have been repaired there).
    auto head_part = [&](const Tile& g, int fh, int fw, bool kept) {
#pragma unroll
        for (int p = 0; p < MP; ++p) {
            const unsigned m = 32 * (wp * MP + p) + lt;
            const int ty = (int)parts_div(m, a.mg_tx, a.Tx), tx = (int)m - ty * a.Tx;
            const int fy = g.ty0 + ty, fx = g.tx0 + tx;
            const bool exists = ty < a.Ty && fy < fh && fx < fw;
            const T* const mine = out_t + (((long)g.b * a.Ho + (fy * a.d + g.ry)) * a.Wo + (fx * a.d2 + g.rx)) * a.Co;
#pragma unroll
            for (int o = 0; o < MO; ++o)
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    const int oc = oc0 + 32 * o + 8 * n + 4 * lg;
                    const v4f bias = *reinterpret_cast<const v4f*>(bias_l + oc);
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        float v = acc[o][p][4 * n + z];
                        if constexpr (P == 2) v *= down.first;
                        acc[o][p][4 * n + z] = (float)(T)finish(v, P == 2 ? down.second : P == 3 ? kPartsDown : 1.f, bias[z]);
                        if (P == 3 && kept && exists && oc < a.Co) acc[o][p][4 * n + z] = load1(mine + oc + z);
                    }
                }
        }
        if (oc0 + 32 * MO > a.Co)                     // channels that do not exist: zeros (an infinite input times no weight is not a number; uniform)
#pragma unroll
            for (int o = 0; o < MO; ++o)
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    if (oc0 + 32 * o + 8 * n + 4 * lg >= a.Co)
#pragma unroll
                        for (int p = 0; p < MP; ++p)
#pragma unroll
                            for (int z = 0; z < 4; ++z) acc[o][p][4 * n + z] = 0.f;
        const int n_cls = head_args()->n;
        float* const sums = head_wl + n_cls * kChannels;
        for (int c = 0; c < n_cls; ++c) {
            const float* const w_c = head_wl + c * kChannels + oc0 + 4 * lg;
            float sum[MP];
#pragma unroll
            for (int o = 0; o < MO; ++o) {
                float quad[4][MP];
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    const v4f wv = *reinterpret_cast<const v4f*>(w_c + 32 * o + 8 * n);
#pragma unroll
                    for (int p = 0; p < MP; ++p) {
                        quad[n][p] = acc[o][p][4 * n] * wv[0];
#pragma unroll
                        for (int z = 1; z < 4; ++z) quad[n][p] = fmaf(acc[o][p][4 * n + z], wv[z], quad[n][p]);
                    }
                }
                // both lane groups' quads of n (neighbours), then n = 0 + 1, 2 + 3, and these: a half of the wave adds one pair, the other the next
                auto halves = [](float u, float v) {
                    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, u), __builtin_bit_cast(unsigned, v), false, false);
                    return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
                };
#pragma unroll
                for (int p = 0; p < MP; ++p) {
                    const float pairs = halves(halves(quad[0][p], quad[1][p]), halves(quad[2][p], quad[3][p]));
                    const float tile = halves(pairs, pairs);
                    sum[p] = o ? sum[p] + tile : tile;
                }
            }
            if (lg == 0)
#pragma unroll
                for (int p = 0; p < MP; ++p) sums[(wo * n_cls + c) * kPositions + 32 * (wp * MP + p) + lt] = sum[p];
        }
    };
    // a thread's position: the waves' sums in pairs, fours and eights, softmax, loss
    auto head_end = [&](const Tile& g) {
        if (tid >= kPositions) return;
        const int fh = g.ry < a.Ho ? (int)parts_div(a.Ho - g.ry + a.d - 1, a.mg_d, a.d) : 0;
        const int fw = g.rx < a.Wo ? (int)parts_div(a.Wo - g.rx + a.d2 - 1, a.mg_d2, a.d2) : 0;
        const int ty = (int)parts_div(tid, a.mg_tx, a.Tx), tx = tid - ty * a.Tx;
        const int fy = g.ty0 + ty, fx = g.tx0 + tx;
        if (ty >= a.Ty || fy >= fh || fx >= fw) return;
        const int y = fy * a.d + g.ry, x = fx * a.d2 + g.rx;
        constexpr int kMost = 4;                      // classes
        float z[kMost], pr[kMost];
        const HeadPtr h = head_args();
        const int n = h->n;
        const float* const sums = head_wl + n * kChannels;
#pragma unroll
        for (int c = 0; c < kMost; ++c) {
            if (c >= n) break;
            float s[WO];
#pragma unroll
            for (int i = 0; i < WO; ++i) s[i] = 32 * MO * i < a.Co ? sums[(i * n + c) * kPositions + tid] : 0.f;
#pragma unroll
            for (int w = 1; w < WO; w *= 2)
#pragma unroll
                for (int i = 0; i < WO; i += 2 * w) s[i] += s[i + w];
            z[c] = s[0] + h->Wk[a.Co * n + c];
        }
        float zmax = z[0], sum = 0.f;
#pragma unroll
        for (int c = 1; c < kMost; ++c) if (c < n) zmax = fmaxf(zmax, z[c]);
#pragma unroll
        for (int c = 0; c < kMost; ++c) {
            if (c >= n) break;
            z[c] -= zmax;
            pr[c] = __builtin_amdgcn_exp2f(1.4426950408889634f * z[c]);
            sum += pr[c];
        }
        const float inv = h->mse ? 1.f : __builtin_amdgcn_rcpf(sum);
#pragma unroll
        for (int c = 0; c < kMost; ++c) {
            if (c >= n) break;
            pr[c] = (h->mse ? z[c] + zmax : pr[c]) * inv;
            if (h->probs) h->probs[((long)(g.b * n + c) * h->probs_rows + y) * a.Wo + x] = pr[c];
        }
        if (!h->labels) return;
        const long at = (long)(g.b * h->H + y + h->ctr) * h->W + x + h->ctr;
        const int label = h->labels[at];
        if (label < 0 || label >= n) return;
        const float wt = h->pixw ? h->pixw[at] : 1.f;
        float zt = 0.f, sq = 0.f;
#pragma unroll
        for (int c = 0; c < kMost; ++c) {
            if (c >= n) break;
            const float e = pr[c] - (c == label ? 1.f : 0.f);
            if (c == label) zt = z[c];
            sq += e * e;
        }
        head_loss[tid] += h->mse ? (double)wt * 0.5 * (double)sq : (double)wt * ((double)logf(sum) - (double)zt);
    };

    // ---- walk the tiles
    int t = blockIdx.x;
    if (t >= a.tiles_total) return;                   // (uniform; the host launches no such workgroup)
    Tile cur = decode(t);
    if constexpr (P == 1) bring(cur, true, 0, 0);
    else { aim(cur, true, 0); issue(0); }
#pragma unroll
    for (int s = 0; s < NS; ++s) {                    // the ring's first steps
#pragma unroll
        for (int i = 0; i < P; ++i) fetch_w(s, i);
        next_w();
    }
    if constexpr (P == 1) brought(0, false);
    else to_lds();
    __syncthreads();
    if constexpr (P == 1)
#pragma unroll
        for (int i = 0; i < parts_sets(P, MO * MP) - 1 + kPartsTabAhead; ++i) head[i] = table[i];
    for (; t < a.tiles_total; t += gridDim.x) {
#pragma unroll
        for (int o = 0; o < MO; ++o)
#pragma unroll
            for (int p = 0; p < MP; ++p)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    acc[o][p][r] = 0.f;
                    if constexpr (kF32) low[o][p][r] = 0.f;
                    if constexpr (P == 2) tot[o][p][r] = 0.f;
                }
        if constexpr (P == 2) { period_left = run.period; new_run(); }
        Tile nxt = cur;
        int cb = 0, row0 = 0;                         // channel block, first filter row
        bool last;
        do {
            // the next item's halo starts its trip
            int cn = cb, rn = row0 + a.kr;
            if (rn >= a.k) { rn = 0; ++cn; }
            last = cn == nblk;
            if (last) {
                const int tn = t + gridDim.x;
                nxt = decode(tn < a.tiles_total ? tn : t);
                if constexpr (P != 1) aim(nxt, tn < a.tiles_total, 0);
                cn = 0;
            } else if (P != 1 && a.kr < a.k)
                aim(cur, true, rn);
            if constexpr (P != 1) issue(cn);
            const int chunks = (a.CrPad - cb * CB) / 16, rows = a.k - row0;
            if (live) multiply(rows < a.kr ? rows : a.kr, chunks < NSUB ? chunks : NSUB);
            if constexpr (P == 1) {                   // one part: under the epilogue, and under the other workgroups' instructions
                __syncthreads();                      // every wave has left this block's halo
                bring(last ? nxt : cur, !last || t + (int)gridDim.x < a.tiles_total, rn, cn);
            }
            if (last && live) {
                const int fh = cur.ry < a.Ho ? (int)parts_div(a.Ho - cur.ry + a.d - 1, a.mg_d, a.d) : 0;   // extent of this residue class
                const int fw = cur.rx < a.Wo ? (int)parts_div(a.Wo - cur.rx + a.d2 - 1, a.mg_d2, a.d2) : 0;
                bool odd = false;
                if constexpr (kF32)
#pragma unroll
                    for (int o = 0; o < MO; ++o)
#pragma unroll
                        for (int p = 0; p < MP; ++p) {
                            if constexpr (P == 2) {
                                acc[o][p] += tot[o][p];
#pragma unroll
                                for (int r = 0; r < 16; ++r) acc[o][p][r] = fmaf(low[o][p][r], kLowDown, acc[o][p][r]);   // (as whole vectors: spills)
                            } else
                                acc[o][p] += low[o][p];
                        }
                if constexpr (P == 3) {
                    float z = 0.f;                    // NaN as soon as one of the sums is not finite
#pragma unroll
                    for (int o = 0; o < MO; ++o)
#pragma unroll
                        for (int p = 0; p < MP; ++p)
#pragma unroll
                            for (int r = 0; r < 16; ++r) z = fmaf(acc[o][p][r], 0.f, z);
                    odd = __any(z != z);
                }
                if constexpr (HEAD) {
                    if (P == 3 && odd) epilogue(cur, fh, fw);
                } else if constexpr (kF32) epilogue(cur, fh, fw);
                else epilogue_pieces(cur, fh, fw);
                if constexpr (P == 3) {
                    if (odd) {
                        unsigned bad[MO][MP];
#pragma unroll
                        for (int o = 0; o < MO; ++o)
#pragma unroll
                            for (int p = 0; p < MP; ++p) {
                                bad[o][p] = 0;
#pragma unroll
                                for (int r = 0; r < 16; ++r) bad[o][p] |= __builtin_isfinite(acc[o][p][r]) ? 0u : 1u << r;
                            }
                        repair(cur, fh, fw, bad);
                    }
                }
                if constexpr (HEAD) head_part(cur, fh, fw, odd);
            }
            if constexpr (P == 1) {
                int stored = BACK && last && live && (a.Co & 7) == 0;
                if constexpr (BACK) asm volatile("" : "+s"(stored));   // (else the paths with and without an epilogue are compiled apart, and spill)
                brought(cn, stored != 0);
            } else {
                __syncthreads();                      // every wave has left this block's halo
                if constexpr (HEAD)
                    if (last) head_end(cur);
                if (!last || t + (int)gridDim.x < a.tiles_total) to_lds();
            }
            __syncthreads();
            if constexpr (HEAD && P == 1)             // (the next tile's sums come behind a barrier of its own)
                if (last) head_end(cur);
            cb = cn; row0 = rn;
        } while (!last);
        wq -= live ? wend : 0;                        // (the ring holds the first steps again)
        cur = nxt;
    }
    if constexpr (HEAD)
        if (head_args()->loss_partial) {              // (uniform; the threads' losses are behind the last barrier)
            __syncthreads();
            double sum = tid < kPositions ? head_loss[tid] : 0.0;
            double* const each = reinterpret_cast<double*>(lds);
#pragma unroll
            for (int w = 1; w < 64; w *= 2) sum += __shfl_xor(sum, w, 64);
            if (lane == 0) each[wave] = sum;
            __syncthreads();
            if (tid == 0) {
                for (int i = 1; i < WO * WP; ++i) sum += each[i];
                head_args()->loss_partial[blockIdx.x] = sum;
            }
        }
    if (kF32 && BACK && a.out_peak) {                 // (uniform)
        unsigned* const four = reinterpret_cast<unsigned*>(lds);   // (the last barrier above is behind every read of the LDS)
        unsigned most = wave_largest(bits_of(peak));
        if (lane == 0) four[wave] = most;
        __syncthreads();
        if (tid == 0) {
            for (int i = 1; i < 4; ++i) most = four[i] > most ? four[i] : most;
            // (weights that are wide may leave a map of deltas far below the others')
            a.out_peak[blockIdx.y * gridDim.x + blockIdx.x] = weights_wide(a) ? kNoPeak : most;
        }
    }
}

// fp32 storage: in two parts where everything is known to suit them
template <typename T, bool BACK, int CB, int WO, int WP, int MO, int MP, bool HEAD = false>
__global__ __launch_bounds__(64 * WO * WP, parts_wgs(sizeof(T) == 4 ? 3 : 1, MO * MP)) void conv_parts_kernel(ConvArgs a)
{
    if constexpr (sizeof(T) == 4) {
        unsigned peak = kNoPeak;
        if (a.wpack2) peak = weights_wide(a) || (!BACK && weights_large(a)) ? kNoPeak : BACK ? peak_of(a.in_peak, a.in_words) : 0;
        if (peak < kNoPeak) conv_parts_body<T, 2, BACK, CB, WO, WP, MO, MP, HEAD>(a, peak);
        else conv_parts_body<T, 3, BACK, CB, WO, WP, MO, MP, HEAD>(a, peak);
    } else
        conv_parts_body<T, 1, BACK, CB, WO, WP, MO, MP, HEAD>(a, 0);
}

}  // namespace mpcnn
