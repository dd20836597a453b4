// What the matrix-core kernels of the dilated convolutions share.
//
// Tiling rule.  A layer whose taps are d elements apart never mixes the d*d residue
// classes (y mod d, x mod d) of its dense map - each class is one "fragment" of the
// paper's MPF storage (Method, MPF layer) and, seen alone, an ordinary undilated
// convolution.  So a workgroup takes a Ty x Tx tile of ONE class: its (Ty+k-1) x (Tx+k-1)
// input halo is staged in LDS, each element a contiguous channel vector in the
// channels-last tensor, and is reused by all k*k taps.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "storage.hpp"

namespace mpcnn {

enum ConvMode { kFwdTanh = 0, kFwdLinear = 1, kDgradTanh = 2, kDgradPlain = 3 };

// What a class layer does with the outputs of the layer below it (conv_parts_kernel with HEAD; the fields as in ClassArgs)
struct HeadArgs {
    const float* Wk;     // [K][n] then bias [n]
    float* probs;        // [B][n][probs_rows][Wo] or null
    const int32_t* labels;
    const float* pixw;
    double* loss_partial;   // [workgroups], or null
    int n, mse, H, W, ctr, probs_rows;
};
struct ConvArgs {
    // tensors are fp32 or bf16 (the kernel's template parameter T)
    const void* in;      // [B][Hi][Wi][Cr]   tensor the taps read (activations, or deltas for dgrad)
    const v4f* wpack;    // weights in step order (pack_weights_kernel)
    const float* bias;   // [Co]   (forward modes)
    const void* act;     // [B][Ho][Wo][Co] tanh output at the positions written (kDgradTanh)
    void* out;           // [B][Ho][Wo][Co]
    int B, Hi, Wi, Cr, CrPad;   // CrPad: Cr rounded up to a multiple of 16
    int Ho, Wo, Co, CoPad;
    int k, d;            // filter rows and the spacing of rows
    int kr;              // filter rows of a block: k, or fewer (blocks of 16 channels only)
    int k2, d2;          // filter columns and the spacing of columns (they differ from k, d behind a rectangular pool)
    int origin, origin2; // halo origin (rows, columns) in fragment units relative to the tile: 0 forward, -(k-1), -(k2-1) dgrad
    int Ty, Tx, nty, ntx;
    int mode;
    int logistic;        // squashing function of the Tanh modes: 0 tanh, 1 logistic
    // number of tiles to walk, and ceil(2^32 / x) of the divisors the kernel uses
    // (n / x == umulhi(n, magic) for n * x < 2^32, x > 1)
    int tiles_total;
    unsigned mg_hw, mg_tx, mg_ntx, mg_nty, mg_d, mg_d2;
    // fp32 storage, two fp16 parts per number (conv_parts_kernel): weights in step order, or null: not for this launch; largest magnitude of the
    // weights and number of small ones (pack_weights_kernel), or null; data gradient: the input's in_words words (ranges.hpp; its numbers are at most
    // 2^in_margin times as large), the output's words, or null
    const v4f* wpack2;
    const unsigned *w_peak, *in_peak;
    unsigned* out_peak;
    int in_words, in_margin, small_limit;
    HeadArgs head;
    const float* wraw;   // [k*k2][layer input][layer output], the parameters as they are (conv_parts_kernel: sums that are not finite)
};

}  // namespace mpcnn
