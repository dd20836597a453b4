// Whole nets of few maps and parameters in one launch: a workgroup takes a square of output pixels through every layer, forward and back, in LDS.
//
// A net of one to eight maps per layer has nothing for the matrix cores, and layer by layer its pass is a dozen launches of 4 to 10 us each, whatever
// they compute: a chain of dependent loads behind a start-up, an end and the wait for both.  A pixel depends on its patch only, so the maps above a
// square of T x T pixels - (T + what the filters and windows above take)^2 positions each, a few thousand numbers - and their deltas fit in LDS
// together, and squares need nothing of each other: neighbours compute the positions between them twice, which costs less than a launch as long
// as T is not small against the patch (which nets: small_net_fits; T: plan_small).  Gradients are linear in the deltas, so a square's are the sums over its own pixels.
// A thread owns an element of a map (forward, data gradient, routing) or a parameter and some of the rows (weight gradient); a tap's channels come
// in few wide reads, several taps ahead of the sums.  Bound by instructions and by a microsecond per step and layer (its fields, a barrier).
// Sums are in tap order for every element, wherever the square lies and however large it is: equal bits for a position in every call.
//
// Microseconds, layer by layer -> here, for two convolutions of 2 and 3 maps, 8 hidden units, patch 18 (whole calls; training with its gradients read
// back): training 64 x 64 132 -> 62, 256 x 256 161 -> 101, 2 x 447 x 447 437 -> 323; probabilities 64 x 64 29 -> 13, 600 x 600 104 -> 87.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "storage.hpp"

namespace mpcnn {

constexpr int kSmallThreads = 512;
constexpr int kSmallLayers = 12, kSmallSide = 22;   // layers; side of a square, whose pixels are no more than the threads
constexpr int kSmallWgs = 512;          // workgroups, at most (two share a compute unit); they walk the squares
constexpr int kSmallRed = 2 * kSmallThreads;

struct SmallLayer {
    int pool;                // max-pooling, else a convolution (fully connected: its filter covers the map)
    int k, d, ci, co;
    int squash;              // the output goes through the squashing function
    int w;                   // place of W[u][v][c][o], b[o] among the parameters
    int ex;                  // rows and columns of the output map beyond the square's
    int side;                // T + ex: columns between two rows of the map in LDS
    int act, code;           // places of the output (floats) and of the tap codes (bytes) in LDS
    int rows, cols;          // the whole map
    unsigned mg_co, mg_ci, mg_k, mg_side, mg_items;   // ceil(2^32 / x); items: threads of a share of the weight gradient, (k k ci + 1) co
    float* act_out;          // training: the whole map in the workspace, and its codes
    uint8_t* code_out;
};
struct SmallArgs {
    const float* image;      // [B][C][Hs][Ws], mirrored at its borders; the net's image starts (top, left) above and left of it
    const float* params;
    const int32_t* labels;   // or null: no loss, no deltas
    const float* pixw;       // or null
    float* probs;            // or null
    float* partial;          // [workgroups][n_params]: shares of the gradient (training)
    double* loss_partial;    // [workgroups], or null
    int B, C, Hs, Ws, top, left;
    int W, label_h, ctr, probs_rows;   // columns and rows of the label arrays
    int Ho, Wo, T, nty, ntx, tiles;
    unsigned mg_ntx, mg_nty, mg_c, mg_side0;
    int side0, ex0;          // the image's square
    int n_layers, n_params, n_cls, mse, logistic, training;
    unsigned mg_t;           // ceil(2^32 / T)
    int table;               // place of the layers' words in LDS (64 each)
    int img, red, delta[2], grad;      // places in LDS (floats): image, shares of the weight gradients, deltas, the workgroup's gradient
    SmallLayer layer[kSmallLayers];
};

__device__ __forceinline__ unsigned small_div(unsigned n, unsigned magic, unsigned x) { return __umulhi(n, magic) + (n & -(unsigned)(x == 1)); }   // (no branch)

// n terms of a sum: N are fetched before the first of them is added (in order); fetch(on) goes on to the next place only where `on`
template <int N, typename Fetch, typename Add>
__device__ __forceinline__ void small_sum(int n, Fetch fetch, Add add)
{
#pragma unroll 1
    for (int j = 0; j < n; j += N) {
        decltype(fetch(true)) v[N];
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = fetch(j + i + 1 < n);
#pragma unroll
        for (int i = 0; i < N; ++i) if (j + i < n) add(v[i]);
    }
}
// f for a number of channels that the compiler knows: a tap's numbers come in few wide reads, without counting
constexpr int kSmallChannels = 8;
template <typename F>
__device__ __forceinline__ void small_channels(int n, F f)
{
    switch (n) {
#define CASE(i) case i: f(std::integral_constant<int, i>()); break;
    CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
#undef CASE
    }
}
template <int N> struct SmallTerm { float x[N], w[N]; bool ok; };

// The workgroup's LDS is as every wave left it (__syncthreads would wait for what goes to memory, too)
__device__ __forceinline__ void small_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Field of a struct whose words the lanes hold, one each: fields read from LDS one by one, as they are asked for, took a microsecond per layer
template <typename V>
__device__ __forceinline__ V small_field(unsigned words, int at)
{
    if constexpr (sizeof(V) == 8)
        return __builtin_bit_cast(V, (unsigned long long)(unsigned)__builtin_amdgcn_readlane(words, at + 1) << 32 | (unsigned)__builtin_amdgcn_readlane(words, at));
    else
        return __builtin_bit_cast(V, __builtin_amdgcn_readlane(words, at));
}

__global__ __launch_bounds__(kSmallThreads, 4) void small_net_kernel(SmallArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    static_assert(sizeof(SmallLayer) % 4 == 0 && sizeof(SmallLayer) / 4 <= 64 && offsetof(SmallArgs, layer) % 4 == 0, "a word per lane");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const auto* const words = (const __attribute__((address_space(4))) unsigned*)__builtin_amdgcn_kernarg_segment_ptr();   // `a`
    constexpr int kLayerWords = sizeof(SmallLayer) / 4;
    auto layer_words = [&](int l) { return words[offsetof(SmallArgs, layer) / 4 + l * kLayerWords + (lane < kLayerWords ? lane : 0)]; };
#define FIELD(of, f) small_field<decltype(SmallLayer::f)>(of, offsetof(SmallLayer, f) / 4)
    const float* const par = lds;                     // parameters
    // every layer's words, in LDS
    unsigned* const layers_l = reinterpret_cast<unsigned*>(lds + a.table);
    for (int l = wave; l < a.n_layers; l += kSmallThreads / 64) layers_l[l * 64 + lane] = layer_words(l);
    double loss = 0.0;
    for (int t = blockIdx.x, first = 1; t < a.tiles; t += gridDim.x, first = 0) {
        const int T = a.T;
        const unsigned q = small_div(t, a.mg_ntx, a.ntx);
        const int x0 = (t - (int)q * a.ntx) * T, b = (int)small_div(q, a.mg_nty, a.nty), y0 = ((int)q - b * a.nty) * T;
        const int th = a.Ho - y0 < T ? a.Ho - y0 : T, tw = a.Wo - x0 < T ? a.Wo - x0 : T;   // pixels of this square
        const bool end_y = y0 + th == a.Ho, end_x = x0 + tw == a.Wo;
        // What comes from memory starts its trip, on every path (a load behind a branch is waited for there): this thread's pixel's label and
        // weight, an element of the image's square, a parameter
        const int py = (int)small_div(tid, a.mg_t, T), px = tid - py * T;
        const bool own = py < th && px < tw;          // (one a thread: kSmallSide)
        const int img_n = (th + a.ex0) * a.side0 * a.C;
        auto pixel = [&](int e) {
            const unsigned p = small_div(e, a.mg_c, a.C);
            const int c = e - (int)p * a.C, y = (int)small_div(p, a.mg_side0, a.side0);
            int x = (int)p - y * a.side0;
            x = x < tw + a.ex0 ? x : tw + a.ex0 - 1;  // (past the square's last column: never read)
            int ys = y0 + y - a.top, xs = x0 + x - a.left;
            ys = ys < 0 ? -1 - ys : (ys >= a.Hs ? 2 * a.Hs - 1 - ys : ys);
            xs = xs < 0 ? -1 - xs : (xs >= a.Ws ? 2 * a.Ws - 1 - xs : xs);
            return a.image[(((long)b * a.C + c) * a.Hs + ys) * a.Ws + xs];
        };
        const float param0 = a.params[tid < a.n_params ? tid : 0];
        const float pixel0 = pixel(tid < img_n ? tid : 0);
        const long at_label = a.labels && own ? ((long)b * a.label_h + y0 + py + a.ctr) * a.W + x0 + px + a.ctr : 0;
        const int* const some = a.labels ? a.labels : reinterpret_cast<const int*>(a.params);
        const int label0 = some[at_label];
        const float weight0 = (a.pixw ? a.pixw : reinterpret_cast<const float*>(some))[at_label];
        small_barrier();                              // (the last square's image and deltas have been read)
        asm volatile("" :: "v"(label0), "v"(weight0));   // (here, with the pixel: later their registers' next use would wait for what has been stored since)
        if (tid < img_n) lds[a.img + tid] = pixel0;
        for (int e = tid + kSmallThreads; e < img_n; e += kSmallThreads) lds[a.img + e] = pixel(e);
        if (first) {
            if (tid < a.n_params) lds[tid] = param0;
            for (int e = tid + kSmallThreads; e < a.n_params; e += kSmallThreads) lds[e] = a.params[e];
            if (a.training)
                for (int e = tid; e < a.n_params; e += kSmallThreads) lds[a.grad + e] = 0.f;
        }
        small_barrier();

        // ---- forward
        const float* in = lds + a.img;
        int side_in = a.side0;
        for (int l = 0; l < a.n_layers; ++l) {
            const unsigned lw = layers_l[l * 64 + lane];
            const int k = FIELD(lw, k), d = FIELD(lw, d), ci = FIELD(lw, ci), co = FIELD(lw, co), side = FIELD(lw, side), pool = FIELD(lw, pool);
            const int rows = th + FIELD(lw, ex), cols = tw + FIELD(lw, ex), squashed = FIELD(lw, squash), all_rows = FIELD(lw, rows), all_cols = FIELD(lw, cols);
            const unsigned mg_co = FIELD(lw, mg_co), mg_side = FIELD(lw, mg_side);
            float* const out = lds + FIELD(lw, act);
            uint8_t* const code = reinterpret_cast<uint8_t*>(lds) + FIELD(lw, code);
            const float* const weights = par + FIELD(lw, w);
            float* const act_out = FIELD(lw, act_out);
            uint8_t* const code_out = FIELD(lw, code_out);
            const int tap_on = d * ci, row_on = d * (side_in - k) * ci;   // the way to the next tap, and more behind a row of them
            for (int e = tid; e < rows * side * co; e += kSmallThreads) {
                const unsigned p = small_div(e, mg_co, co);
                const int o = e - (int)p * co, y = (int)small_div(p, mg_side, side), x = (int)p - y * side;
                if (x >= cols) continue;
                const float* src = in + (y * side_in + x) * ci;
                float r = 0.f;
                int tap = 0, v = 0;
                if (pool) {
                    src += o;
                    int n = 0;
                    small_sum<4>(k * k,
                        [&](bool on) {
                            const float f = *src;
                            if (on) { src += tap_on; if (++v == k) { v = 0; src += row_on; } }
                            return f;
                        },
                        [&](float f) { if (n == 0 || f > r) { r = f; tap = n; } ++n; });
                    code[e] = (uint8_t)tap;
                } else {
                    const float* w = weights + o;
                    small_channels(ci, [&](auto n) {
                        constexpr int N = decltype(n)::value;
                        small_sum<(N <= 2 ? 4 : 2)>(k * k,
                            [&](bool on) {
                                SmallTerm<N> f;
#pragma unroll
                                for (int c = 0; c < N; ++c) { f.x[c] = src[c]; f.w[c] = w[c * co]; }
                                if (on) { w += N * co; src += tap_on; if (++v == k) { v = 0; src += row_on; } }
                                return f;
                            },
                            [&](const SmallTerm<N>& f) {
#pragma unroll
                                for (int c = 0; c < N; ++c) r = fmaf(f.x[c], f.w[c], r);
                            });
                    });
                    r += weights[k * k * ci * co + o];
                    if (squashed) r = squash(r, a.logistic);
                }
                out[e] = r;
                if (a.training && (y < th || end_y) && (x < tw || end_x)) {
                    const long g = (((long)b * all_rows + y0 + y) * all_cols + x0 + x) * co + o;
                    act_out[g] = r;
                    if (pool) code_out[g] = (uint8_t)tap;
                }
            }
            in = out; side_in = side;
            small_barrier();
        }

        // ---- probabilities, loss, deltas of the outputs (linear ones with a squared error)
        float* g_from = lds + a.delta[0];             // deltas of the present layer's output, of its input
        float* g_to = lds + a.delta[1];
        if (own) {
            const int n_cls = a.n_cls;
            const float* z = in + tid * n_cls;
            float most = z[0], sum = 0.f, zt = 0.f, sq = 0.f;
            for (int o = 1; o < n_cls; ++o) most = fmaxf(most, z[o]);
            for (int o = 0; o < n_cls; ++o) sum += __builtin_amdgcn_exp2f(1.4426950408889634f * (z[o] - most));
            const float inv = __builtin_amdgcn_rcpf(sum), wt = a.pixw ? weight0 : 1.f;
            const int label = a.labels && label0 >= 0 && label0 < n_cls ? label0 : -1;
            for (int o = 0; o < n_cls; ++o) {
                const float p = a.mse ? z[o] : __builtin_amdgcn_exp2f(1.4426950408889634f * (z[o] - most)) * inv;
                if (a.probs) a.probs[(((long)b * n_cls + o) * a.probs_rows + y0 + py) * a.Wo + x0 + px] = p;
                const float off = p - (o == label ? 1.f : 0.f);
                if (o == label) zt = z[o] - most;
                sq += off * off;
                if (a.training) g_from[tid * n_cls + o] = label >= 0 ? wt * off : 0.f;
            }
            if (label >= 0) loss += a.mse ? (double)wt * 0.5 * (double)sq : (double)wt * ((double)logf(sum) - (double)zt);
        }
        if (!a.training) continue;
        small_barrier();

        // ---- backward.  A layer's weight and data gradient need nothing of each other: half of the waves each.
        int red = 0, due = 0, due_at = 0, due_items = 0;   // shares of the last weight gradient, not yet added: their number, the parameters' place and number
        for (int l = a.n_layers - 1; l >= -1; --l) {
            const unsigned lw = layers_l[(l > 0 ? l : 0) * 64 + lane], below = layers_l[(l > 0 ? l - 1 : 0) * 64 + lane];
            const int k = FIELD(lw, k), d = FIELD(lw, d), ci = FIELD(lw, ci), co = FIELD(lw, co), side = FIELD(lw, side), pool = FIELD(lw, pool);
            const int rows = th + FIELD(lw, ex), cols = tw + FIELD(lw, ex), w_at = FIELD(lw, w);
            const float* const x_in = lds + (l > 0 ? FIELD(below, act) : a.img);
            const int side_b = l > 0 ? FIELD(below, side) : a.side0;
            const int half = !pool && l > 0 ? kSmallThreads / 2 : 0, lanes = kSmallThreads - half;   // the first threads of the weight gradient; their number
            int shares = 0;
            const int items = (k * k * ci + 1) * co;
            if (l >= 0 && !pool) {
                shares = lanes / items;
                if (tid >= half) {
                    // a parameter's products of every `shares`-th row; the shares meet behind the barrier
                    const unsigned mg_co = FIELD(lw, mg_co), mg_ci = FIELD(lw, mg_ci), mg_k = FIELD(lw, mg_k), mg_items = FIELD(lw, mg_items);
                    const int share = (int)small_div(tid - half, mg_items, items), every = shares > 1 ? shares : 1;
                    for (int e = tid - half - share * items; e < items && share < every; e += lanes) {   // (more than one round: one share)
                        const int kk = (int)small_div(e, mg_co, co), o = e - kk * co;
                        const int tap = (int)small_div(kk, mg_ci, ci), c = kk - tap * ci, u = (int)small_div(tap, mg_k, k), v = tap - u * k;
                        const bool bias = kk == k * k * ci;
                        float sum = 0.f;
                        for (int y = share; y < rows; y += every) {
                            const float* g = g_from + y * side * co + o;
                            const float* src = bias ? g : x_in + ((y + u * d) * side_b + v * d) * ci + c;
                            small_sum<8>(cols, [&](bool on) { const SmallTerm<1> f = {{*src}, {*g}, true}; if (on) { src += ci; g += co; } return f; },
                                         [&](const SmallTerm<1>& f) { sum = bias ? sum + f.w[0] : fmaf(f.x[0], f.w[0], sum); });
                        }
                        if (shares > 1) lds[a.red + red + share * items + e] = sum;
                        else lds[a.grad + w_at + e] += sum;
                    }
                }
            }
            if (l > 0 && (pool || tid < half)) {
                const int slope = FIELD(below, squash), rows_b = th + FIELD(below, ex), cols_b = tw + FIELD(below, ex);
                const unsigned mg_c = FIELD(below, mg_co), mg_b = FIELD(below, mg_side);
                const uint8_t* const code = reinterpret_cast<const uint8_t*>(lds) + FIELD(lw, code);
                const int tap_back = d * co, row_back = d * (side - k) * co;
                for (int e = tid; e < rows_b * side_b * ci; e += pool ? kSmallThreads : half) {
                    const unsigned p = small_div(e, mg_c, ci);
                    const int c = e - (int)p * ci, y = (int)small_div(p, mg_b, side_b), x = (int)p - y * side_b;
                    if (x >= cols_b) continue;
                    float sum = 0.f;
                    unsigned in_y = 0, in_x = 0;      // taps whose window or output lies in the map
                    for (int u = 0; u < k; ++u) {
                        in_y |= (y - u * d >= 0 && y - u * d < rows ? 1u : 0u) << u;
                        in_x |= (x - u * d >= 0 && x - u * d < cols ? 1u : 0u) << u;
                    }
                    int at = (y * side + x) * co, u = 0, v = 0;
                    if (pool) {
                        at += c;
                        int n = 0;
                        small_sum<4>(k * k,
                            [&](bool on) {
                                const bool ok = in_y >> u & in_x >> v & 1;
                                const int i = ok ? at : 0;
                                const SmallTerm<1> f = {{g_from[i]}, {0.f}, ok && code[i] == n};
                                ++n;
                                if (on) { at -= tap_back; if (++v == k) { v = 0; ++u; at -= row_back; } }
                                return f;
                            },
                            [&](const SmallTerm<1>& f) { sum += f.ok ? f.x[0] : 0.f; });
                    } else {
                        const float* w = par + w_at + c * co;
                        small_channels(co, [&](auto n) {
                            constexpr int N = decltype(n)::value;
                            small_sum<(N <= 2 ? 4 : 2)>(k * k,
                                [&](bool on) {
                                    SmallTerm<N> f;
                                    f.ok = in_y >> u & in_x >> v & 1;
                                    const float* const g = g_from + (f.ok ? at : 0);
#pragma unroll
                                    for (int o = 0; o < N; ++o) { f.x[o] = g[o]; f.w[o] = w[o]; }
                                    if (on) { w += ci * N; at -= tap_back; if (++v == k) { v = 0; ++u; at -= row_back; } }
                                    return f;
                                },
                                [&](const SmallTerm<N>& f) {
                                    float r = sum;
#pragma unroll
                                    for (int o = 0; o < N; ++o) r = fmaf(f.x[o], f.w[o], r);
                                    sum = f.ok ? r : sum;
                                });
                        });
                    }
                    g_to[e] = slope ? sum * squash_slope(x_in[e], a.logistic) : sum;
                }
            }
            // the shares of the layer before (in a half of their own until the one after this)
            for (int e = tid; e < due_items; e += kSmallThreads) {
                float sum = 0.f;
                const float* p = lds + a.red + (red ^ kSmallThreads) + e;
                small_sum<8>(due, [&](bool on) { const float f = *p; if (on) p += due_items; return f; }, [&](float f) { sum += f; });
                lds[a.grad + due_at + e] += sum;
            }
            due_items = 0;
            if (shares > 1) { due = shares; due_at = w_at; due_items = items; red ^= kSmallThreads; }
            float* const was = g_from; g_from = g_to; g_to = was;
            small_barrier();
        }
    }
    if (a.training)
        for (int e = tid; e < a.n_params; e += kSmallThreads) a.partial[(long)blockIdx.x * a.n_params + e] = lds[a.grad + e];
    if (a.loss_partial) {
        __shared__ double sums[kSmallThreads / 64];
#pragma unroll
        for (int w = 1; w < 64; w *= 2) loss += __shfl_xor(loss, w, 64);
        if (lane == 0) sums[wave] = loss;
        small_barrier();
        if (tid == 0) {
            for (int i = 1; i < kSmallThreads / 64; ++i) loss += sums[i];
            a.loss_partial[blockIdx.x] = loss;
        }
    }
#undef FIELD
}

}  // namespace mpcnn
