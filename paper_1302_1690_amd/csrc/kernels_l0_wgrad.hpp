// Weight and bias gradient of the image layer (1 or 3 input channels, spacing 1, filter side 3, 5 or 7,
// Method: step 3 of back-propagation, Alg. 2 for the sum over positions) on v_mfma_f32_32x32x2_f32, in
// either storage type.  The general weight-gradient kernels tile the input by channel quads or octets;
// with an image's few channels most of what they stage and multiply is padding (12-58 TFLOP/s).
//
// The gradient is the product [k rows of k*C values] x [positions] x [maps], contracted over positions.
// A window row's k*C values are contiguous in a channels-last image, so gradient row m = u*(k*C) + r (which
// is the parameter row (u*k + v)*C + c itself) reads, for the position pair (2s, 2s + 1) of a tile row, the
// word at  lane base + (u row pitch + r) + (2s + half)*C  of the image tile in LDS: per 32 gradient rows one
// 32-bit LDS read at an immediate offset and one matrix instruction; the maps' operand is one read of the
// delta tile, [position][map] in LDS, shared by all row tiles.  Both tiles are staged as fp32.
// A workgroup walks tiles of 8 rows x 32 columns of positions (wave w: rows 2w, 2w + 1) and keeps its sums
// in accumulators; at the end the four waves' sums meet in LDS in a fixed order and the workgroup writes
// one partial result in parameter order, bias row last (added by reduce_all_kernel, flat segments).
#pragma once
#include "kernels_mfma.hpp"
#include "kernels_wgrad_tr.hpp"

namespace mpcnn {

constexpr int kL0wTy = 8, kL0wTx = 32;

struct L0WgradArgs {
    const void* in;       // [B][Hi][Wi][C] channels-last image (T)
    const void* dY;       // [B][Ho][Wo][Co] delta at the layer's output (T)
    float* partial;       // [workgroups][(k*k*C + 1) * Co]
    int B, Hi, Wi, Ho, Wo, Co;
    int ntx, nty, tiles_total;
};

template <int K, int C, typename T>
__global__ __launch_bounds__(256) void l0_wgrad_mfma_kernel(L0WgradArgs a)
{
    constexpr int R = K * C, ROWS = K * R, MT = (ROWS + 31) / 32;
    constexpr int TY = kL0wTy, TX = kL0wTx, HH = TY + K - 1, HWC = (TX + K - 1) * C;
    constexpr int XT = (HH * HWC + 3) & ~3;                // floats of the image tile
    __shared__ __attribute__((aligned(16))) float smem[XT + TY * TX * 32];
    float* xt = smem;                                       // [HH][HWC]
    float* dt = smem + XT;                                  // [TY*TX][32 maps]
    const T* in_t = static_cast<const T*>(a.in);
    const T* dy_t = static_cast<const T*>(a.dY);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lt = lane & 31, lg = lane >> 5;
    const int oc0 = 32 * blockIdx.y;
    const int nco = a.Co - oc0 < 32 ? a.Co - oc0 : 32;      // maps of this slice

    // gradient row of this lane in row tile mt: offset of its value for position 0 of tile row 0
    int roff[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = 32 * mt + lt;
        roff[mt] = m < ROWS ? (m / R) * HWC + (m % R) : 0;  // rows past the last: any in-bounds word, never stored
    }
    v16f acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mt][r] = 0.f;
    float bsum = 0.f;

    // A tile's values wait in registers while the tile before it is multiplied: the loads are issued
    // before the matrix instructions of the current tile and written to LDS after them.
    constexpr int XN = (HH * HWC + 255) / 256;              // image values per thread
    float xr[XN];
    v4f dr[8];                                              // 8 quads of deltas, or 32 single ones
    const bool quads = (a.Co & 3) == 0;
    auto fetch = [&](int t) {
        int bid = t;
        const int txi = bid % a.ntx; bid /= a.ntx;
        const int tyi = bid % a.nty;
        const int b = bid / a.nty;
        const int y0 = tyi * TY, x0 = txi * TX;
        // outside the image: zeros; outside the map, and maps past the last: zeros (a zero delta
        // contributes nothing whatever the image value)
        const T* img = in_t + (long)b * a.Hi * a.Wi * C;
#pragma unroll
        for (int i = 0; i < XN; ++i) {
            const int e = tid + 256 * i;
            const int hy = e / HWC, hx = e - hy * HWC;
            const int iy = y0 + hy, ie = x0 * C + hx;
            const bool ok = e < HH * HWC && iy < a.Hi && ie < a.Wi * C;
            xr[i] = load1(img + (ok ? (long)iy * a.Wi * C + ie : 0));
            if (!ok) xr[i] = 0.f;
        }
        const T* dyb = dy_t + (long)b * a.Ho * a.Wo * a.Co;
        if (quads) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int e = tid + 256 * i, pos = e >> 3, q = e & 7;
                const int y = y0 + pos / TX, x = x0 + pos % TX;
                const bool ok = y < a.Ho && x < a.Wo && 4 * q < nco;
                dr[i] = load4(dyb + (ok ? ((long)y * a.Wo + x) * a.Co + oc0 + 4 * q : 0));
                if (!ok) dr[i] = (v4f){0.f, 0.f, 0.f, 0.f};
            }
        } else {
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                const int e = tid + 256 * i, pos = e >> 5, o = e & 31;
                const int y = y0 + pos / TX, x = x0 + pos % TX;
                const bool ok = y < a.Ho && x < a.Wo && o < nco;
                const float v = load1(dyb + (ok ? ((long)y * a.Wo + x) * a.Co + oc0 + o : 0));
                dr[i >> 2][i & 3] = ok ? v : 0.f;
            }
        }
    };
    auto deposit = [&]() {
#pragma unroll
        for (int i = 0; i < XN; ++i)
            if (tid + 256 * i < HH * HWC) xt[tid + 256 * i] = xr[i];
        if (quads) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int e = tid + 256 * i;
                *reinterpret_cast<v4f*>(dt + (e >> 3) * 32 + 4 * (e & 7)) = dr[i];
            }
        } else {
#pragma unroll
            for (int i = 0; i < 32; ++i) dt[tid + 256 * i] = dr[i >> 2][i & 3];
        }
    };
    fetch(blockIdx.x);                                      // (the launch has no more workgroups than tiles)
    for (int t = blockIdx.x; t < a.tiles_total; t += gridDim.x) {
        deposit();
        __syncthreads();
        const int tn = t + gridDim.x;
        fetch(tn < a.tiles_total ? tn : t);                 // (a last tile fetches itself again: same loads on every path)
        // ---- this wave's two tile rows: 16 position pairs each, MT matrix instructions per pair
#pragma unroll
        for (int rw = 0; rw < 2; ++rw) {
            const int ty = 2 * wave + rw;
            const float* xa = xt + ty * HWC + lg * C;
            const float* db = dt + (ty * TX + lg) * 32 + lt;
#pragma unroll
            for (int s = 0; s < TX / 2; ++s) {
                const float bv = db[2 * s * 32];
                bsum += bv;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt] = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[roff[mt] + 2 * s * C], bv, acc[mt], 0, 0, 0);
            }
        }
        __syncthreads();
    }

    // ---- the four waves' sums meet in LDS, wave after wave; then one partial result in parameter order
    float* red = smem;                                      // [MT*32 rows][32 maps], then the bias row
    static_assert(MT * 1024 + 32 <= XT + TY * TX * 32, "the sums fit the tiles' space");
    bsum += __shfl_xor(bsum, 32, 64);                       // both position halves of a map
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = 32 * mt + 8 * (r >> 2) + 4 * lg + (r & 3);   // register 4n + z: row 8n + 4lg + z, column lt
                    float* p = red + row * 32 + lt;
                    *p = w == 0 ? acc[mt][r] : *p + acc[mt][r];
                }
            if (lg == 0) {
                float* p = red + MT * 1024 + lt;
                *p = w == 0 ? bsum : *p + bsum;
            }
        }
        __syncthreads();
    }
    // partial results: workgroup (x, y) owns slot x; slice y fills its own maps of that slot
    float* part = a.partial + (long)blockIdx.x * ((long)ROWS + 1) * a.Co;
    for (int e = tid; e < (ROWS + 1) * 32; e += 256) {
        const int row = e >> 5, o = e & 31;
        if (o < nco) part[(long)row * a.Co + oc0 + o] = row < ROWS ? red[row * 32 + o] : red[MT * 1024 + o];
    }
}

// The same gradient with bf16 storage on v_mfma_f32_32x32x16_bf16, for map counts that are a multiple of 8 (deltas are
// staged as raw 128-bit copies; other counts stay on the kernel above).  16 positions of a tile row per instruction, a lane supplying 8 of
// them for ONE gradient row or ONE map; image, deltas and their products are exact here, sums are fp32 as above.
//   maps: the delta tile is [position][32 maps], read with the transposing LDS read (kernels_wgrad_tr.hpp).
//   gradient rows: 8 successive columns of one channel, shifted by the tap - a read at any multiple of 2 bytes, which the LDS
// serves lane by lane.  So the tile is kept K times, copy v shifted by v columns: LDS row hy*(K*C) + v*C + c holds channel
// c of image row hy at columns v .. v + 31.  Gradient row m = (u*K + v)*C + c of tile row ty is then LDS row ty*(K*C) + m,
// an aligned 128-bit read, and a pitch of 80 bytes spreads 8 successive rows over all banks.
//   bias: gradient row K*K*C (there is always one left in the last row tile) reads ones, whatever the tile row.
// Bound: memory (deltas once: about 100 us of the case below at a device copy's rate).  Measured on 2 x 2048 x 2048, 3 channels, k7,
// 32 maps: 1066 us (74 TFLOP/s on the fp32 instruction) -> 166 us, 472 TFLOP/s, 3.5 TB/s.
constexpr int kL0bPitch = 80;   // bytes of an LDS row: 32 columns, 16 bytes of padding

template <int K, int C>
__global__ __launch_bounds__(256, 2) void l0_wgrad_bm_kernel(L0WgradArgs a)
{
    constexpr int R = K * C, ROWS = K * R, MT = (ROWS + 31) / 32;
    static_assert(ROWS % 32 != 0, "a row tile has room for the bias row");
    constexpr int TY = kL0wTy, TX = kL0wTx, HH = TY + K - 1, HW = TX + K - 1, HWC = HW * C;
    static_assert(TX == 32 && K <= 7 && 2 * (TX + K - 1) <= kL0bPitch, "two instructions per tile row");
    constexpr int XROWS = (TY - 1) * R + 32 * MT;           // LDS rows that are read (past HH*R: by gradient rows that don't exist)
    constexpr int XA = 16;                                  // the first row's left neighbours
    constexpr int ONES = XA + XROWS * kL0bPitch, DB = ONES + kL0bPitch, DBYTES = TY * TX * 64;
    constexpr int RED = (MT * 1024) * 4;
    constexpr int BYTES = DB + DBYTES > RED ? DB + DBYTES : RED;
    static_assert(DB % 16 == 0 && XROWS >= HH * R && BYTES <= 64 * 1024, "LDS layout");
    __shared__ __attribute__((aligned(16))) char smem[BYTES];
    const unsigned short* in_t = static_cast<const unsigned short*>(a.in);      // bf16, moved as they are
    const bf16* dy_t = static_cast<const bf16*>(a.dY);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lt = lane & 31, lg = lane >> 5;
    const int oc0 = 32 * blockIdx.y;
    const int nco = a.Co - oc0 < 32 ? a.Co - oc0 : 32;      // maps of this slice

    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    // every byte that is read is written: rows of gradient rows that don't exist hold zeros, the ones row ones
    for (int e = tid; e < DB / 4; e += 256) reinterpret_cast<unsigned*>(smem)[e] = e >= ONES / 4 ? 0x3f803f80u : 0u;

    v16f acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mt][r] = 0.f;

    // A tile's values wait in registers while the tile before it is multiplied.
    constexpr int XN = (HH * HWC + 255) / 256;              // image values per thread
    constexpr int DN = TY * TX * 4 / 256;                   // items of 8 deltas
    unsigned short xr[XN];
    u4 dr[DN];
    auto fetch = [&](int t) {
        int bid = t;
        const int txi = bid % a.ntx; bid /= a.ntx;
        const int tyi = bid % a.nty;
        const int b = bid / a.nty;
        const int y0 = tyi * TY, x0 = txi * TX;
        // outside the image, outside the map, maps past the last: zeros
        const unsigned short* img = in_t + (long)b * a.Hi * a.Wi * C;
#pragma unroll
        for (int i = 0; i < XN; ++i) {
            const int e = tid + 256 * i;
            const int hy = e / HWC, hx = e - hy * HWC;
            const int iy = y0 + hy, ie = x0 * C + hx;
            const bool ok = e < HH * HWC && iy < a.Hi && ie < a.Wi * C;
            xr[i] = img[ok ? (long)iy * a.Wi * C + ie : 0];
            if (!ok) xr[i] = 0;
        }
        const bf16* dyb = dy_t + (long)b * a.Ho * a.Wo * a.Co;
#pragma unroll
        for (int i = 0; i < DN; ++i) {
            const int e = tid + 256 * i, pos = e >> 2, q = e & 3;
            const int y = y0 + pos / TX, x = x0 + pos % TX;
            const bool ok = y < a.Ho && x < a.Wo && 8 * q < nco;
            dr[i] = *reinterpret_cast<const u4*>(dyb + (ok ? ((long)y * a.Wo + x) * a.Co + oc0 + 8 * q : 0));
            if (!ok) dr[i] = (u4){0u, 0u, 0u, 0u};
        }
    };
    auto deposit = [&]() {
#pragma unroll
        for (int i = 0; i < XN; ++i) {
            const int e = tid + 256 * i;
            const int hy = e / HWC, hx = e - hy * HWC, col = hx / C, c = hx - col * C;
            // (columns a copy has no place for, up to K - 1 on either side, fall into the padding of its row or of the one before)
            char* p = smem + XA + (hy * R + c) * kL0bPitch + 2 * col;
            if (i + 1 < XN || e < HH * HWC) {
#pragma unroll
                for (int v = 0; v < K; ++v) *reinterpret_cast<unsigned short*>(p + v * (C * kL0bPitch - 2)) = xr[i];
            }
        }
#pragma unroll
        for (int i = 0; i < DN; ++i) *reinterpret_cast<u4*>(smem + DB + (tid + 256 * i) * 16) = dr[i];
    };
    // operands: gradient row 32 mt + lt, columns 8 lg ..; maps as kernels_wgrad_tr.hpp lays them out
    const int grp = lane >> 4, r16 = lane & 15;
    const unsigned lds_base = (unsigned)reinterpret_cast<size_t>(smem);
    const unsigned bbase = lds_base + DB + (unsigned)((8 * (grp >> 1) + (r16 >> 2)) * 64 + (16 * (grp & 1) + 4 * (r16 & 3)) * 2);
    const bool bias_lane = 32 * (MT - 1) + lt == ROWS;      // of the last row tile
    fetch(blockIdx.x);                                      // (the launch has no more workgroups than tiles)
    __syncthreads();                                        // the cleared LDS
    for (int t = blockIdx.x; t < a.tiles_total; t += gridDim.x) {
        deposit();
        __syncthreads();
        const int tn = t + gridDim.x;
        fetch(tn < a.tiles_total ? tn : t);                 // (a last tile fetches itself again: same loads on every path)
        // ---- this wave's two tile rows: 2 x 16 positions each
#pragma unroll
        for (int rw = 0; rw < 2; ++rw) {
            const int ty = 2 * wave + rw;
            const int xa = XA + (ty * R + lt) * kL0bPitch + 16 * lg;
            const int xl = bias_lane ? ONES + 16 * lg : xa + (MT - 1) * 32 * kL0bPitch;
            const unsigned ba = bbase + (unsigned)(ty * TX * 64);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const tr_bf16x8 bv = s ? tr_fetch<1024>(ba) : tr_fetch<0>(ba);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const int off = (mt == MT - 1 ? xl : xa + mt * 32 * kL0bPitch) + 32 * s;
                    acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const tr_bf16x8*>(smem + off), bv, acc[mt], 0, 0, 0);
                }
            }
        }
        __syncthreads();
    }

    // ---- the four waves' sums meet in LDS, wave after wave; then one partial result in parameter order
    float* red = reinterpret_cast<float*>(smem);            // [MT*32 rows][32 maps]; row ROWS is the bias
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = 32 * mt + 8 * (r >> 2) + 4 * lg + (r & 3);   // register 4n + z: row 8n + 4lg + z, column lt
                    float* p = red + row * 32 + lt;
                    *p = w == 0 ? acc[mt][r] : *p + acc[mt][r];
                }
        }
        __syncthreads();
    }
    float* part = a.partial + (long)blockIdx.x * ((long)ROWS + 1) * a.Co;
    for (int e = tid; e < (ROWS + 1) * 32; e += 256) {
        const int row = e >> 5, o = e & 31;
        if (o < nco) part[(long)row * a.Co + oc0 + o] = red[row * 32 + o];
    }
}

}  // namespace mpcnn
