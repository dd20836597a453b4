// libmpcnn: host side of the whole-image MPCNN forward / backward (see include/mpcnn.h).
//
// The paper keeps each layer's data as a set of fragments, k*k new ones per pooling
// layer (Method, Notation and MPF layer).  Here the whole set is ONE dense tensor per
// layer, [B][rows][cols][channels]: element (r,s) of the patch with top-left (i,j) sits at
// (i + r*d, j + s*d), d = product of the pooling factors so far, so fragment (a,b) of the
// paper is the sub-lattice {y = a mod d, x = b mod d}.  Pooling becomes a stride-1 max
// filter with taps d apart, later C / FC kernels read taps d apart, and the first FC is
// a convolution whose kernel covers the q x q map that remains of a patch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "../../include/mpcnn.h"
#include "kernels_direct.hpp"
#include "launchers.hpp"
#include "kernels_conv_parts.hpp"   // its LDS geometry (no instance is built here)
#include "kernels_wgrad_tr.hpp"     // its LDS geometry
#include "kernels_wgrad_bf16.hpp"   // its LDS geometry, which the planner shares (no instance is built here)
#include "kernels_pack.hpp"
#include "kernels_reduce.hpp"
#include "kernels_lbfgs.hpp"
#include "kernels_first_bf16.hpp"
#include "kernels_first_f32.hpp"
#include "kernels_l0_wgrad.hpp"
#include "kernels_fused.hpp"
#include "kernels_small.hpp"

// Device memory of mpcnn_seg_forward_static: a fixed array in the library's device image, so that
// the call needs no allocation.  Every GPU the library runs on holds its own copy, at its own
// address, until the process ends.  In host code the name below is only a handle for
// hipGetSymbolAddress; the kernels are given the address that call returns.
static __device__ __align__(256) unsigned char scratch[MPCNN_STATIC_WORKSPACE_BYTES];

namespace {

thread_local char g_err[512] = "";

mpcnn_status fail(mpcnn_status st, const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return st;
}

#define HIP_TRY(expr)                                                                      \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                              \
            return fail(MPCNN_EHIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), \
                        __FILE__, __LINE__);                                               \
    } while (0)

constexpr int kLossBlocks = 2048;         // most per-workgroup loss shares (= most workgroups of the class-layer kernel)
static_assert(kLossBlocks <= mpcnn::kDeltaWords, "each has a word");
constexpr int kSoftmaxBlocks = 512;       // workgroups of the unfused softmax kernel
constexpr int kDirectWgradChunks = 512;   // split of the position reduction, direct kernel
constexpr size_t kWgradLdsCap = 144 * 1024;
constexpr int kNumCU = 256;

inline size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }
inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Output-channel tiling of the convolution kernel: tiles of 32 channels, OT tiles per workgroup,
// `split` groups of them (blockIdx.y), `pad` = channels covered.
struct ChanTiling { int OT, split, pad; };
ChanTiling tile_channels(int channels, int W, const int* allowed, int n_allowed)
{
    const int max_ot = allowed[n_allowed - 1];
    const int tiles = ceil_div(channels, W);
    const int split = ceil_div(tiles, max_ot);
    const int per = ceil_div(tiles, split);
    int OT = max_ot;
    for (int i = 0; i < n_allowed; ++i) if (allowed[i] >= per) { OT = allowed[i]; break; }
    return {OT, split, OT * split * W};
}
ChanTiling chan_tiling(int channels)   // convolution kernel instances
{
    static const int allowed[] = {1, 2, 4};
    return tile_channels(channels, 32, allowed, 3);
}

struct Layer {
    int kind;     // mpcnn_kind
    int k;        // kernel side (C, FC) or pooling side (MP)
    int cin, cout;
    int dil;      // spacing of this layer's taps in its input map
    int drop = 0; // MP: trailing rows / columns of the patch-level map that no window covers (side mod k)
    // columns, where they differ from the rows (a rectangular pool, and every layer after it):
    int k2 = 0, dil2 = 0, drop2 = 0;
    bool rect = false;   // k2 != k or dil2 != dil: not for the bf16 weight gradients, the image layer's kernels and the paired pools
    bool tanh_out;
    size_t p_off; // offset of this layer's [(k*k*cin + 1) x cout] block in the parameter buffer
    size_t p_len;
    // matrix-core paths (decided once from the channel counts)
    bool fwd_mfma = false, dgrad_mfma = false, wgrad_mfma = false;
    bool class_fused = false;             // last FC handled by class_layer_kernel
    ChanTiling fwd_ct{}, dgrad_ct{};
    int fwd_rpad = 0, dgrad_rpad = 0;     // reduced channels padded to 16
    size_t fwd_pack_off = 0, fwd_pack_len = 0, dgrad_pack_off = 0, dgrad_pack_len = 0;
    // fp32 storage: sums long enough for two fp16 parts per number (mpcnn_net_create), whose packs lie beside the others
    bool fwd_half = false, dgrad_half = false;
    size_t fwd_half_off = 0, fwd_half_len = 0, dgrad_half_off = 0, dgrad_half_len = 0;
};

struct TilePlan {          // conv_parts_kernel: 32 PT positions per workgroup, `wgs` workgroups per channel group walk the tiles
    int PT = 0, Ty = 0, Tx = 0, nty = 0, ntx = 0, wgs = 0, kr = 0;
    mpcnn::PartsInstance in{};
    size_t lds = 0;
    double cost = 0;       // cycles, by the planner's estimate
    bool ok = false;
};
struct WgradPlan {
    bool ok = false;
    bool bm = false;      // bf16 storage: the bf16 matrix instruction, 16 positions per MFMA
    bool tr = false;      // ... with operands from the transposing LDS read (wgrad_tr_kernel)
    int Tx = 0, TxP = 0, nty = 0, ntx = 0, tiles_total = 0, tiles_per_slab = 0, slabs = 0;
    int Mt = 0, Nt = 0, wm = 0, wn = 0, wk = 0, mw = 0, gm = 0, gn = 0;
    size_t lds = 0;
    size_t plen = 0;      // floats per partial result (tiled layout)
    int hl = 0;           // halo items per loading thread and tile (fp32 matrix instruction kernel)
    int PM = 0, R = 0, nch = 0, RT = 0, ppg = 0, tpg = 0, ntg = 0;   // PM > 0: wgrad_parts_kernel (gm x gn groups, tile R rows x 16 nch columns)
    double chain = 0;     // ... positions that a wave adds into one accumulator
    bool two = false;     // ... in two fp16 parts where the deltas suit them
    // direct kernel fallback
    int rows_per_chunk = 0, chunks = 0;
    bool l0m = false;     // the image layer's own kernel (l0_wgrad_mfma_kernel): `chunks` workgroups, flat partial results
};

// Per-call geometry: dense map sizes, launch plans and workspace offsets.
struct Geom {
    int B = 0, H = 0, W = 0;
    bool training = false;
    std::vector<int> rows, cols;      // output map of layer l
    std::vector<size_t> act_off;      // byte offset of layer l's output in the workspace
    std::vector<size_t> code_off;     // MP layers: byte offset of the argmax map
    std::vector<TilePlan> fwd, dgrad;
    std::vector<WgradPlan> wgrad;
    int pad_top = 0, pad_left = 0;    // same-size forward: H, W are the mirrored image's, which starts
    int src_h = 0, src_w = 0;         //   this far above / left of the caller's src_h x src_w image
    bool staged = false;              // the image is copied to channels-last storage first
    int label_h = 0, probs_rows = 0;  // rows of the label / weight arrays and of the probs array (bands: the whole image's)
    bool accumulate = false;          // gradients and loss are added to what the net holds (bands after the first)
    bool fixed_partials = false;      // partial-sum buffers sized by bounds that hold for every map size (bands)
    size_t staged_off = 0;            // that copy (C0 > 1, or bf16 storage)
    size_t delta_off[2] = {0, 0};     // two delta buffers, each as large as the largest map
    std::vector<size_t> partial_off;  // per parametrised layer: its slab / block partial sums
    std::vector<int> partial_n;
    std::vector<size_t> partial_len;  // floats per partial result
    size_t loss_partial_off = 0;
    // Largest magnitudes of the deltas (ranges.hpp).  Layer whose words hold those of the delta at layer l's output, -1: nobody notes them
    // (pools take them from above); number of the words, octaves that routing passes may add, place of the words.  `squashed`: layer l's
    // output is a squashing function's
    std::vector<int> delta_peak, delta_words, delta_margin;
    std::vector<bool> squashed;
    size_t delta_words_off = 0;
    // first convolution followed by a pool: routing through the pool and the convolution's
    // parameter gradient run as one kernel (l0_wgrad_fused_kernel), in l0_blocks workgroups
    bool l0_fused = false;
    int l0_blocks = 0, l0_nty = 0, l0_ntx = 0;
    size_t l0_lds = 0;
    // nets of few maps: the whole pass in one launch (small_net_kernel; what depends on a call's buffers is filled in then)
    bool small_net = false;
    mpcnn::SmallArgs small{};
    bool head = false;        // forward only: the hidden layer below the class layer ends with it (conv_parts_kernel, HEAD)
    int small_wgs = 0;
    size_t small_lds = 0, small_partial_off = 0;
    size_t total = 0;
};

struct ProfSite {
    char name[48];
    int layer, step, launches;
    double ms, flops, bytes;
};
struct ProfPending { int site; hipEvent_t e0, e1; };

// Plans are kept per (sizes, mode, tiling hints): a call with sizes seen before plans nothing.
struct GeomKey {
    int B, H, W, training, same, hint_pt, hint_mp;
    bool operator==(const GeomKey& o) const
    {
        return B == o.B && H == o.H && W == o.W && training == o.training && same == o.same &&
               hint_pt == o.hint_pt && hint_mp == o.hint_mp;
    }
};
constexpr size_t kGeomCacheSize = 8;

}  // namespace

struct mpcnn_net {
    std::vector<Layer> layers;
    int in_ch = 0, patch = 0, n_cls = 0;
    size_t n_params = 0, pack_len = 0;
    int loss_kind = MPCNN_LOSS_MCCE;
    int loss_shares = 0;          // per-workgroup loss shares the forward left for the closing reduce
    double* loss_out = nullptr;   // where that reduce puts their sum
    bool bf16 = false;            // activations and deltas stored in bf16 (arithmetic stays fp32)
    float* d_params = nullptr;
    float* d_params0 = nullptr;   // copy of the parameters a safeguarded step starts from
    double* d_scalar = nullptr;   // fp64 results of that step's reductions (8)
    int logistic = 0;             // squashing function of C and hidden FC layers: 0 tanh, 1 logistic
    int hint_pt = 0, hint_mp = 0; // mpcnn_set_conv_tiling: 0 = the planner's choice
    int class_max_blocks = 512;   // workgroups of the class-layer kernel's training form resident on the chip
    // limited-memory BFGS: pairs in a ring of lb_m + 1 slots (one always free for the candidate)
    int lb_m = 0, lb_head = 0, lb_count = 0;
    bool lb_have_prev = false;
    float *d_lb_S = nullptr, *d_lb_Y = nullptr;            // [lb_m + 1][n_params]
    float *d_lb_theta_prev = nullptr, *d_lb_g_prev = nullptr, *d_lb_p = nullptr;
    double *d_lb_part = nullptr, *d_lb_alpha = nullptr;    // partial sums (5 x kLbBlocks), first-loop coefficients
    std::vector<double> lb_sy, lb_yy;                      // per slot
    float* d_wread = nullptr;     // what the kernels read: d_params, or its copy rounded to bf16 values
    bool wread_stale = true;
    float* d_grads = nullptr;
    float* d_packs = nullptr;
    bool halves = false;          // some layer has packs of two fp16 parts,
    unsigned* d_words = nullptr;  // and every layer kPeakWords words (kernels_pack.hpp)
    bool packs_stale = true;
    int device = -1;
    float* h_stage = nullptr;     // pinned host memory for one parameter vector: set / get of parameters and gradients (longer than kSmallVector)
    mutable std::mutex stage_mu;  // (gets are const calls)
    bool lds_attr_set = false;
    // plans of the sizes seen so far (oldest dropped first)
    mutable std::vector<std::pair<GeomKey, std::shared_ptr<const Geom>>> geoms;
    // what the last forward / backward left behind (for the test hooks)
    std::shared_ptr<const Geom> last;
    void* last_ws = nullptr;
    // profiling
    bool prof_on = false;
    std::vector<ProfSite> sites;
    std::vector<ProfPending> pending;
    std::vector<hipEvent_t> pool;
};

namespace {

// ------------------------------------------------------------------ profiling
struct ProfScope {
    mpcnn_net* net;
    hipStream_t st;
    hipEvent_t e1 = nullptr;
    ProfScope(mpcnn_net* n, hipStream_t s, const char* name, int layer, int step, double flops,
              double bytes) : net(n), st(s)
    {
        if (!net->prof_on) return;
        int site = -1;
        for (size_t i = 0; i < net->sites.size(); ++i)
            if (net->sites[i].layer == layer && strcmp(net->sites[i].name, name) == 0) { site = (int)i; break; }
        if (site < 0) {
            ProfSite ps{};
            snprintf(ps.name, sizeof ps.name, "%s", name);
            ps.layer = layer; ps.step = step;
            net->sites.push_back(ps);
            site = (int)net->sites.size() - 1;
        }
        net->sites[site].flops = flops;
        net->sites[site].bytes = bytes;
        hipEvent_t e0 = take(), e = take();
        if (!e0 || !e) return;
        (void)hipEventRecord(e0, st);
        e1 = e;
        net->pending.push_back({site, e0, e1});
    }
    ~ProfScope() { if (e1) (void)hipEventRecord(e1, st); }
    hipEvent_t take()
    {
        if (!net->pool.empty()) { hipEvent_t e = net->pool.back(); net->pool.pop_back(); return e; }
        hipEvent_t e = nullptr;
        if (hipEventCreate(&e) != hipSuccess) return nullptr;
        return e;
    }
};
#define LAUNCH(name, layer, step, flops, bytes, ...)                                  \
    do {                                                                              \
        ProfScope ps_(net, st, name, (int)(layer), step, (double)(flops), (double)(bytes)); \
        __VA_ARGS__;                                                                  \
    } while (0)

// ------------------------------------------------------------------ planning
// Tile plan of conv_parts_kernel (P parts per number, mults
// products per step and tile - three parts' plans serve two parts as well -, es bytes per stored element).  Cost of the busiest compute
// unit in cycles: its tiles' matrix instructions on its four SIMDs, a quarter of their staging and stores (most of it lies under the other
// resident workgroup's instructions), and one tile's staging in full at the start.
// `head` classes: with the class layer behind it, all channels in one workgroup.
TilePlan plan_conv_parts(int B, int in_c, int out_r, int out_c, int d, int d2, int k, int k2, int cr, int rpad, int co,
                         const ChanTiling& ct, int P, int mults, size_t es, bool back, int hint_pt, int hint_mp, int head = 0)
{
    TilePlan best;
    const int fh = ceil_div(out_r, d), fw = ceil_div(out_c, d2);
    const int steps = k * k2 * rpad / 16;
    const mpcnn::PartsInstance* list = mpcnn::kParts1;
    size_t list_bytes = sizeof(mpcnn::kParts1);
#define LIST(name) { list = mpcnn::name; list_bytes = sizeof(mpcnn::name); }
    if (head && P == 3) LIST(kHead3) else if (head) LIST(kHead1) else if (P == 3) LIST(kParts3) else if (!back) LIST(kParts1Fwd)
#undef LIST
    const int n_list = (int)(list_bytes / sizeof(list[0]));
    for (int li = 0; li < n_list; ++li) {
        const mpcnn::PartsInstance& in = list[li];
        const int waves = in.WO * in.WP, OT = in.WO * in.MO;
        const bool all = !head && OT == 8;            // (one group where the list's others need two: six tiles and more)
        const int split = head || all ? 1 : ct.split;
        const int CB = in.CB, RP = mpcnn::parts_round(CB, waves), nblk = ceil_div(rpad, CB);
        const int PT = in.WP * in.MP, per_wave = in.MO * in.MP, resident = mpcnn::parts_wgs(P, per_wave) * 4 / waves;
        const size_t pitch = (size_t)mpcnn::parts_pitch(P, CB);   // (two parts take less)
        if ((head ? 32 * OT < co || 16 * OT >= co || 32 * OT > ct.pad : all ? ct.OT * ct.split != 8 || co <= 160 : OT != ct.OT) || (CB > 16 && rpad <= CB / 2)) continue;
        // two channel tiles per wave where the last group fills them (a wave skips its tiles only together)
        if (!head && in.MO == 2 && per_wave <= 4 && ceil_div(co, 32) % 2) continue;
        if (per_wave > 4 && (hint_pt || hint_mp || !mpcnn::half_filter(k, k2))) continue;
        if ((hint_pt && PT != hint_pt) || (hint_mp && in.MP != hint_mp)) continue;
        // Time per matrix instruction against four tiles' per wave.  One part: 2 x 4 tiles take 0.86-0.88 of the time (2 x 2048 x 2048, us,
        // 2 x 2 against 2 x 4: forward 1096, 1745, 1763, 3383 against 954, 1541, 1519, 3103; on 3 x 501 x 389 and smaller, where they are
        // two rounds and less, even: 103 against 100.5), 2 x 2 are ahead of 1 x 4 (2 x 600 x 640, deep net: 110, 169, 152 us against 117,
        // 182, 159), two tiles take 1.17 to 1.3 times as long on large maps; three parts: two tiles against one.  A workgroup alone on its
        // compute unit, its waits in the open, takes 1.4 times as long with one part.
        const double eff = P == 3 ? (per_wave == 2 ? 1.08 : 1.3) : (per_wave > 4 ? 0.88 : per_wave == 4 ? (in.MO == 2 ? 0.98 : 1.0) : 1.2);
        const double alone = P == 3 ? 1.15 : 1.4;
        const double t_mul = (double)steps * mults * OT * PT * 8.0 * eff;   // (on four SIMDs, whatever the waves)
        // filter rows of a block.  All of them, or, from 8 rows on, where blocks are 16 channels, a half, a third ..: a halo of 640
        // positions (fp32) holds a 25 x 25 filter and one position; in rows it holds any.  (32 channels in and out, 160 x 160 positions,
        // forward / data gradient, microseconds whole -> in rows: fp32 20 x 20 435 / 446 -> 207 / 257, 24 x 24 4174 / 5239 -> 401 / 466, 32
        // x 32 16304 / 56978 (plain kernel) -> 696 / 805; bf16 32 x 32 274 / 412 -> 272 / 271, 40 x 40 24336 / 88069 (plain kernel) -> 419
        // / 418.  12 x 12 and less: whole is as fast.)
        for (int parts : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 64, 128}) {
            if (parts > 1 && (k < 8 || CB > 16 || parts > k)) break;
            const int kr = ceil_div(k, parts), nkr = ceil_div(k, kr);
            const size_t beside = (32 * OT + (head ? mpcnn::parts_head_at(CB, rpad, kr * k2) + mpcnn::parts_head(head, in.WO, in.MO, 32 * PT)
                                                   : mpcnn::parts_table(CB, rpad, kr * k2))) * sizeof(float);   // the bias, the steps' places, the class layer's
            const size_t room_lds = std::min((size_t)160 * 1024 / resident, (size_t)(head ? 64 : 160) * 1024);   // (more has to be asked for, some 10 us an instance)
            if (beside + RP * pitch > room_lds) continue;
            const int lds_pos = (int)((room_lds - beside) / (RP * pitch)) * RP;
            const int max_pos = std::min(lds_pos, mpcnn::parts_items(P, per_wave) * RP);   // positions of the halo
            // (tiles that share a residue class's rows, and its columns, as evenly as their number allows; of those with ty rows
            // the widest that fits)
            int last_ty = 0;
            for (int ny = fh; ny >= ceil_div(fh, std::min(fh, 32 * PT)); --ny) {
                const int ty = ceil_div(fh, ny);
                if (ty == last_ty) continue;
                last_ty = ty;
                const int room = std::min(std::min(fw, 32 * PT / ty), max_pos / (ty + kr - 1) - (k2 - 1));
                if (room < 1) continue;
                const int ntx = ceil_div(fw, room), tx = ceil_div(fw, ntx), nty = ceil_div(fh, ty);
                const int npos = (ty + kr - 1) * (tx + k2 - 1);
                const size_t lds = ceil_div(npos, RP) * RP * pitch + beside;   // the halo in whole rounds
                // (byte offsets inside a tile's halo are 31 bits)
                if (((size_t)(ty + kr - 1) * d * in_c + (size_t)(tx + k2 - 1) * d2) * cr * es >= (1ull << 31)) continue;
                if (P == 1 && ((size_t)ty * d * out_c + (size_t)tx * d2) * co * es >= (1ull << 31)) continue;
                const long tiles = (long)B * d * d2 * nty * ntx;
                if (tiles * std::max(std::max(ntx, nty), std::max(d, d2)) >= (1ll << 31)) continue;
                const long wgs = std::min<long>(tiles, std::max(1, resident * kNumCU / split));
                const double per_cu = std::ceil((double)tiles * split / kNumCU);
                const double t_rest = (double)nkr * npos * cr * es / 10 + 2500.0 * nblk * nkr + (head ? 0 : (double)ty * tx * OT * 32 * es * (back ? 2 : 1) / 10) + 1500.0;
                // (narrow tiles count a tenth more: the 32 positions of an operand then lie in more than four rows of the halo, and
                // only successive positions are sure to lie on different LDS banks)
                const double cost = per_cu * ((per_cu < 2 ? alone : 1.0) * (tx >= 8 ? 1.0 : 1.1) * t_mul + 0.25 * t_rest) + t_rest;
                if (!best.ok || cost < best.cost) {
                    best.PT = PT; best.Ty = ty; best.Tx = tx; best.kr = kr;
                    best.nty = nty; best.ntx = ntx; best.lds = lds; best.ok = true;
                    best.wgs = (int)wgs; best.in = in;
                    best.cost = cost;
                }
            }
        }
    }
    if (!best.ok && (hint_pt || hint_mp))   // a pair that no instance serves
        return plan_conv_parts(B, in_c, out_r, out_c, d, d2, k, k2, cr, rpad, co, ct, P, mults, es, back, 0, 0);
    return best;
}

unsigned magic_of(unsigned x) { return x <= 1 ? 0u : (unsigned)(((1ull << 32) + x - 1) / x); }

// Plan of wgrad_parts_kernel.  Candidates: how the result's row tiles (units of 16 channels of one tap) and column
// tiles are dealt to groups of workgroups and to the eight waves, and the tile of positions.  Cost in cycles of the
// busiest compute unit: its tiles' matrix instructions (two waves share a SIMD's), half of what taking a tile in costs
// (its conversions lie under the other wave's instructions, not all of them), a barrier, and the share of the closing
// reduce, which reads every slab's partial result at about 7 bytes per cycle and compute unit.
// `bound`, if given, receives the most floats of partial sums any map size can ask for.
WgradPlan plan_wgrad_parts_in(const Layer& ly, int B, int in_c, int out_r, int out_c, int parts, size_t* bound)
{
    WgradPlan best;
    double best_cost = -1;
    const size_t es = parts == 1 ? 2 : 4;
    const bool two = parts == 2;
    const int planes = ceil_div(ly.cin, 16), kk = ly.k * ly.k2, Nt = ceil_div(ly.cout, 32);
    const int fh = ceil_div(out_r, ly.dil), fw = ceil_div(out_c, ly.dil2);
    if (bound) *bound = 0;
    for (int wn : {1, 2, 4, 8}) {
        if (wn >= 2 * Nt) continue;
        const int gn = ceil_div(Nt, wn);
        for (int ppg = 1; ppg <= planes; ++ppg)
            for (int groups_t = 1; groups_t <= (ppg == 1 ? kk : 1); ++groups_t) {
                const int tpg = ceil_div(kk, groups_t), ntg = ceil_div(kk, tpg), gm = ceil_div(planes, ppg) * ntg;
                if (ntg != groups_t || gm * gn > kNumCU) continue;
                const int RT = ceil_div(ppg * tpg, 2), target = kNumCU / (gm * gn);
                const size_t plen = (size_t)gm * RT * Nt * 1024 + (size_t)Nt * 32;
                for (int wm = 1; wm <= 8 / wn; wm *= 2) {
                    const int wk = 8 / (wn * wm), PM = ceil_div(RT, wm);
                    if (PM > mpcnn::kWpMaxTiles || (wm > 1 && ceil_div(RT, PM) <= wm / 2)) continue;
                    if (bound) *bound = std::max(*bound, (size_t)target * plen);
                    for (int R : {1, 2, 4, 8})
                        for (int nch = 1; nch <= 4; ++nch) {
                            if (R * nch < wk || (R > 1 && R / 2 >= fh) || (nch > 1 && 16 * (nch - 1) >= fw)) continue;
                            const mpcnn::WpGeom g = mpcnn::wp_geom(R, nch, ly.k, ly.k2, ppg, wn, two ? 3 : parts);   // (two parts' plans serve three as well)
                            size_t lds = std::max((size_t)2 * g.buf_b, (size_t)16 * 1024);
                            if (wk > 1) lds = std::max(lds, (size_t)4 * PM * 4096);
                            if (lds > (size_t)160 * 1024 || g.nh + g.nd > mpcnn::kWpItems * mpcnn::kWpThreads) continue;
                            // (byte offsets inside a tile are 31 bits)
                            if (((size_t)g.hh * ly.dil * in_c + (size_t)g.hwp * ly.dil2) * ly.cin * es >= (1ull << 31) ||
                                ((size_t)R * ly.dil * out_c + (size_t)16 * nch * ly.dil2) * ly.cout * es >= (1ull << 31)) continue;
                            const int nty = ceil_div(fh, R), ntx = ceil_div(fw, 16 * nch);
                            const long tiles = (long)B * ly.dil * ly.dil2 * nty * ntx;
                            if (tiles * std::max(std::max(ntx, nty), std::max(ly.dil, ly.dil2)) >= (1l << 31)) continue;
                            const long tps = (tiles + target - 1) / target, slabs = (tiles + tps - 1) / tps;
                            const double chunks = (double)fh / nty * ceil_div(fw, 16) / ntx / wk;   // of a wave and tile, on average
                            const double t_mul = chunks * PM * (parts == 1 ? 1.5 : two ? 3 : 6) * 32 * 2;   // (one part: bound by its operand reads)
                            const double t_load = (g.nh + g.nd) * (8.0 * es / 10 + (parts == 1 ? 15.0 : two ? 40.0 : 75.0) * 6 / 256);
                            const double cost = tps * (std::max(t_mul, 0.5 * t_load) + 0.5 * t_load + 800.0) + (double)slabs * plen * 4 / (7.0 * kNumCU);
                            if (best_cost < 0 || cost < best_cost) {
                                best_cost = cost;
                                best.PM = PM; best.R = R; best.nch = nch; best.RT = RT; best.ppg = ppg; best.tpg = tpg; best.ntg = ntg;
                                best.wm = wm; best.wn = wn; best.wk = wk; best.gm = gm; best.gn = gn; best.Nt = Nt;
                                best.nty = nty; best.ntx = ntx; best.tiles_total = (int)tiles; best.tiles_per_slab = (int)tps;
                                best.slabs = (int)slabs; best.lds = lds; best.plen = plen; best.chain = 16 * chunks * tps; best.two = two; best.ok = true;
                            }
                        }
                }
            }
    }
    return best;
}
// fp32 storage, `half` (two fp16 parts may be used): they are where a wave of the three parts' plan adds at least kHalfChain positions into
// one accumulator.  What two parts leave out is 5e-8 of a gradient (2-norm) whatever the length, what three parts' six products are rounded
// by grows with it.  Three / two parts: 16 positions 2.7e-8 / 4.6e-8 and 64 2.7e-8 / 5.0e-8 (32 -> 64, 5 x 5), 112 3.9e-8 / 4.6e-8 (128 ->
// 200, 2 x 2), 128 4.2e-8 / 4.9e-8, 160 6.5e-8 / 4.7e-8 (64 -> 128, 3 x 3), 256 1.24e-7 / 4.9e-8, 640 3.5e-7 / 5.3e-8, 3904 1.9e-6 /
// 1.05e-6.
constexpr double kHalfChain = 144;
WgradPlan plan_wgrad_parts(const Layer& ly, int B, int in_c, int out_r, int out_c, bool bf16, bool half)
{
    const WgradPlan w = plan_wgrad_parts_in(ly, B, in_c, out_r, out_c, bf16 ? 1 : 3, nullptr);
    return half && w.ok && w.chain >= kHalfChain ? plan_wgrad_parts_in(ly, B, in_c, out_r, out_c, 2, nullptr) : w;
}
// The image layer's weight gradient multiplies on the bf16 instruction where both operands are bf16 and a position's
// deltas are whole 128-bit items; with fp32 storage, and for other map counts, on the fp32 one.
inline bool l0_wgrad_on_bm(const Layer& ly, bool bf16) { return bf16 && ly.cout % 8 == 0; }
// A launch of wgrad_parts_kernel takes some 6 us more than one of wgrad_mfma_kernel whatever it computes (512 threads, both tiles
// converted, up to eight waves' sums to meet): 16 -> 16 channels, 2 x 2 taps, 1300 positions (2.6 MFLOP) 15.0 us against 8.8, 16 -> 16, 3 x
// 3, 2700 positions (12 MFLOP) 16.3 against 12.6; 32 -> 100, 2 x 2, 2600 positions (67 MFLOP) 17.4 against 14.8, but 2 us less in the
// reduce for its fewer slabs.
constexpr double kPartsWgradFlops = 4e7;
// With bf16 storage, one part (us there -> here): in place of wgrad_mfma_kernel (32 maps or fewer, rectangular filters) 16 -> 32, 5 x 5,
// 2.8e8 operations 17.5 -> 20.4, 4.7e8 21.2 -> 21.0, 1.7e10 171 -> 51; 16 -> 16, 3 x 3, 1.1e8 16.4 -> 18.5, 4.3e8 24.3 -> 20.9; 64 -> 32
// 1.4e10 141 -> 49.  Of wgrad_bm_kernel where both counts are multiples of 8: 16 -> 64, 5 x 5, 2.2e9 22.5 -> 25.0, 4.8e9 30.0 -> 27.8; 48
// -> 64, 4 x 4, 4.1e9 29.5 -> 32.7, 9.2e9 45 -> 34, 1.4e11 426 -> 260; 40 -> 200, 2 x 2, 3.2e10 144 -> 146.  Other counts that kernel takes
// channel by channel: 12 -> 100, 4 x 4, 7.8e7 28.0 -> 21.6, 6.3e9 120 -> 43; 100 -> 36, 1 x 1, 6.7e8 72 -> 24.
constexpr double kPart1WgradFlops = 4e8, kPart1WgradFlopsBm = 4.5e9;
// layers that kernel takes: 128-bit (bf16: 64-bit) items of both tensors, more than a sliver of input channels; with bf16 storage those
// that wgrad_tr_kernel does not take, which is ahead (two column tiles per wave, seven operands for ten products: 64 -> 64, 5 x 5, 2 x 2048
// x 2048 1842 against 2304 us)
inline bool wgrad_tr_layer(const Layer& ly) { return !ly.rect && ly.cout > 32 && ly.cin % 32 == 0; }
inline bool wgrad_parts_layer(const Layer& ly, bool bf16)
{
    return ly.wgrad_mfma && ly.cin % 4 == 0 && ly.cin >= 8 && ly.cout % 4 == 0 && !(bf16 && wgrad_tr_layer(ly));
}
inline double parts_wgrad_least(const Layer& ly, bool bf16)
{
    if (!bf16) return kPartsWgradFlops;
    if (ly.rect || ly.cout <= 32) return kPart1WgradFlops;
    return ly.cin % 8 || ly.cout % 8 ? kPartsWgradFlops : kPart1WgradFlopsBm;
}

WgradPlan plan_wgrad(const Layer& ly, int B, int in_r, int in_c, int out_r, int out_c, bool bm)
{
    WgradPlan w;
    const int d = ly.dil, k = ly.k, d2 = ly.dil2, k2 = ly.k2;   // rows; columns
    const int fh = ceil_div(out_r, d), fw = ceil_div(out_c, d2);
    // the kernel forms element offsets inside one image in 32 bits
    // (and, through buffer descriptors, byte offsets inside one image's tensor in 32 bits)
    const size_t es = bm ? 2 : 4;
    const bool fits32 = (size_t)in_r * in_c * ly.cin < (1ull << 31) &&
                        (size_t)out_r * out_c * ly.cout < (1ull << 31) && (k + 3) * d < 65536 &&
                        (size_t)in_r * in_c * ly.cin * es < (1ull << 32) && (size_t)out_r * out_c * ly.cout * es < (1ull << 32);
    // the bf16 instruction's kernels take square filters at one spacing only
    bm = bm && !ly.rect;
    // the bf16 instruction's kernel gives a wave pairs of column tiles: not for 32 maps or fewer
    // - except for an image layer's few channels, where that kernel, half of its instructions wasted,
    // is still ahead of the fp32 instruction's (7 x 7 filters on 2 x 3 x 2048 x 2048, 32 maps: 1.51 -> 1.34 ms)
    bm = bm && (ly.cout > 32 || ly.cin < 8);
    if (bm && ly.wgrad_mfma && fits32 && ly.cin % 32 == 0) {
        // wgrad_tr_kernel: the tiles are raw copies in planes of 32 channels.  Same choices as for
        // wgrad_bm_kernel below: wave split and tile width together, by the busiest workgroup's
        // time - its matrix instructions, or taking the tiles in, whichever is longer.
        const int Mt = k * k * ly.cin / 32 + 1, Nt = ceil_div(ly.cout, 32), Nu = ceil_div(Nt, 2);
        double best = -1;
        for (int wn : {4, 2, 1})
            for (int wm : {1, 2, 4}) {
                if (wm * wn > 4) continue;
                const int wk = 4 / (wm * wn);
                const int gm = ceil_div(Mt, mpcnn::kWgTrMaxTiles * wm), mw = ceil_div(Mt, gm * wm);
                const int gn = ceil_div(Nu, wn);
                const int target = std::max(1, kNumCU / (gm * gn));
                for (int tx = 1; tx <= fw && tx <= 64; ++tx) {
                    const int nch = ceil_div(tx, 16), txp = 16 * nch;
                    const mpcnn::TrGeom tg = mpcnn::tr_geom(nch, k, ly.cin, wn);
                    size_t lds = (size_t)2 * tg.buf_b;
                    if (wk > 1) lds = std::max(lds, (size_t)2 * mw * 2 * 4096);
                    const int h_items = tg.hh * tg.hwp * (ly.cin / 8), d_items = 4 * txp * 8 * wn;
                    if (h_items > mpcnn::kTrStageH * 256 || d_items > mpcnn::kTrStageD * 256 ||
                        lds > kWgradLdsCap || (tg.hwp + 1) * d >= 65536)
                        continue;
                    const int ntx = ceil_div(fw, tx);
                    const long tiles = (long)B * d * d * ceil_div(fh, 4) * ntx;
                    if (tiles * std::max(std::max(ntx, ceil_div(fh, 4)), d) >= (1ll << 31)) continue;
                    const long tps = (tiles + target - 1) / target;
                    const double t_mul = (4.0 / wk) * nch * 2 * mw * 36.0;          // cycles of the instruction stream
                    const double t_load = (h_items + d_items) * 16.0 / 7.0;          // cycles to take the tile in
                    const double cost = (double)tps * (std::max(t_mul, t_load) + 1500.0);
                    if (best < 0 || cost < best) {
                        best = cost;
                        w.wm = wm; w.wn = wn; w.wk = wk; w.mw = mw; w.gm = gm; w.gn = gn;
                        w.Tx = tx; w.TxP = txp; w.lds = std::max(lds, (size_t)1024);
                    }
                }
            }
        if (best >= 0) {
            w.bm = true; w.tr = true; w.Mt = Mt; w.Nt = Nt;
            w.plen = (size_t)Mt * Nt * 1024;
            const int target = std::max(1, kNumCU / (w.gm * w.gn));
            w.nty = ceil_div(fh, 4); w.ntx = ceil_div(fw, w.Tx);
            w.tiles_total = B * d * d * w.nty * w.ntx;
            w.tiles_per_slab = ceil_div(w.tiles_total, target);
            w.slabs = ceil_div(w.tiles_total, w.tiles_per_slab);
            w.ok = true;
            return w;
        }
        w = WgradPlan();
    }
    if (bm && ly.wgrad_mfma && fits32) {
        // wgrad_bm_kernel.  Every group of workgroups (gm x gn of them cover the result) stages
        // all tiles again, and a compute unit takes in roughly 7 bytes per cycle, which at
        // bf16 speed is often the slower side: pick the wave split and the tile width
        // together, by the time of the busiest workgroup.
        const int Mt = ceil_div(k * k * ly.cin + 1, 32), Nt = ceil_div(ly.cout, 32), Nu = ceil_div(Nt, 2);
        const int hh = 4 + k - 1;
        double best = -1;
        for (int wn : {4, 2, 1})
            for (int wm : {1, 2, 4}) {
                if (wm * wn > 4) continue;
                const int wk = 4 / (wm * wn);
                const int gm = ceil_div(Mt, mpcnn::kWgBmMaxTiles * wm), mw = ceil_div(Mt, gm * wm);
                const int gn = ceil_div(Nu, wn);
                const int target = std::max(1, kNumCU / (gm * gn));
                for (int tx = 1; tx <= fw && tx <= 64; ++tx) {
                    const int nch = ceil_div(tx, 16), txp = 16 * nch;
                    const mpcnn::BmGeom bg = mpcnn::bm_geom(nch, k, ly.cin, wn);
                    size_t lds = (size_t)2 * bg.buf_e * 2;
                    if (wk > 1) lds = std::max(lds, (size_t)2 * mw * 2 * 4096);
                    const int h_items = hh * (bg.hwp / 2) * ceil_div(ly.cin, 8), d_items = 4 * (txp / 2) * 8 * wn;
                    if (h_items > mpcnn::kBmStageH * 256 || d_items > mpcnn::kBmStageD * 256 ||
                        lds > kWgradLdsCap || (bg.hwp + 1) * d >= 65536)
                        continue;
                    const int ntx = ceil_div(fw, tx);
                    const long tiles = (long)B * d * d * ceil_div(fh, 4) * ntx;
                    if (tiles * std::max(std::max(ntx, ceil_div(fh, 4)), d) >= (1ll << 31)) continue;
                    const long tps = (tiles + target - 1) / target;
                    const double t_mul = (4.0 / wk) * nch * 2 * mw * 36.0;          // cycles of the instruction stream
                    const double t_load = (h_items + d_items) * 32.0 / 7.0;          // cycles to take the tile in
                    const double cost = (double)tps * (std::max(t_mul, t_load) + 1500.0);
                    if (best < 0 || cost < best) {
                        best = cost;
                        w.wm = wm; w.wn = wn; w.wk = wk; w.mw = mw; w.gm = gm; w.gn = gn;
                        w.Tx = tx; w.TxP = txp; w.lds = std::max(lds, (size_t)1024);
                    }
                }
            }
        if (best >= 0) {
            w.bm = true; w.Mt = Mt; w.Nt = Nt;
            w.plen = (size_t)Mt * Nt * 1024;
            const int target = std::max(1, kNumCU / (w.gm * w.gn));
            w.nty = ceil_div(fh, 4); w.ntx = ceil_div(fw, w.Tx);
            w.tiles_total = B * d * d * w.nty * w.ntx;
            w.tiles_per_slab = ceil_div(w.tiles_total, target);
            w.slabs = ceil_div(w.tiles_total, w.tiles_per_slab);
            w.ok = true;
            return w;
        }
        w = WgradPlan();
    }
    if (ly.wgrad_mfma && fits32) {
        // split of the four waves over result rows / columns / tile rows: least padded work,
        // then fewest workgroup groups (each group stages the tiles again)
        const int Mt = ceil_div(k * k2 * ly.cin, 32), Nt = ceil_div(ly.cout, 32);
        long best_pad = -1; int best_groups = 0;
        for (int wn : {4, 2, 1})
            for (int wm : {1, 2, 4}) {
                if (wm * wn > 4) continue;
                const int wk = 4 / (wm * wn);
                const int gm = ceil_div(Mt, mpcnn::kWgMaxTiles * wm), mw = ceil_div(Mt, gm * wm);
                const int gn = ceil_div(Nt, wn);
                const long pad = (long)gm * wm * mw * gn * wn;
                // (equal on both counts: the split with fewer waves along the tile's rows - measured 3 % ahead
                // on a 16 x 7 tile result, their partial tiles need no meeting in LDS)
                if (best_pad < 0 || pad < best_pad || (pad == best_pad && gm * gn < best_groups) ||
                    (pad == best_pad && gm * gn == best_groups && wk < w.wk)) {
                    best_pad = pad; best_groups = gm * gn;
                    w.wm = wm; w.wn = wn; w.wk = wk; w.mw = mw; w.gm = gm; w.gn = gn;
                }
            }
        w.Mt = Mt; w.Nt = Nt;
        w.plen = (size_t)Mt * Nt * 1024 + (size_t)Nt * 32;
        // tile = 4 rows x Tx columns of a residue class: fewest matrix-core ticks of the busiest
        // workgroup (a tile's work grows with Tx rounded up to 4, plus a fixed cost per tile)
        const int cq = ceil_div(ly.cin, 4), hh = 4 + k - 1;
        const int target = std::max(1, kNumCU / (w.gm * w.gn));
        const double col_ticks = (4.0 / w.wk) * w.mw * 32.0;
        // The loading threads hold a tile's items in registers: 8 halo items each, or, where
        // that keeps the tile narrower than 16 columns (many channels, large filters), 16 -
        // the wider instance issues 8 more loads per tile whether it needs them or not.
        // Staging time of a tile (estimate used to compare the two instances): one trip to
        // memory plus a few hundred cycles per round of 256 items.
        auto tile_time = [&](int txp, bool with_load) {
            const double t_load = 3000.0 + 6.0 * 64.0 * ceil_div(hh * (txp + k2 - 1) * cq + 4 * txp * 8 * w.wn, 256);
            return (with_load ? std::max(txp * col_ticks, t_load) : txp * col_ticks) + 1500.0;
        };
        struct Pick { double cost = -1; int Tx = 0, TxP = 0; size_t lds = 0; long tps = 0; };
        auto pass = [&](int hl, bool with_load) {
            Pick pk;
            for (int tx = 1; tx <= fw; ++tx) {
                const int txp = ceil_div(tx, 4) * 4, hwp = txp + k2 - 1;
                const size_t buf = (size_t)4 * w.wn * (txp * 32 + 32) + (size_t)4 * cq * ((hh * hwp) | 1);
                size_t lds = 2 * buf * sizeof(float) + 128;  // slack: the operand prefetch runs one chunk ahead; 16 unread bytes behind it
                if (w.wk > 1) lds = std::max(lds, (size_t)2 * w.mw * 4096);
                lds = std::max(lds, (size_t)1024);
                if (hh * hwp * cq > hl * 256 || 4 * txp * 8 * w.wn > mpcnn::kWgStageD * 256 || lds > kWgradLdsCap)
                    continue;
                const int ntx = ceil_div(fw, tx);
                const long tiles = (long)B * d * d2 * ceil_div(fh, 4) * ntx;
                if (tiles * std::max(std::max(ntx, ceil_div(fh, 4)), std::max(d, d2)) >= (1ll << 31) || (long)hwp * d2 >= 65536) continue;
                const long tps = (tiles + target - 1) / target;
                const double cost = (double)tps * tile_time(txp, with_load);
                if (pk.cost < 0 || cost <= pk.cost) { pk.cost = cost; pk.Tx = tx; pk.TxP = txp; pk.lds = lds; pk.tps = tps; }
            }
            return pk;
        };
        Pick pk = pass(mpcnn::kWgStageH, false);
        w.hl = mpcnn::kWgStageH;
        if (pk.cost < 0 || (pk.TxP < 16 && pk.Tx < fw)) {
            const Pick wide = pass(2 * mpcnn::kWgStageH, true);
            if (wide.cost >= 0 && (pk.cost < 0 || wide.cost < (double)pk.tps * tile_time(pk.TxP, true))) {
                pk = wide; w.hl = 2 * mpcnn::kWgStageH;
            }
        }
        const double best = pk.cost;
        w.Tx = pk.Tx; w.TxP = pk.TxP; w.lds = pk.lds;
        if (best >= 0) {
            w.nty = ceil_div(fh, 4); w.ntx = ceil_div(fw, w.Tx);
            w.tiles_total = B * d * d2 * w.nty * w.ntx;
            w.tiles_per_slab = ceil_div(w.tiles_total, target);
            w.slabs = ceil_div(w.tiles_total, w.tiles_per_slab);
            w.ok = true;
            return w;
        }
    }
    w = WgradPlan();
    long rows_total = (long)B * out_r;
    w.rows_per_chunk = (int)std::max<long>(1, (rows_total + kDirectWgradChunks - 1) / kDirectWgradChunks);
    w.chunks = (int)((rows_total + w.rows_per_chunk - 1) / w.rows_per_chunk);
    w.plen = ly.p_len;
    return w;
}

// Workgroups of the class-layer kernel: as many as are resident at once (a second, partly
// filled round would double its time; it is a chain of dependent steps per position and lives
// on the bytes in flight), fewer on small maps, whose shares the closing reduce has to add.
int class_blocks(const mpcnn_net* net, long positions)
{
    const long want = std::min<long>(net->class_max_blocks, std::max<long>(512, positions / 1024));
    return (int)std::min<long>(want, (positions + 15) / 16);
}

// Whose largest magnitudes a pass notes, and which tensors squashing functions bound
void plan_peaks(const mpcnn_net* net, Geom* g)
{
    const size_t L = net->layers.size();
    g->delta_peak.assign(L, -1); g->delta_words.assign(L, 0); g->delta_margin.assign(L, 0); g->squashed.assign(L, false);
    for (size_t l = 0; l < L; ++l) g->squashed[l] = net->layers[l].kind == MPCNN_MP ? l > 0 && g->squashed[l - 1] : net->layers[l].tanh_out;
    if (!net->halves || !g->training) return;
    for (size_t l = L - 1; l > 0; --l) {   // the delta at layer l - 1's output
        const Layer& ly = net->layers[l];
        if (ly.kind == MPCNN_MP) {         // every element belongs to at most k x k2 windows
            g->delta_peak[l - 1] = g->delta_peak[l];
            g->delta_words[l - 1] = g->delta_words[l];
            g->delta_margin[l - 1] = g->delta_margin[l];
            for (int w = 1; w < ly.k * ly.k2; w *= 2) ++g->delta_margin[l - 1];
        } else {
            g->delta_words[l - 1] = ly.class_fused ? g->partial_n[l] : g->dgrad[l].ok ? g->dgrad[l].wgs * ly.dgrad_ct.split : 0;
            if (g->delta_words[l - 1] > 0 && g->delta_words[l - 1] <= mpcnn::kDeltaWords) g->delta_peak[l - 1] = (int)l - 1;
        }
    }
}

// Which launches of a layer may work in two fp16 parts: input bounded by a squashing function, deltas whose largest magnitude is noted
bool squashed_input(const Geom& g, size_t l) { return l > 0 && g.squashed[l - 1]; }
bool two_part_forward(const mpcnn_net* net, const Geom& g, size_t l) { return net->layers[l].fwd_half && squashed_input(g, l); }
bool two_part_dgrad(const mpcnn_net* net, const Geom& g, size_t l) { return net->layers[l].dgrad_half && g.delta_peak[l] >= 0; }

// Places in LDS of small_net_kernel's maps above a square of T x T pixels; its bytes, and the multiply-adds of a forward pass over it
size_t small_places(const mpcnn_net* net, int T, bool training, mpcnn::SmallArgs* a, double* work)
{
    const int L = (int)net->layers.size();
    int ex = 0;
    for (int l = L; l-- > 0;) {
        const Layer& ly = net->layers[l];
        mpcnn::SmallLayer& s = a->layer[l];
        s.pool = ly.kind == MPCNN_MP; s.k = ly.k; s.d = ly.dil; s.ci = ly.cin; s.co = ly.cout; s.squash = ly.tanh_out;
        s.w = (int)ly.p_off; s.ex = ex; s.side = T + ex;
        s.mg_co = magic_of(ly.cout); s.mg_ci = magic_of(ly.cin); s.mg_k = magic_of(ly.k); s.mg_side = magic_of(s.side);
        s.mg_items = s.pool ? 0 : magic_of((unsigned)ly.p_len);
        ex += (ly.k - 1 + ly.drop) * ly.dil;
    }
    a->T = T; a->ex0 = ex; a->side0 = T + ex; a->mg_side0 = magic_of(a->side0); a->C = net->in_ch; a->mg_c = magic_of(a->C);
    a->n_layers = L; a->n_params = (int)net->n_params; a->n_cls = net->n_cls; a->training = training ? 1 : 0;
    a->mg_t = magic_of(T);
    size_t off = net->n_params, deltas = (size_t)T * T * net->n_cls;
    a->table = (int)off; off += (size_t)64 * L;
    a->grad = (int)off;
    if (training) off += net->n_params;
    a->red = (int)off;
    if (training) off += mpcnn::kSmallRed;
    a->img = (int)off; off += (size_t)a->side0 * a->side0 * a->C;
    *work = 0;
    for (int l = 0; l < L; ++l) {
        mpcnn::SmallLayer& s = a->layer[l];
        const size_t n = (size_t)s.side * s.side * s.co;
        s.act = (int)off; off += n;
        if (l + 1 < L) deltas = std::max(deltas, n);
        *work += (double)n * s.k * s.k * (s.pool ? 1 : s.ci);
    }
    for (int i = 0; i < 2; ++i) { a->delta[i] = (int)off; if (training) off += deltas; }
    off *= sizeof(float);
    for (int l = 0; l < L; ++l)
        if (a->layer[l].pool) { a->layer[l].code = (int)off; off += (size_t)a->layer[l].side * a->layer[l].side * a->layer[l].co; }
    return align_up(off, 16);
}
constexpr size_t kSmallLds = 64 * 1024 - 2048;   // (the arguments and the sums of the loss lie beside)
// Nets that small_net_kernel takes, at every size and with any tiling hint (so that a pixel's probabilities do not depend on the call that computes
// them): fp32 storage, square windows and filters, nothing for the convolutions' matrix instruction, and of these the ones that it does not slow down on
// large images, where launches cost nothing.  235 nets drawn at random, one image of 1536 x 1536 or 2048 x 2048, time of training / probabilities
// against layer by layer:
//   three layers with parameters or more.  Two are four launches (hidden 8, filter 6 x 6 on one map 1.44 / 1.40, on 3 x 3 .62 / .66; 3, 3 x 3, behind it 5,
//     5 x 5 .61 / 1.07), one is two (.53 / 1.17);
//   no convolution of four or eight maps: the layers' kernels take four maps per thread (8, 3 x 3, pool, 2 on 6 x 6 1.70 / .51; 8, 5 x 5, pool, 7 on 5 x 5
//     1.43 / .79; 4, 3 x 3, pool, 4 on 4 x 4 1.09 / .66);
//   150 filter taps, of which 64 on a single map: with one channel a product costs two reads of LDS (7, 7 x 7, 5, 2 .87 / 1.26; 1, 5 x 5, pool, 6 on 6 x 6
//     .75 / 1.26; 6, 7 x 7, 6, 4 x 4, 5, 2 1.16 / .77; 6, 5 x 5, pool, 7 on 5 x 5 1.08 / .96);
//   LDS for training's squares of 14 x 14 (5, 3 x 3, pool of 3, 4 on 4 x 4, 2 in squares of 12 x 12 1.24 / 1.02), at a halo of two thirds more than the
//     pixels themselves at most (5, 2 x 2, between pools of 3 and 2 1.07 / .87).
// The 93 nets that are left: 1.00 / 1.01 at most, .52 / .64 in the middle; on 64 x 64 pixels .3 to .6.
constexpr int kSmallTaps = 150, kSmallTapsOnOne = 64, kSmallLeast = 14;
bool small_net_fits(const mpcnn_net* net)
{
    if (net->bf16 || net->layers.size() > (size_t)mpcnn::kSmallLayers) return false;
    long taps = 0, on_one = 0;
    int with_params = 0;
    for (const Layer& ly : net->layers) {
        if (ly.rect || ly.k2 != ly.k || ly.drop2 != ly.drop || ly.dil2 != ly.dil || ly.k > 32 || ly.fwd_mfma || ly.cin > mpcnn::kSmallChannels ||
            ly.cout > mpcnn::kSmallChannels || (ly.kind == MPCNN_C && ly.cout % 4 == 0)) return false;
        if (ly.kind == MPCNN_MP) continue;
        ++with_params;
        taps += (long)ly.k * ly.k * ly.cout;
        if (ly.cin == 1) on_one += (long)ly.k * ly.k * ly.cout;
    }
    if (with_params < 3 || taps > kSmallTaps || on_one > kSmallTapsOnOne) return false;
    mpcnn::SmallArgs a{};
    double pixel = 0;
    for (const Layer& ly : net->layers) pixel += (double)ly.cout * ly.k * ly.k * (ly.kind == MPCNN_MP ? 1 : ly.cin);
    for (int T = kSmallLeast; T <= mpcnn::kSmallSide; T += 2) {
        double work = 0;
        if (small_places(net, T, true, &a, &work) > kSmallLds) break;
        if (3 * work <= 5 * pixel * T * T) return true;
    }
    return false;
}
void plan_small(const mpcnn_net* net, Geom* g, int out_r, int out_c)
{
    g->small_net = false;
    if (!small_net_fits(net)) return;
    double best = -1;
    for (int T = 4; T <= mpcnn::kSmallSide; T += 2) {
        mpcnn::SmallArgs a{};
        double work = 0;
        const size_t lds = small_places(net, T, g->training, &a, &work);
        if (lds > kSmallLds) break;
        a.nty = ceil_div(out_r, T); a.ntx = ceil_div(out_c, T);
        const long tiles = (long)g->B * a.nty * a.ntx;
        if (tiles * std::max(a.nty, a.ntx) >= (1l << 31)) continue;
        // A square takes as long as its multiply-adds and some 7600 more per layer (steps and barriers); two that share a compute unit take 1.35
        // times as long as one.
        const long per_cu = (tiles + kNumCU - 1) / kNumCU;
        const double cost = (per_cu / 2 * 1.35 + per_cu % 2) * (7600.0 * net->layers.size() + work);
        if (best >= 0 && cost >= best) continue;
        best = cost;
        a.tiles = (int)tiles; a.mg_ntx = magic_of(a.ntx); a.mg_nty = magic_of(a.nty);
        g->small_net = true; g->small = a; g->small_lds = lds;
        g->small_wgs = (int)std::min<long>(tiles, mpcnn::kSmallWgs);
    }
}

bool make_geom(const mpcnn_net* net, int B, int H, int W, bool training, Geom* g, bool mirrored = false,
               bool fixed_partials = false)
{
    g->fixed_partials = fixed_partials;
    if (B < 1 || H < net->patch || W < net->patch) return false;
    const size_t L = net->layers.size();
    g->B = B; g->H = H; g->W = W; g->training = training;
    g->rows.assign(L, 0); g->cols.assign(L, 0);
    g->act_off.assign(L, 0); g->code_off.assign(L, 0);
    g->fwd.assign(L, TilePlan()); g->dgrad.assign(L, TilePlan()); g->wgrad.assign(L, WgradPlan());
    g->partial_off.assign(L, 0); g->partial_n.assign(L, 0); g->partial_len.assign(L, 0);
    size_t off = 0, max_act = 0;
    const size_t es = net->bf16 ? 2 : 4;   // bytes per stored activation / delta element
    g->src_h = H; g->src_w = W;
    g->staged = net->in_ch > 1 || net->bf16 || mirrored;
    if (g->staged) {
        g->staged_off = off;
        off = align_up(off + es * (size_t)B * H * W * net->in_ch);
    }
    plan_small(net, g, H - net->patch + 1, W - net->patch + 1);
    int r = H, c = W;
    for (size_t l = 0; l < L; ++l) {
        const Layer& ly = net->layers[l];
        const int in_r = r, in_c = c;
        // a pool that leaves `drop` trailing rows of every patch's map unused shortens the
        // whole-image map by as many rows of this spacing
        r -= (ly.k - 1 + ly.drop) * ly.dil;
        c -= (ly.k2 - 1 + ly.drop2) * ly.dil2;
        if (r < 1 || c < 1) return false;
        g->rows[l] = r; g->cols[l] = c;
        size_t bytes = es * (size_t)B * r * c * ly.cout;
        max_act = std::max(max_act, bytes);
        if (ly.kind == MPCNN_MP || g->small_net) continue;
        if (ly.fwd_mfma)
            g->fwd[l] = plan_conv_parts(B, in_c, r, c, ly.dil, ly.dil2, ly.k, ly.k2, ly.cin, ly.fwd_rpad, ly.cout, ly.fwd_ct,
                                        net->bf16 ? 1 : 3, net->bf16 ? 1 : ly.fwd_half ? 3 : 6, es, false, net->hint_pt, net->hint_mp);
        if (training && ly.class_fused) {
            g->partial_n[l] = class_blocks(net, (long)B * r * c);
            g->partial_len[l] = ly.p_len;
        } else if (training) {
            if (ly.dgrad_mfma && l > 0)
                g->dgrad[l] = plan_conv_parts(B, c, in_r, in_c, ly.dil, ly.dil2, ly.k, ly.k2, ly.cout, ly.dgrad_rpad, ly.cin, ly.dgrad_ct,
                                              net->bf16 ? 1 : 3, net->bf16 ? 1 : ly.dgrad_half ? 3 : 6, es, true, net->hint_pt, net->hint_mp);
        }
    }
    if (r != H - net->patch + 1 || c != W - net->patch + 1) return false;
    g->head = false;
    if (!training && !g->small_net && L >= 2 && net->layers[L - 1].class_fused && g->fwd[L - 2].ok && !net->hint_pt && !net->hint_mp) {
        // Nothing of the hidden layer is kept, so it need not pass through memory on its way to the classes - where that way takes longer than the wait for
        // all channels in one workgroup.  Whole passes, us, two launches / one: a map of few tiles does not fill the chip (64 -> 200, 5 x 5, 60 x 67
        // 36.1 / 41.1, bf16 64 -> 68, 40 x 47 33.5 / 36.4), larger ones do (128 -> 200, 2 x 2, 97 x 104 43 / 33, bf16 1000 x 1007 526 / 397; behind four pools
        // 81 x 98, 256 tiles, 71.3 / 69.7).  The pass over the hidden layer counts 0.006 cycles per element, and 3000 where bf16 would have two groups.
        // Five tiles of 32 units on the eight waves of fp32 storage leave three SIMDs half empty, which many tiles per compute unit show (32 -> 132, 3 x 3,
        // 600 x 607 286 / 317, 32 -> 160 in three parts, 430 x 437 180 / 185, 64 -> 132 192 / 196; few of them 97 x 104 34 / 28): there only from four and a half
        // tiles on and in two parts (64 -> 160, 1000 x 1007 1085 / 990).  Of 900 plans of 68 .. 200 units, 40 x 47 .. 1000 x 1007, two are slower by 2 %.
        const Layer& ly = net->layers[L - 2];
        const TilePlan& apart = g->fwd[L - 2];
        const TilePlan tp = plan_conv_parts(B, L > 2 ? g->cols[L - 3] : W, r, c, ly.dil, ly.dil2, ly.k, ly.k2, ly.cin, ly.fwd_rpad, ly.cout, ly.fwd_ct,
                                            net->bf16 ? 1 : 3, net->bf16 ? 1 : ly.fwd_half ? 3 : 6, es, false, 0, 0, net->n_cls);
        const long tiles = (long)B * ly.dil * ly.dil2 * tp.nty * tp.ntx;
        const bool half_empty = !net->bf16 && ceil_div(ly.cout, 32) == 5 && (ly.cout <= 144 || !ly.fwd_half) && tiles > 4 * kNumCU;
        const double apart_cost = apart.cost + 0.006 * B * r * c * ly.cout + (net->bf16 && ly.cout > 128 ? 3000 : 0);
        if (tp.ok && !half_empty && (tiles >= kNumCU || tp.cost <= apart_cost)) { g->fwd[L - 2] = tp; g->head = true; }
    }
    if (g->small_net) {
        // (A forward pass needs none of it, but asks for what it did layer by layer: what a caller's workspace, or the static one, is too small for does
        // not depend on the kernel that runs.)
        off = training ? 0 : off + 2 * align_up(max_act);
        for (size_t l = 0; training && l < L; ++l) {
            const size_t elems = (size_t)B * g->rows[l] * g->cols[l] * net->layers[l].cout;
            g->act_off[l] = off; off = align_up(off + sizeof(float) * elems);
            if (net->layers[l].kind == MPCNN_MP) { g->code_off[l] = off; off = align_up(off + elems); }
            g->small.layer[l].rows = g->rows[l]; g->small.layer[l].cols = g->cols[l];
        }
        g->small_partial_off = off;
        if (training) off = align_up(off + sizeof(float) * net->n_params * (fixed_partials ? mpcnn::kSmallWgs : g->small_wgs));
        g->loss_partial_off = off;
        g->total = align_up(off + sizeof(double) * kLossBlocks);
        g->label_h = H; g->probs_rows = r; g->accumulate = false;
        g->small.B = B; g->small.W = W; g->small.Ho = r; g->small.Wo = c; g->small.ctr = (net->patch - 1) / 2;
        return true;
    }
    plan_peaks(net, g);
    for (size_t l = 0; training && l < L; ++l) {
        const Layer& ly = net->layers[l];
        if (ly.kind == MPCNN_MP || ly.class_fused) continue;
        const int in_r = l ? g->rows[l - 1] : H, in_c = l ? g->cols[l - 1] : W, out_r = g->rows[l], out_c = g->cols[l];
        if (wgrad_parts_layer(ly, net->bf16) && 2.0 * B * out_r * out_c * ly.cout * ly.k * ly.k2 * ly.cin >= parts_wgrad_least(ly, net->bf16))
            g->wgrad[l] = plan_wgrad_parts(ly, B, in_c, out_r, out_c, net->bf16, squashed_input(*g, l) && g->delta_peak[l] >= 0);
        if (!g->wgrad[l].ok) g->wgrad[l] = plan_wgrad(ly, B, in_r, in_c, out_r, out_c, net->bf16);
        const WgradPlan& w = g->wgrad[l];
        g->partial_n[l] = w.ok ? w.slabs : w.chunks;
        g->partial_len[l] = w.plen;
    }
    g->l0_fused = false;
    if (training && L >= 2) {
        const Layer& l0 = net->layers[0];
        const Layer& l1 = net->layers[1];
        const size_t lds = sizeof(float) * ((size_t)mpcnn::kL0Rows * mpcnn::kL0Cols * l0.cout +
                                            (size_t)(mpcnn::kL0Rows + l0.k - 1) * (mpcnn::kL0Cols + l0.k - 1) * l0.cin);
        if (l0.kind != MPCNN_MP && !l0.class_fused && !l0.rect && l0.dil == 1 && l1.kind == MPCNN_MP && !l1.rect &&
            l1.dil == 1 && l1.k >= 2 && l1.k <= 4 && l0.cout % 4 == 0 && l0.p_len <= (size_t)mpcnn::kL0MaxPerThread * 256 && lds <= 64 * 1024 &&
            (long)B * ceil_div(g->rows[0], mpcnn::kL0Rows) * ceil_div(g->cols[0], mpcnn::kL0Cols) <= 2 * kNumCU) {
            // small images only (one tile per workgroup, where the two separate launches are
            // bound by their round trips to memory): the kernel multiplies on the vector ALU,
            // and on a large image the matrix-core kernel behind a separate routing pass is faster
            g->l0_fused = true;
            g->l0_nty = ceil_div(g->rows[0], mpcnn::kL0Rows); g->l0_ntx = ceil_div(g->cols[0], mpcnn::kL0Cols);
            g->l0_blocks = B * g->l0_nty * g->l0_ntx;
            g->l0_lds = lds;
            g->wgrad[0] = WgradPlan();
            g->partial_n[0] = g->l0_blocks;
            g->partial_len[0] = l0.p_len;
        }
    }
    if (training && !g->l0_fused) {
        // the image layer's weight gradient on its own matrix-instruction kernel
        const Layer& l0 = net->layers[0];
        if (l0.kind != MPCNN_MP && !l0.class_fused && !l0.rect && l0.dil == 1 && (l0.cin == 1 || l0.cin == 3) &&
            (l0.k == 3 || l0.k == 5 || l0.k == 7)) {
            WgradPlan w;
            w.l0m = true;
            const long tiles = (long)B * ceil_div(g->rows[0], mpcnn::kL0wTy) * ceil_div(g->cols[0], mpcnn::kL0wTx);
            w.tiles_total = (int)tiles;
            // two workgroups per compute unit are resident with the largest filter banks (140 registers):
            // a third, waiting its turn, would walk its tiles alone at the end
            w.chunks = (int)std::min<long>(tiles, 2L * kNumCU);
            w.plen = l0.p_len;
            if (tiles < (1l << 30)) {
                g->wgrad[0] = w;
                g->partial_n[0] = w.chunks;
                g->partial_len[0] = l0.p_len;
            }
        }
    }
    if (training) {
        for (size_t l = 0; l < L; ++l) {
            const Layer& ly = net->layers[l];
            size_t elems = (size_t)B * g->rows[l] * g->cols[l] * ly.cout;
            g->act_off[l] = off;
            off = align_up(off + es * elems);
            if (ly.kind == MPCNN_MP) {
                g->code_off[l] = off;
                off = align_up(off + elems);
            }
        }
        g->delta_off[0] = off; off = align_up(off + max_act);
        g->delta_off[1] = off; off = align_up(off + max_act);
        for (size_t l = 0; l < L; ++l) {
            if (!g->partial_n[l]) continue;
            g->partial_off[l] = off;
            // A pass over bands sizes the buffers of the partial sums by bounds that do not depend
            // on the map's size: the number of slabs a plan ends up with is not monotonic in it (a
            // map with a few tiles more than workgroups gets half as many slabs of two tiles),
            // and the workspace is sized by the tallest band, the last one being shorter.  A
            // one-piece pass takes what its plan needs.  (The class layer's share count depends
            // on an occupancy query made when the net first touches the device, which may be
            // after the caller asked for the workspace size: always the bound.)
            const Layer& ly = net->layers[l];
            size_t alloc_f;
            if (ly.class_fused) alloc_f = (size_t)kLossBlocks * g->partial_len[l];
            else if (!fixed_partials) alloc_f = (size_t)g->partial_n[l] * g->partial_len[l];
            else {
                const size_t rows_w = (size_t)ly.k * ly.k2 * ly.cin, Nt = ceil_div(ly.cout, 32);
                const size_t tiled = std::max((size_t)ceil_div((int)rows_w, 32) * Nt * 1024 + Nt * 32,
                                              (size_t)ceil_div((int)rows_w + 1, 32) * Nt * 1024);
                alloc_f = std::max((size_t)kNumCU * tiled,
                                   (size_t)std::max(kDirectWgradChunks, 2 * kNumCU) * ly.p_len);
                if (wgrad_parts_layer(ly, net->bf16)) {
                    size_t bound = 0;
                    (void)plan_wgrad_parts_in(ly, 1, 1, 1, 1, net->bf16 ? 1 : 3, &bound);
                    alloc_f = std::max(alloc_f, bound);
                }
                alloc_f = std::max(alloc_f, (size_t)g->partial_n[l] * g->partial_len[l]);
            }
            off = align_up(off + sizeof(float) * alloc_f);
        }
    } else {
        // forward only: layers alternate between two buffers, nothing is kept
        size_t buf[2];
        buf[0] = off; off = align_up(off + max_act);
        buf[1] = off; off = align_up(off + max_act);
        for (size_t l = 0; l < L; ++l) g->act_off[l] = buf[l & 1];
    }
    g->loss_partial_off = off; off = align_up(off + sizeof(double) * kLossBlocks);
    if (net->halves && training) { g->delta_words_off = off; off = align_up(off + sizeof(unsigned) * mpcnn::kDeltaWords * L); }
    g->total = off;
    g->label_h = H; g->probs_rows = r; g->accumulate = false;
    return true;
}


// Launch geometry of the max-filter kernels: 256 (column, channel quad) items of one map row
// per workgroup.  False if the map is too large for their 32-bit index arithmetic.
bool row_grid(int B, int h, int w, int C4, int d, mpcnn::RowGrid* g)
{
    const long per_row = (long)w * C4, gx = (per_row + 255) / 256, rows = (long)B * h;
    if (gx * rows >= (1l << 31) || gx * rows * gx >= (1l << 32) || (gx * 256) * C4 >= (1l << 32) ||
        rows * h >= (1l << 32))
        return false;
    g->gx = (int)gx; g->rows = (int)rows; g->h = h; g->C4 = C4;
    g->mg_gx = magic_of((unsigned)gx); g->mg_h = magic_of((unsigned)h); g->mg_c4 = magic_of((unsigned)C4);
    // row order: residue classes mod d (h rows: the first h mod d classes have one row more)
    g->d = d < h ? d : 1;
    g->rem = h % g->d; g->n1 = h / g->d + (g->rem ? 1 : 0);
    if (g->rem == 0) g->rem = g->d;          // all classes have n1 rows
    g->mg_n1 = magic_of((unsigned)g->n1); g->mg_n0 = magic_of((unsigned)(g->n1 - 1));
    return true;
}

// Launch geometry of maxfilter_fwd2x2_kernel: row pairs (y, y + d) of one residue class mod d, column
// pairs in blocks of 2 d columns.  False if the map is too large for 32-bit index arithmetic.
bool pair_grid(int B, int h, int w, int C4, int d, mpcnn::PairGrid* g)
{
    const int D2 = 2 * d, q = h / D2, rem = h % D2;
    const int nbig = std::min(rem, d);
    const long S = (long)nbig * (q + 1) + (long)(d - nbig) * q;
    const long Sx = (long)(w / D2) * d + std::min(w % D2, d);
    if (S < 1 || Sx < 1) return false;
    const long per_row = Sx * C4, gx = (per_row + 255) / 256, rows = (long)B * S;
    if (gx * rows >= (1l << 31) || gx * rows * gx >= (1l << 32) || (gx * 256) * C4 >= (1l << 32) ||
        rows * S >= (1l << 32) || (long)h * D2 >= (1l << 31))
        return false;
    g->gx = (int)gx; g->rows = (int)rows; g->S = (int)S; g->C4 = C4; g->Sx = (int)Sx; g->d = d;
    g->nbig = nbig; g->q1 = q + 1;
    g->mg_gx = magic_of((unsigned)gx); g->mg_S = magic_of((unsigned)S); g->mg_c4 = magic_of((unsigned)C4);
    g->mg_q1 = magic_of((unsigned)(q + 1)); g->mg_q0 = magic_of((unsigned)q); g->mg_d = magic_of((unsigned)d);
    return true;
}

inline int grid_for(long total, int block = 256, int cap = 1 << 20)
{
    long g = (total + block - 1) / block;
    return (int)std::min<long>(std::max<long>(g, 1), cap);
}

// ------------------------------------------------------------------ MFMA launches
// conv_parts_kernel: the plan's workgroups walk the tiles; its divisors' magic numbers
void parts_grid(mpcnn::ConvArgs* a, dim3* grid, const TilePlan& tp)
{
    a->tiles_total = (int)grid->x; a->kr = tp.kr;
    a->mg_hw = magic_of((unsigned)(a->Tx + a->k2 - 1)); a->mg_tx = magic_of((unsigned)a->Tx);
    a->mg_ntx = magic_of((unsigned)a->ntx); a->mg_nty = magic_of((unsigned)a->nty);
    a->mg_d = magic_of((unsigned)a->d); a->mg_d2 = magic_of((unsigned)a->d2);
    grid->x = (unsigned)tp.wgs;
}

// (the kernel instances live in launch_*.hip, one translation unit per family)
template <typename T>
bool launch_conv(const mpcnn::ConvArgs& a, const TilePlan& tp, dim3 grid, hipStream_t st)
{
    const bool back = a.mode >= mpcnn::kDgradTanh;
    if constexpr (std::is_same<T, float>::value)
        return (back ? mpcnn::launch_conv_parts_f32_back : mpcnn::launch_conv_parts_f32_fwd)(a, tp.in, grid, tp.lds, st);
    else
        return (back ? mpcnn::launch_conv_parts_b16_back : mpcnn::launch_conv_parts_b16_fwd)(a, tp.in, grid, tp.lds, st);
}
template <typename T>
bool launch_wgrad_mfma(const mpcnn::WgradArgs& a, int hl, dim3 grid, size_t lds, hipStream_t st)
{
    if constexpr (std::is_same<T, float>::value) return mpcnn::launch_wgrad_f32(a, hl, grid, lds, st);
    else return mpcnn::launch_wgrad_b16(a, hl, grid, lds, st);
}
void launch_first_bm(const mpcnn::FirstBmArgs& a, unsigned wgs, hipStream_t st)
{
    const int nt = a.Co <= 32 ? 1 : 2;
#define CASE(n, kk) if (nt == n && a.k == kk) { mpcnn::first_layer_bm_kernel<n, kk><<<wgs, 256, 0, st>>>(a); return; }
    CASE(1, 3) CASE(1, 5) CASE(1, 7) CASE(2, 3) CASE(2, 5) CASE(2, 7)
#undef CASE
}
// Estimated cycles of the image layer's launch with `mp` rows per wave, ct slices of 32 maps: a compute unit's matrix instructions, and for every round of
// its resident workgroups what a round takes besides (image in, LDS, squashing, pool, stores).
double first_cost(int k, int ci, int B, int rows, int cols, int ct, int mp, bool pool)
{
    const bool large = k == 7 && ci == 3;             // (its filters take the registers)
    const int resident = mp == 4 ? (pool || large ? 2 : 3) : large ? 3 : mp == 2 ? 4 : 5, less = pool ? 1 : 0;
    const long per_cu = ((long)B * ceil_div(rows, 4 * mp - less) * ceil_div(cols, 32 - less) * ct + kNumCU - 1) / kNumCU;
    return per_cu * mp * 64.0 * k * ceil_div(k * ci, 2) + (per_cu + resident - 1) / resident * (2000.0 + 1500.0 * mp);
}
// Rows per wave.  Alone: as many as still give every compute unit two workgroups.  With the pool behind it: the least time.  Whole forward passes, us,
// 1 / 2 / 4 rows: 16 maps, 3 x 3, 256 x 265 27.3 / 28.2 / 29.4, 512 x 521 56.0 / 55.8 / 59.8; 64 maps, 5 x 5 of three channels, 360 x 369 67.4 / 63.9 / 72.0;
// 7 x 7 of three channels, 32 maps, 300 x 309 50.1 / 47.0 / 49.3, 420 x 429 76.2 / 73.7 / 71.5, 512 x 521 101 / 88 / 98, 128 maps, 1024 x 1033
// 1127 / 903 / 868.
int first_rows(int k, int ci, int B, int rows, int cols, int ct, bool pool)
{
    int mp = 4;
    if (!pool) {
        while (mp > 1 && (long)B * ceil_div(rows, 4 * mp) * ceil_div(cols, 32) * ct < 2L * kNumCU) mp >>= 1;
        return mp;
    }
    for (int i : {2, 1}) if (first_cost(k, ci, B, rows, cols, ct, i, true) <= first_cost(k, ci, B, rows, cols, ct, mp, true)) mp = i;
    return mp;
}
// fp32 storage, the image layer on the fp32 matrix instruction: instance by filter side, channels and rows per wave
bool launch_first_mfma(const mpcnn::FirstMfmaArgs& a0, int k, int ci, int B, bool pool, hipStream_t st)
{
    mpcnn::FirstMfmaArgs a = a0;
    const int ct = ceil_div(a.Co, 32), rows = pool ? a.Hp : a.Ho, cols = pool ? a.Wp : a.Wo, less = pool ? 1 : 0;
    const int mp = first_rows(k, ci, B, rows, cols, ct, pool);
    a.nty = ceil_div(rows, 4 * mp - less); a.ntx = ceil_div(cols, 32 - less);
    const dim3 grid((unsigned)(B * a.nty * a.ntx), (unsigned)ct);
#define CASE(kk, cc, mm)                                                                              \
    if (k == kk && ci == cc && mp == mm) {                                                            \
        if (pool) mpcnn::first_layer_mfma_kernel<kk, cc, mm, true><<<grid, 256, 0, st>>>(a);          \
        else mpcnn::first_layer_mfma_kernel<kk, cc, mm><<<grid, 256, 0, st>>>(a);                     \
        return true;                                                                                  \
    }
#define CASES(kk, cc) CASE(kk, cc, 1) CASE(kk, cc, 2) CASE(kk, cc, 4)
    CASES(3, 1) CASES(5, 1) CASES(7, 1) CASES(3, 3) CASES(5, 3) CASES(7, 3)
#undef CASES
#undef CASE
    return false;
}
// fp32 storage: layers of one or three channels at spacing 1 - the image's, and any other layer that narrow before the first pool - on the fp32
// matrix instruction; they are too narrow for conv_parts_kernel, and the plain kernel multiplies on the vector ALU.
bool narrow_on_mfma(const mpcnn_net* net, const Geom& g, size_t l)
{
    const Layer& ly = net->layers[l];
    return !net->bf16 && ly.kind != MPCNN_MP && !ly.class_fused && !g.fwd[l].ok && !ly.rect && ly.dil == 1 && (ly.cin == 1 || ly.cin == 3) &&
           (ly.k == 3 || ly.k == 5 || ly.k == 7) && (long)g.B * g.rows[l] * g.cols[l] < (1l << 31) / 32;
}
// ... the image layer's with the pool behind it: nothing kept, 2 x 2, and where what its tiles compute twice is less than the pool's own launch and its
// way to memory and back, 12000 cycles and 0.002 per number that the L2 caches do not hold.  (7 x 7 filters on three channels, whole passes, us, two
// launches / one: 128 maps, 200 x 209 58.3 / 60.1, 256 x 256 71.0 / 77.0, 256 x 265 96.7 / 78.0.  Of 220 sizes one is slower, by 0.3 us.)
bool first_with_pool(const mpcnn_net* net, const Geom& g)
{
    if (g.training || net->layers.size() < 2 || !narrow_on_mfma(net, g, 0) || net->layers[1].kind != MPCNN_MP || net->layers[1].rect || net->layers[1].k != 2) return false;
    const Layer& ly = net->layers[0];
    const int ct = ceil_div(ly.cout, 32);
    auto cost = [&](int l, bool pool) {
        return first_cost(ly.k, ly.cin, g.B, g.rows[l], g.cols[l], ct, first_rows(ly.k, ly.cin, g.B, g.rows[l], g.cols[l], ct, pool), pool);
    };
    return cost(1, true) <= cost(0, false) + 12000 + 0.002 * std::max(0.0, (double)g.B * g.rows[0] * g.cols[0] * ly.cout - 8e6);
}
template <typename T>
bool launch_l0_wgrad(const mpcnn::L0WgradArgs& a, int k, int ci, dim3 grid, hipStream_t st)
{
#define CASE(kk, cc) if (k == kk && ci == cc) { mpcnn::l0_wgrad_mfma_kernel<kk, cc, T><<<grid, 256, 0, st>>>(a); return true; }
    CASE(3, 1) CASE(5, 1) CASE(7, 1) CASE(3, 3) CASE(5, 3) CASE(7, 3)
#undef CASE
    return false;
}
bool launch_l0_wgrad_bm(const mpcnn::L0WgradArgs& a, int k, int ci, dim3 grid, hipStream_t st)
{
#define CASE(kk, cc) if (k == kk && ci == cc) { mpcnn::l0_wgrad_bm_kernel<kk, cc><<<grid, 256, 0, st>>>(a); return true; }
    CASE(3, 1) CASE(5, 1) CASE(7, 1) CASE(3, 3) CASE(5, 3) CASE(7, 3)
#undef CASE
    return false;
}
// Kernels that may ask for more than 64 KiB of dynamic LDS must say so once.
mpcnn_status set_lds_attrs(bool bf16_storage)
{
    if (bf16_storage) { HIP_TRY(mpcnn::conv_parts_attrs_b16_fwd()); HIP_TRY(mpcnn::conv_parts_attrs_b16_back());
                        HIP_TRY(mpcnn::wgrad_attrs_b16()); HIP_TRY(mpcnn::wgrad_parts_attrs<mpcnn::bf16>()); }
    else { HIP_TRY(mpcnn::conv_parts_attrs_f32_fwd()); HIP_TRY(mpcnn::conv_parts_attrs_f32_back());
           HIP_TRY(mpcnn::wgrad_attrs_f32()); HIP_TRY(mpcnn::wgrad_parts_attrs<float>()); }
    return MPCNN_OK;
}

// Quads of channels per lane of class_layer_kernel, 16 lanes a position.  (Three classes and more in bf16 are bound by instructions: three quads of 64 bits
// rather than two accesses of 128 where these are a quarter empty and more: 160 -> 3, 1200 x 1200 positions, 243 -> 223 us.  Two are bound by memory.)
int class_quads(int K, int ncls, bool bf16)
{
    return bf16 && K % 8 == 0 && !(ncls > 2 && K > 128 && K <= 192) ? (K <= 128 ? 2 : 4) : (K + 63) / 64;
}
// bf16 storage with a multiple of 8 channels: 8 channels per 128-bit access (Q = 2)
template <int NCLS, int KV, typename T>
void launch_class_inst(const mpcnn::ClassArgs& a, bool train, int blocks, hipStream_t st)
{
    constexpr bool kPairs = sizeof(T) == 2 && KV % 2 == 0;
    if (kPairs && a.K % 8 == 0) {
        if (train) mpcnn::class_layer_kernel<NCLS, KV, true, T, kPairs ? 2 : 1><<<blocks, 256, 0, st>>>(a);
        else mpcnn::class_layer_kernel<NCLS, KV, false, T, kPairs ? 2 : 1><<<blocks, 256, 0, st>>>(a);
    } else {
        if (train) mpcnn::class_layer_kernel<NCLS, KV, true, T><<<blocks, 256, 0, st>>>(a);
        else mpcnn::class_layer_kernel<NCLS, KV, false, T><<<blocks, 256, 0, st>>>(a);
    }
}
template <int NCLS, int KV, typename T>
int class_occupancy_inst(int K)
{
    constexpr bool kPairs = sizeof(T) == 2 && KV % 2 == 0;
    int n = 0;
    hipError_t e;
    if (kPairs && K % 8 == 0)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, mpcnn::class_layer_kernel<NCLS, KV, true, T, kPairs ? 2 : 1>, 256, 0);
    else
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, mpcnn::class_layer_kernel<NCLS, KV, true, T>, 256, 0);
    return e == hipSuccess ? n : 0;
}
// workgroups of the training form that one CU holds at once (0 if unknown)
template <typename T>
int class_occupancy(int ncls, int KV, int K)
{
#define CASE(n, v) if (ncls == n && KV == v) return class_occupancy_inst<n, v, T>(K)
    CASE(2, 1); CASE(3, 1); CASE(4, 1); CASE(2, 2); CASE(3, 2); CASE(4, 2); CASE(2, 3); CASE(3, 3); CASE(4, 3); CASE(2, 4); CASE(3, 4); CASE(4, 4);
#undef CASE
    return 0;
}
template <typename T>
void launch_class(const mpcnn::ClassArgs& a, int ncls, int KV, bool train, int blocks, hipStream_t st)
{
#define CASE(n, v) if (ncls == n && KV == v) return launch_class_inst<n, v, T>(a, train, blocks, st)
    CASE(2, 1); CASE(3, 1); CASE(4, 1); CASE(2, 2); CASE(3, 2); CASE(4, 2); CASE(2, 3); CASE(3, 3); CASE(4, 3); CASE(2, 4); CASE(3, 4); CASE(4, 4);
#undef CASE
}

mpcnn_status refresh_packs(mpcnn_net* net, hipStream_t st)
{
    if (net->bf16 && net->wread_stale) {
        const long n = (long)net->n_params;
        LAUNCH("round_params", -1, 0, 0, 8.0 * n,
               mpcnn::round_params_kernel<<<grid_for(n), 256, 0, st>>>(net->d_params, net->d_wread, n));
    }
    net->wread_stale = false;
    if (!net->packs_stale || !net->d_packs) { net->packs_stale = false; return MPCNN_OK; }
    mpcnn::PackArgs pa{};
    pa.W = net->d_wread; pa.Q = net->d_packs;
    double bytes = 0;
    bool first = false;
    auto flush = [&]() {
        if (!pa.n_seg) return;
        if (first)
            LAUNCH("weight_peaks", -1, 0, 0, 4.0 * net->n_params,
                   (mpcnn::weight_peaks_kernel<<<dim3(mpcnn::kPeakParts, (unsigned)pa.n_seg), 256, 0, st>>>(pa)));
        LAUNCH("pack_weights", -1, 0, 0, bytes,
               net->bf16 ? mpcnn::pack_weights_kernel<true><<<(unsigned)pa.total_blocks, 256, 0, st>>>(pa)
                         : mpcnn::pack_weights_kernel<false><<<(unsigned)pa.total_blocks, 256, 0, st>>>(pa));
        pa.n_seg = pa.total_blocks = 0; bytes = 0; first = false;
    };
    auto add = [&](size_t l, size_t off, size_t len, int rpad, int opad, int back, int parts, bool notes) {
        if (pa.n_seg == mpcnn::kMaxPackSegs) flush();
        const Layer& ly = net->layers[l];
        notes = notes && net->halves;
        first = first || notes;
        pa.seg[pa.n_seg++] = {(long)ly.p_off, (long)off, net->halves ? net->d_words + mpcnn::kPeakWords * l : nullptr, ly.k * ly.k2, ly.cin, ly.cout, rpad, opad, back,
                              pa.total_blocks, parts, notes ? 1 : 0};
        pa.total_blocks += (int)((len / (4 * parts) + 255) / 256);   // 16 bytes per part and thread
        bytes += 4.0 * (len + ly.p_len);
    };
    const int parts = net->bf16 ? 1 : 3;
    for (size_t l = 0; l < net->layers.size(); ++l) {
        const Layer& ly = net->layers[l];
        if (ly.kind == MPCNN_MP) continue;
        if (ly.fwd_mfma) add(l, ly.fwd_pack_off, ly.fwd_pack_len, ly.fwd_rpad, ly.fwd_ct.pad, 0, parts, true);
        if (ly.dgrad_mfma && l > 0) add(l, ly.dgrad_pack_off, ly.dgrad_pack_len, ly.dgrad_rpad, ly.dgrad_ct.pad, 1, parts, !ly.fwd_mfma);
        if (ly.fwd_half) add(l, ly.fwd_half_off, ly.fwd_half_len, ly.fwd_rpad, ly.fwd_ct.pad, 0, 2, false);
        if (ly.dgrad_half) add(l, ly.dgrad_half_off, ly.dgrad_half_len, ly.dgrad_rpad, ly.dgrad_ct.pad, 1, 2, false);
    }
    flush();
    HIP_TRY(hipGetLastError());
    net->packs_stale = false;
    return MPCNN_OK;
}

// Words of the delta at layer l's output, null where nobody notes them
unsigned* delta_words(const Geom& g, char* ws, size_t l)
{
    return g.training && g.delta_peak[l] >= 0 ? (unsigned*)(ws + g.delta_words_off) + mpcnn::kDeltaWords * g.delta_peak[l] : nullptr;
}
// What conv_parts_kernel has to know of a layer's weights
void weights_of(mpcnn::ConvArgs* a, const mpcnn_net* net, size_t l)
{
    const Layer& ly = net->layers[l];
    a->w_peak = net->d_words + mpcnn::kPeakWords * l;
    a->small_limit = ly.k * ly.k2 * std::min(ly.cin, ly.cout);
}

// Forward through every layer; in training mode everything is kept for the backward.
// T = storage type of activations and deltas (float, or bf16 with fp32 arithmetic).
template <typename T>
mpcnn_status run_forward(mpcnn_net* net, const Geom& g, const float* image, char* ws,
                         const int32_t* labels, const float* pixw, float* probs, void* dZ_,
                         double* loss_dev, hipStream_t st)
{
    using namespace mpcnn;
    constexpr bool kF32 = std::is_same<T, float>::value;
    constexpr double es = sizeof(T);
    mpcnn_status rc = refresh_packs(net, st);
    if (rc != MPCNN_OK) return rc;
    if constexpr (kF32)
        if (g.small_net) {
            SmallArgs a = g.small;
            a.image = image; a.params = net->d_params; a.labels = labels; a.pixw = pixw; a.probs = probs;
            a.partial = (float*)(ws + g.small_partial_off);
            a.loss_partial = labels && loss_dev ? (double*)(ws + g.loss_partial_off) : nullptr;
            a.Hs = g.src_h; a.Ws = g.src_w; a.top = g.pad_top; a.left = g.pad_left;
            a.label_h = g.label_h; a.probs_rows = g.probs_rows;
            a.mse = net->loss_kind == MPCNN_LOSS_MSE; a.logistic = net->logistic;
            double flops = 0;
            for (int l = 0; l < a.n_layers; ++l) {
                const Layer& ly = net->layers[l];
                if (ly.kind != MPCNN_MP) flops += 2.0 * g.B * g.rows[l] * g.cols[l] * ly.cout * ly.k * ly.k * ly.cin * (g.training ? (l ? 3.0 : 2.0) : 1.0);
                if (!g.training) continue;
                a.layer[l].act_out = (float*)(ws + g.act_off[l]);
                if (a.layer[l].pool) a.layer[l].code_out = (uint8_t*)(ws + g.code_off[l]);
            }
            net->loss_out = loss_dev;
            net->loss_shares = a.loss_partial ? g.small_wgs : 0;
            LAUNCH("small_net", -1, 1, flops, 4.0 * g.B * ((double)a.C * g.H * g.W + (double)net->n_cls * a.Ho * a.Wo),
                   small_net_kernel<<<(unsigned)g.small_wgs, kSmallThreads, g.small_lds, st>>>(a));
            HIP_TRY(hipGetLastError());
            return MPCNN_OK;
        }
    const int B = g.B;
    T* dZ = static_cast<T*>(dZ_);
    const T* in = nullptr;
    int Hi = g.H, Wi = g.W, Ci = net->in_ch;
    const bool pooled_first = kF32 && first_with_pool(net, g);
    if (pooled_first) in = reinterpret_cast<const T*>(image);
    else if (g.staged) {
        T* staged = (T*)(ws + g.staged_off);
        long total = (long)B * Ci * Hi * Wi;
        LAUNCH("stage_input", -1, 0, 0, (4.0 + es) * total,
               stage_input_kernel<T><<<grid_for(total), 256, 0, st>>>(image, staged, B, Ci, Hi, Wi, g.src_h,
                                                                       g.src_w, g.pad_top, g.pad_left));
        in = staged;
    } else if constexpr (kF32) {
        in = image;
    }
    const size_t L = net->layers.size();
    double* lp = (double*)(ws + g.loss_partial_off);
    const bool want_loss = labels && loss_dev;
    net->loss_shares = 0; net->loss_out = loss_dev;
    for (size_t l = 0; l < L; ++l) {
        const Layer& ly = net->layers[l];
        T* out = (T*)(ws + g.act_off[l]);
        const int Ho = g.rows[l], Wo = g.cols[l];
        const double n_in = (double)B * Hi * Wi * Ci, n_out = (double)B * Ho * Wo * ly.cout;
        if (ly.kind == MPCNN_MP) {
            uint8_t* code = g.training ? (uint8_t*)(ws + g.code_off[l]) : nullptr;
            long total = (long)B * Ho * Wo * ly.cout;
            mpcnn::RowGrid rg;
            mpcnn::PairGrid pg;
            constexpr int kQ = kF32 ? 1 : 2;   // channels per thread / 4 (bf16: 8 channels = one 128-bit access)
            if (!ly.rect && ly.k == 2 && ly.cout % (4 * kQ) == 0 && pair_grid(B, Ho, Wo, ly.cout / (4 * kQ), ly.dil, &pg))
                LAUNCH("maxfilter_fwd", l, 2, 0, n_out * (2.0 * es + (code ? 1.0 : 0.0)),
                       (maxfilter_fwd2x2_kernel<T, kQ><<<(unsigned)(pg.gx * pg.rows), 256, 0, st>>>(
                           in, out, code, pg, Hi, Wi, ly.cout, Ho, Wo)));
            else if (!kF32 && ly.cout % 8 == 0 && row_grid(B, Ho, Wo, ly.cout / 8, ly.dil, &rg))   // bf16: 8 channels per thread (fp32: measured slower)
                LAUNCH("maxfilter_fwd", l, 2, 0, n_out * (2.0 * es + (code ? 1.0 : 0.0)),
                       (maxfilter_fwd4_kernel<T, kF32 ? 1 : 2><<<(unsigned)(rg.gx * rg.rows), 256, 0, st>>>(
                           in, out, code, rg, Hi, Wi, ly.cout, Ho, Wo, ly.k, ly.k2, ly.dil, ly.dil2)));
            else if (ly.cout % 4 == 0 && row_grid(B, Ho, Wo, ly.cout / 4, ly.dil, &rg))
                LAUNCH("maxfilter_fwd", l, 2, 0, n_out * (2.0 * es + (code ? 1.0 : 0.0)),
                       (maxfilter_fwd4_kernel<T, 1><<<(unsigned)(rg.gx * rg.rows), 256, 0, st>>>(
                           in, out, code, rg, Hi, Wi, ly.cout, Ho, Wo, ly.k, ly.k2, ly.dil, ly.dil2)));
            else
                LAUNCH("maxfilter_fwd", l, 2, 0, n_out * (2.0 * es + (code ? 1.0 : 0.0)),
                       maxfilter_fwd_direct_kernel<T><<<grid_for(total), 256, 0, st>>>(
                           in, out, code, B, Hi, Wi, ly.cout, Ho, Wo, ly.k, ly.k2, ly.dil, ly.dil2));
        } else if (ly.class_fused) {
            // last FC + softmax + cross-entropy (+ its own backward when labels are given)
            const long M = (long)B * Ho * Wo;
            ClassArgs a{};
            a.h = in; a.Wk = net->d_wread + ly.p_off; a.probs = probs;
            a.labels = labels; a.pixw = pixw; a.pixw_any = pixw ? pixw : reinterpret_cast<const float*>(labels); a.dH = dZ;
            a.partial = g.training ? (float*)(ws + g.partial_off[l]) : nullptr;   // loss only: no gradient shares
            a.loss_partial = want_loss ? lp : nullptr;
            a.B = B; a.Ho = Ho; a.Wo = Wo; a.H = g.label_h; a.W = g.W; a.ctr = (net->patch - 1) / 2;
            a.probs_rows = g.probs_rows;
            a.K = Ci; a.tanh_below = (l > 0 && net->layers[l - 1].tanh_out) ? 1 + net->logistic : 0;
            a.mse = net->loss_kind == MPCNN_LOSS_MSE;
            a.peak = l > 0 ? delta_words(g, ws, l - 1) : nullptr;
            const int blocks = class_blocks(net, M);
            const bool train = labels != nullptr;
            const double flops = 2.0 * M * Ci * ly.cout * (train ? 3.0 : 1.0);
            const double bytes = es * n_in * (train ? 2.0 : 1.0) + 4.0 * n_out;
            LAUNCH("class_layer", l, train ? 4 : 3, flops, bytes,
                   launch_class<T>(a, ly.cout, class_quads(Ci, ly.cout, !kF32), train, blocks, st));
            // (in training the shares are added by the reduce launch that ends the backward)
            if (train && want_loss) net->loss_shares = blocks;
        } else {
            const float* Wk = net->d_wread + ly.p_off;
            const double flops = 2.0 * B * Ho * Wo * ly.cout * ly.k * ly.k2 * Ci;
            const double bytes = es * (n_in + n_out) + 4.0 * ly.p_len;
            const int step = (l == L - 1) ? 3 : 1;
            if (ly.fwd_mfma && g.fwd[l].ok) {
                const TilePlan& tp = g.fwd[l];
                ConvArgs a{};
                a.in = in; a.wpack = (const v4f*)(net->d_packs + ly.fwd_pack_off);
                a.bias = Wk + (size_t)ly.k * ly.k2 * Ci * ly.cout; a.act = nullptr; a.out = out;
                a.B = B; a.Hi = Hi; a.Wi = Wi; a.Cr = Ci; a.CrPad = ly.fwd_rpad;
                a.Ho = Ho; a.Wo = Wo; a.Co = ly.cout; a.CoPad = ly.fwd_ct.pad;
                a.k = ly.k; a.d = ly.dil; a.origin = 0; a.k2 = ly.k2; a.d2 = ly.dil2; a.origin2 = 0;
                a.Ty = tp.Ty; a.Tx = tp.Tx; a.nty = tp.nty; a.ntx = tp.ntx;
                a.mode = ly.tanh_out ? kFwdTanh : kFwdLinear; a.logistic = net->logistic;
                dim3 grid((unsigned)(B * ly.dil * ly.dil2 * tp.nty * tp.ntx), (unsigned)(tp.in.WO * tp.in.MO == ly.fwd_ct.OT ? ly.fwd_ct.split : 1));
                parts_grid(&a, &grid, tp); a.wraw = Wk;
                if (two_part_forward(net, g, l)) {
                    weights_of(&a, net, l);
                    a.wpack2 = (const v4f*)(net->d_packs + ly.fwd_half_off);
                }
                bool launched = false;
                if (g.head && l == L - 2) {
                    const Layer& last = net->layers[L - 1];
                    a.head = {net->d_wread + last.p_off, probs, labels, pixw, want_loss ? lp : nullptr, net->n_cls, net->loss_kind == MPCNN_LOSS_MSE,
                              g.label_h, g.W, (net->patch - 1) / 2, g.probs_rows};
                    const double n_probs = (double)B * Ho * Wo * last.cout;
                    LAUNCH(kF32 ? "conv_class_parts" : "conv_class_bm", l, step, flops + 2.0 * n_probs * ly.cout, es * n_in + 4.0 * (ly.p_len + n_probs),
                           launched = (kF32 ? mpcnn::launch_conv_head_f32 : mpcnn::launch_conv_head_b16)(a, tp.in, grid, tp.lds, st));
                    if (want_loss) net->loss_shares = tp.wgs;
                } else
                    LAUNCH(kF32 ? "conv_fwd_parts" : "conv_fwd_bm", l, step, flops, bytes, launched = launch_conv<T>(a, tp, grid, st));
                if (!launched)   // a plan without a kernel instance: a planner bug, never a silent skip
                    return fail(MPCNN_EUNSUPPORTED, "layer %zu: no convolution kernel instance for its forward plan", l);
            } else if (!kF32 && l == 0 && ly.dil == 1 && Ci <= 4 && ly.cout <= 64 && (ly.k == 3 || ly.k == 5 || ly.k == 7)) {
                // bf16 storage, the image layer: short reduction on the bf16 matrix instruction
                FirstBmArgs a{};
                a.in = (const mpcnn::bf16*)in; a.Wk = Wk; a.out = (mpcnn::bf16*)out;
                a.B = B; a.Hi = Hi; a.Wi = Wi; a.Ci = Ci; a.Ho = Ho; a.Wo = Wo; a.Co = ly.cout; a.k = ly.k;
                a.squash = ly.tanh_out ? 1 + net->logistic : 0;
                a.nty = ceil_div(Ho, kFirstBmTy); a.ntx = ceil_div(Wo, kFirstBmTx);
                const unsigned wgs = (unsigned)std::min<long>((long)B * a.nty * a.ntx, 4L * kNumCU);
                LAUNCH("first_layer_bm", l, step, flops, bytes, launch_first_bm(a, wgs, st));
            } else if (kF32 && narrow_on_mfma(net, g, l)) {
                // short reduction on the fp32 matrix instruction
                FirstMfmaArgs a{};
                a.in = (const float*)in; a.Wk = Wk; a.out = (float*)out;
                a.B = B; a.Hi = Hi; a.Wi = Wi; a.Ho = Ho; a.Wo = Wo; a.Co = ly.cout;
                a.squash = ly.tanh_out ? 1 + net->logistic : 0;
                bool launched = false;
                if (pooled_first) {
                    a.Hs = g.src_h; a.Ws = g.src_w; a.top = g.pad_top; a.left = g.pad_left;
                    a.Hp = g.rows[1]; a.Wp = g.cols[1];
                    a.out = (float*)(ws + g.act_off[1]);
                }
                LAUNCH(pooled_first ? "first_pool_mfma" : "first_layer_mfma", l, step, flops, pooled_first ? es * (n_in + (double)B * a.Hp * a.Wp * a.Co) : bytes,
                       launched = launch_first_mfma(a, ly.k, Ci, B, pooled_first, st));
                if (!launched) return fail(MPCNN_EUNSUPPORTED, "layer %zu: no image-layer kernel instance", l);
                if (pooled_first) {                   // (the next layer's work is done)
                    in = (const T*)a.out; Hi = a.Hp; Wi = a.Wp; Ci = ly.cout;
                    ++l;
                    continue;
                }
            } else {
                const int og = ceil_div(ly.cout, 4);
                const long total = (long)B * Ho * Wo * og;
                const size_t wbytes = sizeof(float) * ((size_t)ly.k * ly.k2 * Ci + 1) * 4 * og;
                const int w_in_lds = wbytes <= 48 * 1024;
                LAUNCH("first_layer", l, step, flops, bytes,
                       first_layer_kernel<T><<<(unsigned)((total + 255) / 256), 256, w_in_lds ? wbytes : 0, st>>>(
                           in, Wk, out, B, Hi, Wi, Ci, Ho, Wo, ly.cout, ly.k, ly.k2, ly.dil, ly.dil2,
                           ly.tanh_out ? 1 + net->logistic : 0,
                           w_in_lds));
            }
        }
        if (g.head && l == L - 2) break;              // (the class layer's work is done)
        in = out; Hi = Ho; Wi = Wo; Ci = ly.cout;
    }
    if (!net->layers[L - 1].class_fused) {
        // class logits -> probabilities, deltas, loss
        long total = (long)B * Hi * Wi;
        int blocks = (int)std::min<long>(kSoftmaxBlocks, (total + 255) / 256);
        LAUNCH("softmax_ce", L - 1, 3, 0, total * ((4.0 + 2.0 * es) * net->n_cls + 8.0),
               softmax_ce_kernel<T><<<blocks, 256, 0, st>>>(in, probs, labels, pixw, dZ,
                                                         want_loss ? lp : nullptr, B, Hi, Wi, g.label_h, g.W,
                                                         (net->patch - 1) / 2, net->n_cls,
                                                         net->loss_kind == MPCNN_LOSS_MSE, g.probs_rows));
        if (want_loss) net->loss_shares = blocks;
    }
    HIP_TRY(hipGetLastError());
    return MPCNN_OK;
}

template <typename T>
mpcnn_status run_backward(mpcnn_net* net, const Geom& g, const float* image, char* ws,
                          hipStream_t st)
{
    using namespace mpcnn;
    constexpr bool kF32 = std::is_same<T, float>::value;
    constexpr double es = sizeof(T);
    const int B = g.B;
    const size_t L = net->layers.size();
    const T* in0 = nullptr;
    if (g.staged) in0 = (const T*)(ws + g.staged_off);
    else if constexpr (kF32) in0 = image;
    T* dbuf[2] = {(T*)(ws + g.delta_off[0]), (T*)(ws + g.delta_off[1])};
    int cur = 0;  // dbuf[cur] holds dL/d(pre-activation) of layer l's output (dL/d(output) for MP)
    // a fused class layer has already done its own backward and left the delta below it (a small net's pass has done all)
    for (size_t li = g.small_net ? 0 : net->layers[L - 1].class_fused ? L - 1 : L; li-- > 0;) {
        const Layer& ly = net->layers[li];
        const int Ho = g.rows[li], Wo = g.cols[li];
        const T* A = li == 0 ? in0 : (const T*)(ws + g.act_off[li - 1]);
        const int Hi = li == 0 ? g.H : g.rows[li - 1], Wi = li == 0 ? g.W : g.cols[li - 1];
        const int Ci = ly.cin;
        const bool below_tanh = li > 0 && net->layers[li - 1].tanh_out;
        const T* dY = dbuf[cur];
        T* dA = dbuf[cur ^ 1];
        const double n_in = (double)B * Hi * Wi * Ci, n_out = (double)B * Ho * Wo * ly.cout;
        if (ly.kind == MPCNN_MP) {
            if (li == 0) break;  // nothing below has parameters
            const uint8_t* code = (const uint8_t*)(ws + g.code_off[li]);
            if (li == 1 && g.l0_fused) {
                const Layer& l0 = net->layers[0];
                L0Args a{};
                a.in = in0; a.act1 = A; a.dP = dY; a.code = code;
                a.partial = (float*)(ws + g.partial_off[0]);
                a.B = B; a.Hi = g.H; a.Wi = g.W; a.Ci = l0.cin; a.H1 = Hi; a.W1 = Wi; a.C1 = Ci;
                a.k = l0.k; a.Hp = Ho; a.Wp = Wo;
                a.nty = g.l0_nty; a.ntx = g.l0_ntx;
                a.slope = below_tanh ? (net->logistic ? 2 : 1) : 0;
                const double wflops = 2.0 * B * Hi * Wi * Ci * l0.k * l0.k * l0.cin;
                const double wbytes = n_out * (es + 1.0) + n_in * (below_tanh ? es : 0.0) + es * B * g.H * g.W * l0.cin + 4.0 * l0.p_len;
                if (ly.k == 2)
                    LAUNCH("l0_wgrad_fused", 0, 5, wflops, wbytes,
                           (l0_wgrad_fused_kernel<T, 2><<<(unsigned)g.l0_blocks, 256, g.l0_lds, st>>>(a)));
                else if (ly.k == 3)
                    LAUNCH("l0_wgrad_fused", 0, 5, wflops, wbytes,
                           (l0_wgrad_fused_kernel<T, 3><<<(unsigned)g.l0_blocks, 256, g.l0_lds, st>>>(a)));
                else
                    LAUNCH("l0_wgrad_fused", 0, 5, wflops, wbytes,
                           (l0_wgrad_fused_kernel<T, 4><<<(unsigned)g.l0_blocks, 256, g.l0_lds, st>>>(a)));
                break;  // the image needs no gradient
            }
            long total = (long)B * Hi * Wi * Ci;
            const double bytes = n_out * (es + 1.0) + n_in * es * (below_tanh ? 2.0 : 1.0);
            mpcnn::RowGrid rg;
            mpcnn::PairGrid pg;
            // 2 x 2 windows: 2 x 2 elements per thread, 8 channels each (4 where the count is no multiple of 8);
            // not where a position is under one 128-byte line and neighbours are adjacent (measured slower)
            const int pq = Ci % 8 == 0 ? 2 : 1;
            if (!ly.rect && ly.k == 2 && Ci % 4 == 0 && (ly.dil > 1 || Ci * es >= 128) && pair_grid(B, Hi, Wi, Ci / (4 * pq), ly.dil, &pg)) {
                const unsigned wgs = (unsigned)(pg.gx * pg.rows);
#define PAIR_BWD(TP, QQ) LAUNCH("maxfilter_bwd", li, 7, 0, bytes, (maxfilter_bwd2x2_kernel<TP, T, QQ><<<wgs, 256, 0, st>>>( \
                             dY, code, A, dA, pg, Hi, Wi, Ci, Ho, Wo, net->logistic)))
                if (below_tanh && pq == 2) PAIR_BWD(true, 2);
                else if (below_tanh) PAIR_BWD(true, 1);
                else if (pq == 2) PAIR_BWD(false, 2);
                else PAIR_BWD(false, 1);
#undef PAIR_BWD
                cur ^= 1;
                continue;
            }
            const bool octs = Ci % 8 == 0 && row_grid(B, Hi, Wi, Ci / 8, ly.dil, &rg);   // 8 channels per thread (measured faster in both storage types)
            const bool quads = !octs && Ci % 4 == 0 && row_grid(B, Hi, Wi, Ci / 4, ly.dil, &rg);
            if (octs && below_tanh)
                LAUNCH("maxfilter_bwd", li, 7, 0, bytes,
                       (maxfilter_bwd4_kernel<true, T, 2><<<(unsigned)(rg.gx * rg.rows), 256, 0, st>>>(
                           dY, code, A, dA, rg, Hi, Wi, Ci, Ho, Wo, ly.k, ly.k2, ly.dil, ly.dil2, net->logistic)));
            else if (octs)
                LAUNCH("maxfilter_bwd", li, 7, 0, bytes,
                       (maxfilter_bwd4_kernel<false, T, 2><<<(unsigned)(rg.gx * rg.rows), 256, 0, st>>>(
                           dY, code, A, dA, rg, Hi, Wi, Ci, Ho, Wo, ly.k, ly.k2, ly.dil, ly.dil2, net->logistic)));
            else if (quads && below_tanh)
                LAUNCH("maxfilter_bwd", li, 7, 0, bytes,
                       (maxfilter_bwd4_kernel<true, T, 1><<<(unsigned)(rg.gx * rg.rows), 256, 0, st>>>(
                           dY, code, A, dA, rg, Hi, Wi, Ci, Ho, Wo, ly.k, ly.k2, ly.dil, ly.dil2, net->logistic)));
            else if (quads)
                LAUNCH("maxfilter_bwd", li, 7, 0, bytes,
                       (maxfilter_bwd4_kernel<false, T, 1><<<(unsigned)(rg.gx * rg.rows), 256, 0, st>>>(
                           dY, code, A, dA, rg, Hi, Wi, Ci, Ho, Wo, ly.k, ly.k2, ly.dil, ly.dil2, net->logistic)));
            else if (below_tanh)
                LAUNCH("maxfilter_bwd", li, 7, 0, bytes,
                       (maxfilter_bwd_direct_kernel<true, T><<<grid_for(total), 256, 0, st>>>(
                           dY, code, A, dA, B, Hi, Wi, Ci, Ho, Wo, ly.k, ly.k2, ly.dil, ly.dil2, net->logistic)));
            else
                LAUNCH("maxfilter_bwd", li, 7, 0, bytes,
                       (maxfilter_bwd_direct_kernel<false, T><<<grid_for(total), 256, 0, st>>>(
                           dY, code, A, dA, B, Hi, Wi, Ci, Ho, Wo, ly.k, ly.k2, ly.dil, ly.dil2, net->logistic)));
        } else {
            const double flops = 2.0 * B * Ho * Wo * ly.cout * ly.k * ly.k2 * Ci;
            const int wstep = (li == L - 1) ? 4 : 5, dstep = (li == L - 1) ? 4 : 6;
            // parameter gradient: partial sums over slabs of positions, then a fixed-order sum
            const WgradPlan& wp = g.wgrad[li];
            float* partial = (float*)(ws + g.partial_off[li]);
            if (wp.ok && wp.PM > 0) {
                {
                    WgradPartsArgs a{};
                    a.in = A; a.dY = dY; a.partial = partial;
                    a.B = B; a.Hi = Hi; a.Wi = Wi; a.Ci = Ci; a.Ho = Ho; a.Wo = Wo; a.Co = ly.cout;
                    a.k = ly.k; a.k2 = ly.k2; a.d = ly.dil; a.d2 = ly.dil2;
                    a.R = wp.R; a.nch = wp.nch; a.nty = wp.nty; a.ntx = wp.ntx;
                    a.tiles_total = wp.tiles_total; a.tiles_per_slab = wp.tiles_per_slab;
                    a.Nt = wp.Nt; a.RT = wp.RT; a.wm = wp.wm; a.wn = wp.wn; a.wk = wp.wk;
                    a.ppg = wp.ppg; a.tpg = wp.tpg; a.ntg = wp.ntg;
                    a.dy_peak = delta_words(g, ws, li); a.dy_words = g.delta_words[li]; a.dy_margin = g.delta_margin[li];
                    a.out = net->logistic && kF32 && ly.tanh_out ? (const float*)(ws + g.act_off[li]) : nullptr;
                    if (!wp.two) a.dy_peak = nullptr;
                    a.mg_nqh = magic_of(2 * wp.ppg); a.mg_hwp = magic_of(16 * wp.nch + ly.k2 - 1); a.mg_txp = magic_of(16 * wp.nch);
                    a.mg_tpg = magic_of(wp.tpg); a.mg_k2 = magic_of(ly.k2); a.mg_ntx = magic_of(wp.ntx); a.mg_nty = magic_of(wp.nty);
                    a.mg_d = magic_of(ly.dil); a.mg_d2 = magic_of(ly.dil2);
                    dim3 grid((unsigned)wp.slabs, (unsigned)wp.gm, (unsigned)wp.gn);
                    bool launched = false;
                    LAUNCH(kF32 ? "wgrad_parts" : "wgrad_bm", li, wstep, flops, es * (n_in + n_out) + 4.0 * ly.p_len,
                           launched = mpcnn::launch_wgrad_parts<T>(a, wp.PM, grid, wp.lds, st));
                    if (!launched)
                        return fail(MPCNN_EUNSUPPORTED, "layer %zu: no weight-gradient kernel instance for its plan", li);
                }
            } else if (wp.ok) {
                WgradArgs a{};
                a.in = A; a.dY = dY; a.partial = partial;
                a.B = B; a.Hi = Hi; a.Wi = Wi; a.Ci = Ci;
                a.Ho = Ho; a.Wo = Wo; a.Co = ly.cout; a.k = ly.k; a.d = ly.dil; a.k2 = ly.k2; a.d2 = ly.dil2;
                a.Tx = wp.Tx; a.TxP = wp.TxP; a.nty = wp.nty; a.ntx = wp.ntx;
                a.tiles_total = wp.tiles_total; a.tiles_per_slab = wp.tiles_per_slab;
                a.Mt = wp.Mt; a.Nt = wp.Nt; a.wm = wp.wm; a.wn = wp.wn; a.wk = wp.wk; a.mw = wp.mw;
                a.mg_cq = magic_of(ceil_div(Ci, 4)); a.mg_hwp = magic_of(wp.TxP + ly.k2 - 1);
                if (wp.tr) {   // items of one position x 8 channels
                    a.mg_cq = magic_of(Ci / 8);
                    a.mg_hwp = magic_of(mpcnn::tr_geom(wp.TxP / 16, ly.k, Ci, wp.wn).hwp);
                } else if (wp.bm) {   // items of two positions x 8 channels
                    a.mg_cq = magic_of(ceil_div(Ci, 8));
                    a.mg_hwp = magic_of(mpcnn::bm_geom(wp.TxP / 16, ly.k, Ci, wp.wn).hwp / 2);
                }
                a.mg_txp = magic_of(wp.TxP); a.mg_ci = magic_of(Ci); a.mg_k2 = magic_of(ly.k2);
                a.mg_ntx = magic_of(wp.ntx); a.mg_nty = magic_of(wp.nty); a.mg_d = magic_of(ly.dil); a.mg_d2 = magic_of(ly.dil2);
                dim3 grid((unsigned)wp.slabs, (unsigned)wp.gm, (unsigned)wp.gn);
                bool launched = false;
                if (wp.tr)
                    LAUNCH("wgrad_bm", li, wstep, flops, es * (n_in + n_out) + 4.0 * ly.p_len,
                           launched = mpcnn::launch_wgrad_tr(a, wp.TxP / 16, grid, wp.lds, st));
                else if (wp.bm)
                    LAUNCH("wgrad_bm", li, wstep, flops, es * (n_in + n_out) + 4.0 * ly.p_len,
                           launched = mpcnn::launch_wgrad_bm(a, wp.TxP / 16, grid, wp.lds, st));
                else
                    LAUNCH("wgrad_mfma", li, wstep, flops, es * (n_in + n_out) + 4.0 * ly.p_len,
                           launched = launch_wgrad_mfma<T>(a, wp.hl, grid, wp.lds, st));
                if (!launched)
                    return fail(MPCNN_EUNSUPPORTED, "layer %zu: no weight-gradient kernel instance for its plan", li);
            } else if (wp.l0m) {
                L0WgradArgs a{};
                a.in = A; a.dY = dY; a.partial = partial;
                a.B = B; a.Hi = Hi; a.Wi = Wi; a.Ho = Ho; a.Wo = Wo; a.Co = ly.cout;
                a.nty = ceil_div(Ho, mpcnn::kL0wTy); a.ntx = ceil_div(Wo, mpcnn::kL0wTx); a.tiles_total = wp.tiles_total;
                bool launched = false;
                const dim3 grid((unsigned)wp.chunks, (unsigned)ceil_div(ly.cout, 32));
                if (l0_wgrad_on_bm(ly, !kF32))
                    LAUNCH("wgrad_image_bm", li, wstep, flops, es * (n_in + n_out) + 4.0 * ly.p_len,
                           launched = launch_l0_wgrad_bm(a, ly.k, Ci, grid, st));
                else
                    LAUNCH("wgrad_image_mfma", li, wstep, flops, es * (n_in + n_out) + 4.0 * ly.p_len,
                           launched = launch_l0_wgrad<T>(a, ly.k, Ci, grid, st));
                if (!launched) return fail(MPCNN_EUNSUPPORTED, "layer 0: no image-layer weight-gradient kernel instance");
            } else {
                dim3 grid((unsigned)((ly.p_len + 255) / 256), (unsigned)wp.chunks);
                LAUNCH("wgrad_direct", li, wstep, flops, es * (n_in + n_out) + 4.0 * ly.p_len,
                       conv_wgrad_direct_kernel<T><<<grid, 256, 0, st>>>(A, dY, partial, B, Hi, Wi, Ci, Ho,
                                                                      Wo, ly.cout, ly.k, ly.k2, ly.dil, ly.dil2,
                                                                      wp.rows_per_chunk));
            }
            if (li == 0) break;  // the image needs no gradient
            const float* Wk = net->d_wread + ly.p_off;
            const double dbytes = es * (n_in * (below_tanh ? 2.0 : 1.0) + n_out) + 4.0 * ly.p_len;
            if (ly.dgrad_mfma && g.dgrad[li].ok) {
                const TilePlan& tp = g.dgrad[li];
                ConvArgs a{};
                a.in = dY; a.wpack = (const v4f*)(net->d_packs + ly.dgrad_pack_off);
                a.bias = nullptr; a.act = A; a.out = dA;
                a.B = B; a.Hi = Ho; a.Wi = Wo; a.Cr = ly.cout; a.CrPad = ly.dgrad_rpad;
                a.Ho = Hi; a.Wo = Wi; a.Co = Ci; a.CoPad = ly.dgrad_ct.pad;
                a.k = ly.k; a.d = ly.dil; a.origin = -(ly.k - 1); a.k2 = ly.k2; a.d2 = ly.dil2; a.origin2 = -(ly.k2 - 1);
                a.Ty = tp.Ty; a.Tx = tp.Tx; a.nty = tp.nty; a.ntx = tp.ntx;
                a.mode = below_tanh ? kDgradTanh : kDgradPlain; a.logistic = net->logistic;
                dim3 grid((unsigned)(B * ly.dil * ly.dil2 * tp.nty * tp.ntx), (unsigned)ly.dgrad_ct.split);
                parts_grid(&a, &grid, tp); a.wraw = Wk;
                if (net->halves) {
                    weights_of(&a, net, li);
                    a.out_peak = delta_words(g, ws, li - 1);
                    a.in_peak = delta_words(g, ws, li); a.in_words = g.delta_words[li]; a.in_margin = g.delta_margin[li];
                    if (two_part_dgrad(net, g, li)) a.wpack2 = (const v4f*)(net->d_packs + ly.dgrad_half_off);
                }
                bool launched = false;
                LAUNCH(kF32 ? "conv_dgrad_parts" : "conv_dgrad_bm", li, dstep, flops, dbytes, launched = launch_conv<T>(a, tp, grid, st));
                if (!launched)
                    return fail(MPCNN_EUNSUPPORTED, "layer %zu: no convolution kernel instance for its data-gradient plan", li);
            } else {
                long total = (long)B * Hi * Wi * Ci;
                if (below_tanh)
                    LAUNCH("conv_dgrad_direct", li, dstep, flops, dbytes,
                           (conv_dgrad_direct_kernel<true, T><<<grid_for(total), 256, 0, st>>>(
                               dY, Wk, A, dA, B, Hi, Wi, Ci, Ho, Wo, ly.cout, ly.k, ly.k2, ly.dil, ly.dil2, net->logistic)));
                else
                    LAUNCH("conv_dgrad_direct", li, dstep, flops, dbytes,
                           (conv_dgrad_direct_kernel<false, T><<<grid_for(total), 256, 0, st>>>(
                               dY, Wk, A, dA, B, Hi, Wi, Ci, Ho, Wo, ly.cout, ly.k, ly.k2, ly.dil, ly.dil2, net->logistic)));
            }
        }
        cur ^= 1;
    }
    // one launch adds the partial sums of every layer in a fixed order (Alg. 2)
    ReduceArgs ra{};
    ra.accumulate = g.accumulate ? 1 : 0;
    double rbytes = 0;
    if (g.small_net) {
        ReduceSeg& sg = ra.seg[ra.n_seg++];
        sg.partial = (const float*)(ws + g.small_partial_off);
        sg.out = net->d_grads;
        sg.plen = (long)net->n_params; sg.n = g.small_wgs; sg.tiled = 5; sg.items = (int)net->n_params;
        ra.total_blocks = ceil_div(sg.items, 16);
        rbytes = 4.0 * net->n_params * (g.small_wgs + 1.0);
    }
    for (size_t l = 0; l < L; ++l) {
        if (!g.partial_n[l] || ra.n_seg >= kMaxReduceSegs) continue;
        const Layer& ly = net->layers[l];
        ReduceSeg& sg = ra.seg[ra.n_seg++];
        sg.partial = (const float*)(ws + g.partial_off[l]);
        sg.out = net->d_grads + ly.p_off;
        sg.plen = (long)g.partial_len[l]; sg.n = g.partial_n[l];
        const WgradPlan& wp = g.wgrad[l];
        sg.tiled = wp.ok ? (wp.PM > 0 ? 4 : wp.bm ? 3 : 1) : 0;
        sg.items = !wp.ok ? (int)ly.p_len : (wp.PM > 0 ? wp.gm * wp.RT : wp.Mt) * wp.Nt * 256 + (wp.bm ? 0 : wp.Nt * 8);
        sg.RT = wp.RT; sg.ppg = wp.ppg; sg.tpg = wp.tpg; sg.ntg = wp.ntg; sg.Ci = ly.cin; sg.kk = ly.k * ly.k2;
        sg.Nt = wp.Nt; sg.rows_total = ly.k * ly.k2 * ly.cin; sg.Co = ly.cout;
        sg.block0 = ra.total_blocks;
        ra.total_blocks += (sg.items + 63) / 64;
        rbytes += 4.0 * ((double)sg.plen * sg.n + ly.p_len);
    }
    if (net->loss_shares > 0 && net->loss_out && ra.n_seg < kMaxReduceSegs) {
        ReduceSeg& sg = ra.seg[ra.n_seg++];
        sg.partial = (const float*)(ws + g.loss_partial_off);
        sg.out = (float*)net->loss_out;
        sg.plen = 0; sg.n = net->loss_shares; sg.tiled = 2; sg.items = 1;
        sg.block0 = ra.total_blocks;
        ra.total_blocks += 1;
    }
    LAUNCH("reduce_all", -1, 0, 0, rbytes, reduce_all_kernel<<<(unsigned)ra.total_blocks, 256, 0, st>>>(ra));
    HIP_TRY(hipGetLastError());
    return MPCNN_OK;
}

// One parameter vector between its device order W[u][v][c][o], b[o] and pinned host memory in host order
// W[o][c][u][v], b[o]; waits for it.
mpcnn_status order_params(const mpcnn_net* net, float* dev, bool to_host)
{
    mpcnn::ParamOrder a{};
    for (const Layer& ly : net->layers) {
        if (ly.kind == MPCNN_MP) continue;
        a.off[a.n_seg] = (long)ly.p_off; a.ci[a.n_seg] = ly.cin; a.co[a.n_seg] = ly.cout; a.kk[a.n_seg] = ly.k * ly.k2;
        ++a.n_seg;
    }
    a.off[a.n_seg] = (long)net->n_params;
    long longest = 1;
    for (int i = 0; i < a.n_seg; ++i) longest = std::max(longest, a.off[i + 1] - a.off[i]);
    mpcnn::params_order_kernel<<<dim3((unsigned)grid_for(longest, 256, 1024), (unsigned)a.n_seg), 256>>>(dev, net->h_stage, a, to_host ? 1 : 0);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(nullptr));
    return MPCNN_OK;
}

void lbfgs_free(mpcnn_net* net)
{
    (void)hipFree(net->d_lb_S); (void)hipFree(net->d_lb_Y);
    (void)hipFree(net->d_lb_theta_prev); (void)hipFree(net->d_lb_g_prev); (void)hipFree(net->d_lb_p);
    (void)hipFree(net->d_lb_part); (void)hipFree(net->d_lb_alpha);
    net->d_lb_S = net->d_lb_Y = net->d_lb_theta_prev = net->d_lb_g_prev = net->d_lb_p = nullptr;
    net->d_lb_part = net->d_lb_alpha = nullptr;
    net->lb_m = net->lb_head = net->lb_count = 0;
    net->lb_have_prev = false;
}

// Vectors up to this size are permuted here: read back by a copy, written by launches that carry the numbers as arguments.  Longer ones are
// permuted by the GPU, out of and into pinned memory.  The line lies where pinned memory is not worth its allocation, some 100 us per net.
// Microseconds, copy / GPU: read back alone 22 / 15 at 128 .. 2446 numbers, 12 / 15 at 4790, 18 / 17 at 22 K, 40 / 27 at 83 K (a copy of up to
// 16 KB takes the runtime twice as long as a larger one); behind a training step 104 / 105 at 128, 132 / 131 at 1292, 117 / 117 at
// 2446, 123 / 123 at 4790, 146 / 143 at 22 K.
constexpr size_t kSmallVector = 2048;

// One vector between host order W[o][c][u][v], b[o] and device order W[u][v][c][o], b[o], both on the host
void permute_params(const mpcnn_net* net, const float* src, float* dst, bool to_host)
{
    for (const Layer& ly : net->layers) {
        if (ly.kind == MPCNN_MP) continue;
        const int kk = ly.k * ly.k2, ci = ly.cin, co = ly.cout;
        const float* s = src + ly.p_off;
        float* d = dst + ly.p_off;
        for (int o = 0; o < co; ++o)
            for (int c = 0; c < ci; ++c)
                for (int t = 0; t < kk; ++t) {
                    const size_t host = ((size_t)o * ci + c) * kk + t, dev = ((size_t)t * ci + c) * co + o;
                    d[to_host ? host : dev] = s[to_host ? dev : host];
                }
        memcpy(d + (size_t)kk * ci * co, s + (size_t)kk * ci * co, sizeof(float) * co);
    }
}

mpcnn_status read_back(const mpcnn_net* net, const float* dev, float* host, size_t n)
{
    if (!net || !host) return fail(MPCNN_EINVAL, "null argument");
    if (n != net->n_params) return fail(MPCNN_EINVAL, "n = %zu, net has %zu parameters", n, net->n_params);
    if (!dev) return fail(MPCNN_EINVAL, "parameters were never set");
    HIP_TRY(hipSetDevice(net->device));
    HIP_TRY(hipDeviceSynchronize());
    if (n <= kSmallVector) {
        float tmp[kSmallVector];
        HIP_TRY(hipMemcpy(tmp, dev, sizeof(float) * n, hipMemcpyDeviceToHost));
        permute_params(net, tmp, host, true);
        return MPCNN_OK;
    }
    std::lock_guard<std::mutex> lock(net->stage_mu);
    const mpcnn_status rc = order_params(net, const_cast<float*>(dev), true);
    if (rc == MPCNN_OK) memcpy(host, net->h_stage, sizeof(float) * n);
    return rc;
}

// The plan for these sizes: from the net's cache, or made now and kept (same != 0: the
// same-size forward, H x W being the caller's image).  Null if the sizes do not fit the net.
std::shared_ptr<const Geom> geom_for(const mpcnn_net* net, int B, int H, int W, bool training, bool same)
{
    const GeomKey key{B, H, W, training ? 1 : 0, same ? 1 : 0, net->hint_pt, net->hint_mp};
    for (auto& kv : net->geoms)
        if (kv.first == key) return kv.second;
    auto g = std::make_shared<Geom>();
    if (same) {
        // the net runs on the image extended by P-1 mirrored rows / columns
        const int c = (net->patch - 1) / 2;
        if (!make_geom(net, B, H + net->patch - 1, W + net->patch - 1, false, g.get(), true)) return nullptr;
        g->pad_top = c; g->pad_left = c; g->src_h = H; g->src_w = W;
    } else if (!make_geom(net, B, H, W, training, g.get())) {
        return nullptr;
    }
    if (net->geoms.size() >= kGeomCacheSize) net->geoms.erase(net->geoms.begin());
    net->geoms.emplace_back(key, g);
    return g;
}

// Address of `scratch` on device `dev`, which must be the current device; looked up once per
// device and kept.
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mu;
mpcnn_status scratch_address(int dev, void** out)
{
    if (dev < 0 || dev >= kMaxDevices) return fail(MPCNN_EINVAL, "device %d: at most %d devices", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(MPCNN_EHIP, "hipGetSymbolAddress returned a null address");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return MPCNN_OK;
}

// What set_params allocates on its first call: parameters, gradients, weight packs (all of it, or free_params).
// d_params being there is what every other call takes for all of it.
void free_params(mpcnn_net* net)
{
    if (net->d_wread != net->d_params) (void)hipFree(net->d_wread);
    (void)hipFree(net->d_params);
    (void)hipFree(net->d_grads);
    (void)hipFree(net->d_packs);
    (void)hipFree(net->d_words);
    (void)hipHostFree(net->h_stage);
    net->d_params = net->d_grads = net->d_packs = net->d_wread = net->h_stage = nullptr;
    net->d_words = nullptr;
}
mpcnn_status alloc_params(mpcnn_net* net)
{
    const size_t bytes = sizeof(float) * net->n_params;
    HIP_TRY(hipGetDevice(&net->device));
    HIP_TRY(hipMalloc((void**)&net->d_params, bytes));
    HIP_TRY(hipMalloc((void**)&net->d_grads, bytes));
    if (net->n_params > kSmallVector) HIP_TRY(hipHostMalloc((void**)&net->h_stage, bytes, hipHostMallocDefault));
    HIP_TRY(hipMemset(net->d_grads, 0, bytes));
    if (net->pack_len) HIP_TRY(hipMalloc((void**)&net->d_packs, sizeof(float) * net->pack_len));
    if (net->halves) HIP_TRY(hipMalloc((void**)&net->d_words, sizeof(unsigned) * mpcnn::kPeakWords * net->layers.size()));
    if (net->bf16) HIP_TRY(hipMalloc((void**)&net->d_wread, bytes));
    else net->d_wread = net->d_params;
    const mpcnn_status rc = set_lds_attrs(net->bf16);
    if (rc != MPCNN_OK) return rc;
    void* unused = nullptr;   // (the static workspace's address on this device, for later calls)
    return scratch_address(net->device, &unused);
}

}  // namespace

extern "C" {

const char* mpcnn_last_error(void) { return g_err; }

mpcnn_status mpcnn_net_create(const mpcnn_layer_desc* layers, int n_layers, int in_channels,
                              int patch, mpcnn_dtype dtype, mpcnn_net** out)
{
    if (!layers || !out) return fail(MPCNN_EINVAL, "null argument");
    *out = nullptr;
    if (n_layers < 1 || n_layers > 48 || in_channels < 1 || patch < 1)
        return fail(MPCNN_EINVAL, "n_layers=%d in_channels=%d patch=%d", n_layers, in_channels, patch);
    if (dtype != MPCNN_F32 && dtype != MPCNN_BF16) return fail(MPCNN_EINVAL, "unknown dtype %d", (int)dtype);
    mpcnn_net* net = new (std::nothrow) mpcnn_net;
    if (!net) return fail(MPCNN_ENOMEM, "out of host memory");
    net->in_ch = in_channels; net->patch = patch; net->bf16 = dtype == MPCNN_BF16;
    int side = patch, side2 = patch, ch = in_channels, dil = 1, dil2 = 1;   // rows; columns
    bool seen_fc = false;
    size_t off = 0, pack = 0;
    mpcnn_status st = MPCNN_OK;
    for (int l = 0; l < n_layers && st == MPCNN_OK; ++l) {
        const mpcnn_layer_desc& d = layers[l];
        Layer ly{};
        ly.kind = d.kind; ly.cin = ch; ly.dil = dil; ly.dil2 = dil2;
        if (d.kind == MPCNN_C) {
            if (d.maps < 1 || d.k < 1) st = fail(MPCNN_EINVAL, "layer %d: C needs maps >= 1, k >= 1", l);
            else if (seen_fc) st = fail(MPCNN_ESHAPE, "layer %d: C after FC", l);
            else if (side - d.k + 1 < 1 || side2 - d.k + 1 < 1) st = fail(MPCNN_ESHAPE, "layer %d: %dx%d filter on a %dx%d map", l, d.k, d.k, side, side2);
            else { ly.k = ly.k2 = d.k; ly.cout = d.maps; ly.tanh_out = true; side -= d.k - 1; side2 -= d.k - 1; }
        } else if (d.kind == MPCNN_MP) {
            const int pc = d.k2 > 0 ? d.k2 : d.k;   // columns of the window
            if (d.k < 1 || d.k2 < 0) st = fail(MPCNN_EINVAL, "layer %d: MP needs k >= 1, k2 >= 0", l);
            else if (seen_fc) st = fail(MPCNN_ESHAPE, "layer %d: MP after FC", l);
            else if (side / d.k < 1 || side2 / pc < 1) st = fail(MPCNN_ESHAPE, "layer %d: %dx%d pooling on a %dx%d map", l, d.k, pc, side, side2);
            else if (d.k * pc > 255) st = fail(MPCNN_EUNSUPPORTED, "layer %d: pooling window too large for byte tap codes", l);
            else {
                ly.k = d.k; ly.k2 = pc; ly.cout = ch; ly.tanh_out = false;
                ly.drop = side % d.k; ly.drop2 = side2 % pc;
                side /= d.k; side2 /= pc; dil *= d.k; dil2 *= pc;
            }
        } else if (d.kind == MPCNN_FC) {
            if (d.maps < 1) st = fail(MPCNN_EINVAL, "layer %d: FC needs maps >= 1", l);
            else {
                ly.k = seen_fc ? 1 : side; ly.k2 = seen_fc ? 1 : side2;
                ly.cout = d.maps; ly.tanh_out = (l != n_layers - 1); side = side2 = 1; seen_fc = true;
            }
        } else st = fail(MPCNN_EINVAL, "layer %d: unknown kind %d", l, d.kind);
        if (st != MPCNN_OK) break;
        // rows and columns differ (a rectangular pool or anything behind one): the convolution kernel, wgrad_parts_kernel,
        // wgrad_mfma_kernel and the plain kernels take such a layer; the bf16 weight gradients, the image layer's kernels and
        // the max-filter kernels with several elements per thread do not
        ly.rect = ly.k2 != ly.k || (ly.dil2 != ly.dil && (ly.k > 1 || ly.k2 > 1));
        if (ly.kind != MPCNN_MP) {
            ly.p_off = off;
            ly.p_len = ((size_t)ly.k * ly.k2 * ly.cin + 1) * ly.cout;
            off += ly.p_len;
            // matrix cores take layers whose reduced channel count is a multiple of 4 and at
            // least 8, and that produce at least 8 channels; the rest run on the direct kernels
            const bool last = l == n_layers - 1;
            ly.class_fused = last && ly.k == 1 && ly.cin % 4 == 0 && ly.cin <= 256 &&
                             ly.cout >= 2 && ly.cout <= 4;
            ly.fwd_mfma = !last && ly.cin % 4 == 0 && ly.cin >= 8 && ly.cout >= 8;
            ly.dgrad_mfma = l > 0 && ly.cout % 4 == 0 && ly.cout >= 8 && ly.cin >= 8;
            ly.wgrad_mfma = !ly.class_fused;   // any shape: gradient rows are tiled in parameter order
            // (of a layer with 2 GiB of parameters there are no packs besides)
            const size_t pack_bound = (size_t)ly.k * ly.k2 * (ceil_div(std::max(ly.cin, ly.cout), 32) * 32 + 32) *
                                      (ceil_div(std::max(ly.cin, ly.cout), 32) * 32 + 32) * 4;
            if (pack_bound >= (1ull << 31)) ly.fwd_mfma = ly.dgrad_mfma = false;
            const int parts = net->bf16 ? 1 : 3;
            auto pack_floats = [&](int rpad, int pad) { return ((size_t)ly.k * ly.k2 * (rpad / 16) + mpcnn::parts_ahead(parts)) * parts * 2 * pad * 4; };
            if (ly.fwd_mfma) {
                ly.fwd_ct = chan_tiling(ly.cout);
                ly.fwd_rpad = ceil_div(ly.cin, 16) * 16;
                ly.fwd_pack_len = pack_floats(ly.fwd_rpad, ly.fwd_ct.pad);
                ly.fwd_pack_off = pack; pack += ly.fwd_pack_len;
            }
            if (ly.dgrad_mfma) {
                ly.dgrad_ct = chan_tiling(ly.cin);
                ly.dgrad_rpad = ceil_div(ly.cout, 16) * 16;
                ly.dgrad_pack_len = pack_floats(ly.dgrad_rpad, ly.dgrad_ct.pad);
                ly.dgrad_pack_off = pack; pack += ly.dgrad_pack_len;
            }
            // Two fp16 parts per number lose a last bit of one number in four; in a sum whose runs of leading products are added up
            // (kernels_conv_parts.hpp) that is less than what three parts' roundings come to from about 500 products on.
            auto half_floats = [&](int rpad, int pad) { return ((size_t)ly.k * ly.k2 * (rpad / 16) + mpcnn::parts_ahead(2)) * 2 * 2 * pad * 4; };
            ly.fwd_half = !net->bf16 && ly.fwd_mfma && l > 0 && mpcnn::half_filter(ly.k, ly.k2) && (long)ly.k * ly.k2 * ly.cin >= mpcnn::kHalfLeast;
            ly.dgrad_half = !net->bf16 && ly.dgrad_mfma && mpcnn::half_filter(ly.k, ly.k2) && (long)ly.k * ly.k2 * ly.cout >= mpcnn::kHalfLeast;
            if (ly.fwd_half) { ly.fwd_half_len = half_floats(ly.fwd_rpad, ly.fwd_ct.pad); ly.fwd_half_off = pack; pack += ly.fwd_half_len; }
            if (ly.dgrad_half) { ly.dgrad_half_len = half_floats(ly.dgrad_rpad, ly.dgrad_ct.pad); ly.dgrad_half_off = pack; pack += ly.dgrad_half_len; }
            net->halves = net->halves || ly.fwd_half || ly.dgrad_half;
        }
        ch = ly.cout;
        net->layers.push_back(ly);
    }
    if (st == MPCNN_OK && layers[n_layers - 1].kind != MPCNN_FC)
        st = fail(MPCNN_ESHAPE, "the last layer must be FC");
    if (st == MPCNN_OK && ch > mpcnn::kMaxClasses)
        st = fail(MPCNN_EUNSUPPORTED, "%d classes, at most %d are built", ch, mpcnn::kMaxClasses);
    if (st != MPCNN_OK) { delete net; return st; }
    net->n_cls = ch; net->n_params = off; net->pack_len = pack;
    *out = net;
    return MPCNN_OK;
}

void mpcnn_net_destroy(mpcnn_net* net)
{
    if (!net) return;
    if (net->d_params) {
        (void)hipSetDevice(net->device);
        (void)hipDeviceSynchronize();
        (void)hipFree(net->d_params0);
        (void)hipFree(net->d_scalar);
        lbfgs_free(net);
        free_params(net);
    }
    for (auto& p : net->pending) { (void)hipEventDestroy(p.e0); (void)hipEventDestroy(p.e1); }
    for (auto e : net->pool) (void)hipEventDestroy(e);
    delete net;
}

int mpcnn_net_patch(const mpcnn_net* net) { return net ? net->patch : 0; }
int mpcnn_net_classes(const mpcnn_net* net) { return net ? net->n_cls : 0; }
size_t mpcnn_param_count(const mpcnn_net* net) { return net ? net->n_params : 0; }

mpcnn_status mpcnn_layer_shape(const mpcnn_net* net, int H, int W, int layer, int* rows, int* cols,
                               int* channels, int* spacing)
{
    if (!net) return fail(MPCNN_EINVAL, "null net");
    if (layer < 0 || layer >= (int)net->layers.size()) return fail(MPCNN_EINVAL, "layer %d out of range", layer);
    const auto gp = (H >= net->patch && W >= net->patch) ? geom_for(net, 1, H, W, false, false) : nullptr;
    if (!gp) return fail(MPCNN_ESHAPE, "image %dx%d smaller than the %d patch", H, W, net->patch);
    const Geom& g = *gp;
    const Layer& ly = net->layers[layer];
    if (rows) *rows = g.rows[layer];
    if (cols) *cols = g.cols[layer];
    if (channels) *channels = ly.cout;
    if (spacing) *spacing = ly.kind == MPCNN_MP ? ly.dil * ly.k : ly.dil;
    return MPCNN_OK;
}

mpcnn_status mpcnn_plan_describe(const mpcnn_net* net, int B, int H, int W, int training, char* text_host,
                                 size_t cap)
{
    if (!net || !text_host || cap < 1) return fail(MPCNN_EINVAL, "null argument");
    text_host[0] = 0;
    if (B < 1 || H < net->patch || W < net->patch) return fail(MPCNN_ESHAPE, "image %dx%d smaller than the %d patch", H, W, net->patch);
    const auto gp = geom_for(net, B, H, W, training != 0, false);
    if (!gp) return fail(MPCNN_ESHAPE, "layer plan does not fit a %dx%d image", H, W);
    const Geom& g = *gp;
    size_t used = 0;
    auto put = [&](const char* fmt, ...) {
        if (used + 1 >= cap) return;
        va_list ap;
        va_start(ap, fmt);
        const int n = vsnprintf(text_host + used, cap - used, fmt, ap);
        va_end(ap);
        if (n > 0) used = std::min(cap - 1, used + (size_t)n);
    };
    auto parts = [&](bool half) {
        return net->bf16 ? "one part per number" : half ? "three parts per number or two of fp16" : "three parts per number";
    };
    auto conv = [&](const char* what, const TilePlan& tp, const ChanTiling& ct, bool half) {
        if (!tp.ok) { put("  %s: plain kernel\n", what); return; }
        put("  %s: bf16 MFMA, %s, %d channel tiles x %d groups, %d position tiles, waves %d x %d of %d x %d tiles, "
            "%d channels and %d filter rows per block, tile %d x %d of a residue class, %d x %d tiles, %d workgroups, %zu B LDS\n", what,
            parts(half), tp.in.WO * tp.in.MO, tp.in.WO * tp.in.MO == ct.OT ? ct.split : 1, tp.PT, tp.in.WO, tp.in.WP, tp.in.MO, tp.in.MP,
            tp.in.CB, tp.kr, tp.Ty, tp.Tx, tp.nty, tp.ntx, tp.wgs, tp.lds);
    };
    put("workspace %zu bytes\n", g.total);
    if (g.small_net) put("whole net in one launch: squares of %d x %d pixels, %d x %d of them, %d workgroups, %zu B LDS\n",
                         g.small.T, g.small.T, g.small.nty, g.small.ntx, g.small_wgs, g.small_lds);
    for (size_t l = 0; l < net->layers.size(); ++l) {
        const Layer& ly = net->layers[l];
        put("layer %zu: %s %d -> %d channels, k %d x %d, spacing %d x %d, map %d x %d\n", l,
            ly.kind == MPCNN_MP ? "MP" : (ly.kind == MPCNN_C ? "C" : "FC"), ly.cin, ly.cout, ly.k, ly.k2, ly.dil, ly.dil2,
            g.rows[l], g.cols[l]);
        if (ly.kind == MPCNN_MP || g.small_net) continue;
        if (ly.class_fused && g.head) { put("  class layer: at the end of the layer below\n"); continue; }
        if (ly.class_fused) { put("  fused class layer, %d workgroups\n", g.partial_n[l]); continue; }
        const bool img_sides = ly.dil == 1 && !ly.rect && (ly.k == 3 || ly.k == 5 || ly.k == 7);
        if (!g.fwd[l].ok && l == 0 && net->bf16 && img_sides && ly.cin <= 4 && ly.cout <= 64)
            put("  forward: image-layer kernel on the bf16 MFMA\n");
        else if (narrow_on_mfma(net, g, l)) {
            put("  forward: image-layer kernel on the fp32 MFMA");
            if (l == 0 && first_with_pool(net, g))
                put(", the pool behind it in the same launch, %d rows per wave", first_rows(ly.k, ly.cin, B, g.rows[1], g.cols[1], ceil_div(ly.cout, 32), true));
            put("\n");
        } else
            conv("forward", g.fwd[l], ly.fwd_ct, two_part_forward(net, g, l));
        if (!training) continue;
        if (l > 0) conv("data gradient", g.dgrad[l], ly.dgrad_ct, two_part_dgrad(net, g, l));
        const WgradPlan& w = g.wgrad[l];
        if (l == 0 && g.l0_fused) put("  weight gradient: fused with the routing of the pool above, %d workgroups\n", g.l0_blocks);
        else if (w.l0m) put("  weight gradient: image-layer kernel on the %s MFMA, %d tiles of 8 x 32, %d workgroups\n",
                            l0_wgrad_on_bm(ly, net->bf16) ? "bf16" : "fp32", w.tiles_total, w.chunks);
        else if (!w.ok) put("  weight gradient: plain kernel, %d chunks\n", w.chunks);
        else if (w.PM > 0)
            put("  weight gradient: bf16 MFMA, %s, %d x %d x %d waves (rows x columns x positions) of %d row tiles, %d x %d workgroup "
                "groups (%d planes, %d taps), tile %d x %d, %d tiles in %d slabs of %d, %zu B LDS\n", parts(w.two),
                w.wm, w.wn, w.wk, w.PM, w.gm, w.gn, w.ppg, w.tpg, w.R, 16 * w.nch, w.tiles_total, w.slabs, w.tiles_per_slab, w.lds);
        else
            put("  weight gradient: %s MFMA, %d x %d result tiles, waves %d x %d x %d (rows x columns x tile rows), %d row "
                "tiles per wave, %d x %d workgroup groups, tile 4 x %d (%d), %d tiles in %d slabs of %d, %zu B LDS\n",
                w.tr ? "bf16 (transposing reads)" : (w.bm ? "bf16" : "fp32"), w.Mt, w.Nt, w.wm, w.wn, w.wk, w.mw, w.gm, w.gn, w.Tx, w.TxP, w.tiles_total, w.slabs,
                w.tiles_per_slab, w.lds);
    }
    return MPCNN_OK;
}

mpcnn_status mpcnn_set_params(mpcnn_net* net, const float* params_host, size_t n)
{
    if (!net || !params_host) return fail(MPCNN_EINVAL, "null argument");
    if (n != net->n_params) return fail(MPCNN_EINVAL, "n = %zu, net has %zu parameters", n, net->n_params);
    if (!net->d_params) {
        const mpcnn_status rc = alloc_params(net);
        if (rc != MPCNN_OK) {   // nothing stays: the next call starts from here again
            free_params(net);
            (void)hipGetLastError();   // (a failed allocation is not the next launch's error)
            return rc;
        }
        const Layer& last = net->layers.back();
        if (last.class_fused) {
            const int kv = class_quads(last.cin, last.cout, net->bf16);
            const int occ = net->bf16 ? class_occupancy<mpcnn::bf16>(last.cout, kv, last.cin) : class_occupancy<float>(last.cout, kv, last.cin);
            if (occ > 0) net->class_max_blocks = std::min(kLossBlocks, kNumCU * occ);
        }
        net->geoms.clear();   // plans made before this point counted the class layer's shares differently
    }
    HIP_TRY(hipSetDevice(net->device));
    HIP_TRY(hipDeviceSynchronize());
    if (n <= kSmallVector) {
        float tmp[kSmallVector];
        permute_params(net, params_host, tmp, false);
        for (size_t at = 0; at < n; at += mpcnn::kCarried) {
            mpcnn::CarriedNumbers c;
            c.n = (int)std::min<size_t>(mpcnn::kCarried, n - at);
            memcpy(c.v, tmp + at, sizeof(float) * c.n);
            mpcnn::write_numbers_kernel<<<1, 256>>>(net->d_params + at, c);
        }
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipStreamSynchronize(nullptr));
    } else {
        std::lock_guard<std::mutex> lock(net->stage_mu);
        memcpy(net->h_stage, params_host, sizeof(float) * n);
        const mpcnn_status rc = order_params(net, net->d_params, false);
        if (rc != MPCNN_OK) return rc;
    }
    net->packs_stale = true; net->wread_stale = true;
    net->lb_head = net->lb_count = 0; net->lb_have_prev = false;   // a new starting point has no history
    return MPCNN_OK;
}

mpcnn_status mpcnn_set_loss(mpcnn_net* net, mpcnn_loss kind)
{
    if (!net) return fail(MPCNN_EINVAL, "null net");
    if (kind != MPCNN_LOSS_MCCE && kind != MPCNN_LOSS_MSE) return fail(MPCNN_EINVAL, "unknown loss %d", (int)kind);
    net->loss_kind = kind;
    return MPCNN_OK;
}

mpcnn_status mpcnn_set_activation(mpcnn_net* net, mpcnn_activation kind)
{
    if (!net) return fail(MPCNN_EINVAL, "null net");
    if (kind != MPCNN_TANH && kind != MPCNN_LOGISTIC) return fail(MPCNN_EINVAL, "unknown activation %d", (int)kind);
    net->logistic = kind == MPCNN_LOGISTIC ? 1 : 0;
    return MPCNN_OK;
}

mpcnn_status mpcnn_set_conv_tiling(mpcnn_net* net, int position_tiles, int tiles_per_wave)
{
    if (!net) return fail(MPCNN_EINVAL, "null net");
    const bool pt_ok = position_tiles == 0 || position_tiles == 2 || position_tiles == 4 || position_tiles == 8 ||
                       position_tiles == 16;
    const bool mp_ok = tiles_per_wave == 0 || tiles_per_wave == 1 || tiles_per_wave == 2 || tiles_per_wave == 4;
    if (!pt_ok || !mp_ok)
        return fail(MPCNN_EINVAL, "conv tiling (%d, %d): position tiles 0/2/4/8/16, tiles per wave 0/1/2/4", position_tiles, tiles_per_wave);
    net->hint_pt = position_tiles; net->hint_mp = tiles_per_wave;
    net->geoms.clear();
    return MPCNN_OK;
}

mpcnn_status mpcnn_class_balance_weights(const mpcnn_net* net, const int32_t* labels_dev, int B, int H,
                                         int W, float* pixw_dev, void* counts_dev, void* hip_stream)
{
    if (!net || !labels_dev || !pixw_dev || !counts_dev) return fail(MPCNN_EINVAL, "null argument");
    if (B < 1) return fail(MPCNN_EINVAL, "B = %d", B);
    if (H < net->patch || W < net->patch)
        return fail(MPCNN_ESHAPE, "image %dx%d smaller than the %dx%d patch", H, W, net->patch, net->patch);
    hipStream_t st = (hipStream_t)hip_stream;
    const int Ho = H - net->patch + 1, Wo = W - net->patch + 1, ctr = (net->patch - 1) / 2;
    unsigned* counts = (unsigned*)counts_dev;
    mpcnn::clear_counts_kernel<<<1, 64, 0, st>>>(counts);
    mpcnn::label_count_kernel<<<grid_for((long)B * Ho * Wo, 256, 1024), 256, 0, st>>>(labels_dev, counts, B, H, W, Ho,
                                                                                    Wo, ctr, net->n_cls);
    mpcnn::balance_fill_kernel<<<grid_for((long)B * H * W), 256, 0, st>>>(labels_dev, counts, pixw_dev, B, H, W, Ho,
                                                                         Wo, ctr, net->n_cls);
    HIP_TRY(hipGetLastError());
    return MPCNN_OK;
}

mpcnn_status mpcnn_get_params(const mpcnn_net* net, float* params_host, size_t n)
{
    return read_back(net, net ? net->d_params : nullptr, params_host, n);
}

mpcnn_status mpcnn_get_grads(const mpcnn_net* net, float* grads_host, size_t n)
{
    return read_back(net, net ? net->d_grads : nullptr, grads_host, n);
}

size_t mpcnn_workspace_bytes(const mpcnn_net* net, int B, int H, int W, int training)
{
    if (!net || B < 1 || H < net->patch || W < net->patch) return 0;
    const auto g = geom_for(net, B, H, W, training != 0, false);
    return g ? g->total : 0;
}

static mpcnn_status check_call(mpcnn_net* net, const float* image, int B, int H, int W, void* ws,
                               size_t ws_bytes, bool training, std::shared_ptr<const Geom>* g)
{
    if (!net || !image || !ws) return fail(MPCNN_EINVAL, "null argument");
    if (!net->d_params) return fail(MPCNN_EINVAL, "parameters were never set");
    if (B < 1) return fail(MPCNN_EINVAL, "B = %d", B);
    if (H < net->patch || W < net->patch)
        return fail(MPCNN_ESHAPE, "image %dx%d smaller than the %dx%d patch", H, W, net->patch, net->patch);
    *g = geom_for(net, B, H, W, training, false);
    if (!*g) return fail(MPCNN_ESHAPE, "layer plan does not fit a %dx%d image", H, W);
    if (ws_bytes < (*g)->total) return fail(MPCNN_EWORKSPACE, "workspace %zu bytes, need %zu", ws_bytes, (*g)->total);
    if (((uintptr_t)ws & 255u) != 0) return fail(MPCNN_EINVAL, "workspace must be 256-byte aligned");
    if (((uintptr_t)image & 15u) != 0) return fail(MPCNN_EINVAL, "image must be 16-byte aligned");
    return MPCNN_OK;
}

static mpcnn_status forward_with(mpcnn_net* net, const std::shared_ptr<const Geom>& g, const float* image_dev,
                                 float* probs_dev, void* ws_dev, hipStream_t stream)
{
    mpcnn_status st = net->bf16 ? run_forward<mpcnn::bf16>(net, *g, image_dev, (char*)ws_dev, nullptr, nullptr, probs_dev,
                                                           nullptr, nullptr, stream)
                                : run_forward<float>(net, *g, image_dev, (char*)ws_dev, nullptr, nullptr, probs_dev, nullptr,
                                                     nullptr, stream);
    net->last = g; net->last_ws = ws_dev;
    return st;
}

mpcnn_status mpcnn_seg_forward(mpcnn_net* net, const float* image_dev, int B, int H, int W,
                               float* probs_dev, void* ws_dev, size_t ws_bytes, void* hip_stream)
{
    std::shared_ptr<const Geom> g;
    mpcnn_status st = check_call(net, image_dev, B, H, W, ws_dev, ws_bytes, false, &g);
    if (st != MPCNN_OK) return st;
    if (!probs_dev) return fail(MPCNN_EINVAL, "null probs_dev");
    return forward_with(net, g, image_dev, probs_dev, ws_dev, (hipStream_t)hip_stream);
}

mpcnn_status mpcnn_seg_forward_static(mpcnn_net* net, const float* image_dev, int B, int H, int W,
                                      float* probs_dev, void* hip_stream)
{
    if (!net || !image_dev || !probs_dev) return fail(MPCNN_EINVAL, "null argument");
    if (!net->d_params) return fail(MPCNN_EINVAL, "parameters were never set");
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != net->device)
        return fail(MPCNN_EINVAL, "device %d is current, the net lives on device %d", dev, net->device);
    void* ws = nullptr;
    mpcnn_status st = scratch_address(dev, &ws);
    if (st != MPCNN_OK) return st;
    std::shared_ptr<const Geom> g;
    st = check_call(net, image_dev, B, H, W, ws, (size_t)MPCNN_STATIC_WORKSPACE_BYTES, false, &g);
    if (st == MPCNN_EWORKSPACE)
        return fail(MPCNN_EWORKSPACE, "a %d x %dx%d batch needs %zu bytes of workspace, the static one holds %zu",
                    B, H, W, g->total, (size_t)MPCNN_STATIC_WORKSPACE_BYTES);
    if (st != MPCNN_OK) return st;
    // (the per-launch timing hooks create events: not in a call that must not allocate)
    const bool prof = net->prof_on;
    net->prof_on = false;
    st = forward_with(net, g, image_dev, probs_dev, ws, (hipStream_t)hip_stream);
    net->prof_on = prof;
    return st;
}

size_t mpcnn_workspace_bytes_same(const mpcnn_net* net, int B, int H, int W)
{
    if (!net || B < 1 || H < 1 || W < 1) return 0;
    const auto g = geom_for(net, B, H, W, false, true);
    return g ? g->total : 0;
}

mpcnn_status mpcnn_seg_forward_same(mpcnn_net* net, const float* image_dev, int B, int H, int W,
                                    float* probs_dev, void* ws_dev, size_t ws_bytes, void* hip_stream)
{
    if (!net || !image_dev || !ws_dev || !probs_dev) return fail(MPCNN_EINVAL, "null argument");
    if (!net->d_params) return fail(MPCNN_EINVAL, "parameters were never set");
    if (B < 1) return fail(MPCNN_EINVAL, "B = %d", B);
    const int widest = net->patch - 1 - (net->patch - 1) / 2;
    if (H < 1 || W < 1 || H < widest || W < widest)
        return fail(MPCNN_ESHAPE, "image %dx%d smaller than the %d-pixel mirrored border", H, W, widest);
    const auto g = geom_for(net, B, H, W, false, true);
    if (!g) return fail(MPCNN_ESHAPE, "layer plan does not fit a %dx%d image", H, W);
    if (ws_bytes < g->total) return fail(MPCNN_EWORKSPACE, "workspace %zu bytes, need %zu", ws_bytes, g->total);
    if (((uintptr_t)ws_dev & 255u) != 0) return fail(MPCNN_EINVAL, "workspace must be 256-byte aligned");
    return forward_with(net, g, image_dev, probs_dev, ws_dev, (hipStream_t)hip_stream);
}

mpcnn_status mpcnn_seg_backward(mpcnn_net* net, const float* image_dev, const int32_t* labels_dev,
                                const float* pixw_dev, int B, int H, int W, float* probs_dev,
                                double* loss_dev, void* ws_dev, size_t ws_bytes, void* hip_stream)
{
    std::shared_ptr<const Geom> gp;
    mpcnn_status st = check_call(net, image_dev, B, H, W, ws_dev, ws_bytes, true, &gp);
    if (st != MPCNN_OK) return st;
    if (!labels_dev) return fail(MPCNN_EINVAL, "null labels_dev");
    const Geom& g = *gp;
    hipStream_t stream = (hipStream_t)hip_stream;
    char* ws = (char*)ws_dev;
    void* dZ = ws + g.delta_off[0];
    st = net->bf16 ? run_forward<mpcnn::bf16>(net, g, image_dev, ws, labels_dev, pixw_dev, probs_dev, dZ, loss_dev, stream)
                   : run_forward<float>(net, g, image_dev, ws, labels_dev, pixw_dev, probs_dev, dZ, loss_dev, stream);
    net->last = gp; net->last_ws = ws_dev;
    if (st != MPCNN_OK) return st;
    return net->bf16 ? run_backward<mpcnn::bf16>(net, g, image_dev, ws, stream)
                     : run_backward<float>(net, g, image_dev, ws, stream);
}

// geometry of one band of output rows [row0, row0 + rows) of a B x H x W image
static bool make_geom_band(const mpcnn_net* net, int B, int H, int W, int row0, int rows, Geom* g)
{
    if (!make_geom(net, B, rows + net->patch - 1, W, true, g, true, true)) return false;
    g->pad_top = -row0; g->pad_left = 0; g->src_h = H; g->src_w = W;   // the band starts row0 rows down the image
    g->label_h = H; g->probs_rows = H - net->patch + 1;
    g->accumulate = row0 > 0;
    return true;
}

size_t mpcnn_workspace_bytes_banded(const mpcnn_net* net, int B, int W, int band_rows)
{
    Geom g;
    if (!net || band_rows < 1 || B < 1 || W < net->patch) return 0;
    if (!make_geom_band(net, B, band_rows + net->patch - 1, W, 0, band_rows, &g)) return 0;
    return g.total;
}

mpcnn_status mpcnn_seg_backward_banded(mpcnn_net* net, const float* image_dev, const int32_t* labels_dev,
                                       const float* pixw_dev, int B, int H, int W, int band_rows,
                                       float* probs_dev, double* loss_dev, void* ws_dev, size_t ws_bytes,
                                       void* hip_stream)
{
    if (!net || !image_dev || !ws_dev || !labels_dev) return fail(MPCNN_EINVAL, "null argument");
    if (!net->d_params) return fail(MPCNN_EINVAL, "parameters were never set");
    if (B < 1 || band_rows < 1) return fail(MPCNN_EINVAL, "B = %d, band_rows = %d", B, band_rows);
    if (H < net->patch || W < net->patch)
        return fail(MPCNN_ESHAPE, "image %dx%d smaller than the %dx%d patch", H, W, net->patch, net->patch);
    if (((uintptr_t)ws_dev & 255u) != 0) return fail(MPCNN_EINVAL, "workspace must be 256-byte aligned");
    if (((uintptr_t)image_dev & 15u) != 0) return fail(MPCNN_EINVAL, "image must be 16-byte aligned");
    const int Ho = H - net->patch + 1, Wo = W - net->patch + 1;
    hipStream_t stream = (hipStream_t)hip_stream;
    char* ws = (char*)ws_dev;
    for (int row0 = 0; row0 < Ho; row0 += band_rows) {
        const int rows = std::min(band_rows, Ho - row0);
        auto gp = std::make_shared<Geom>();
        if (!make_geom_band(net, B, H, W, row0, rows, gp.get()))
            return fail(MPCNN_ESHAPE, "layer plan does not fit a band of %d rows", rows);
        const Geom& g = *gp;
        if (ws_bytes < g.total) return fail(MPCNN_EWORKSPACE, "workspace %zu bytes, need %zu", ws_bytes, g.total);
        // the band's labels, weights and probabilities start row0 rows down their arrays
        const int32_t* lab = labels_dev + (size_t)row0 * W;
        const float* pw = pixw_dev ? pixw_dev + (size_t)row0 * W : nullptr;
        float* pr = probs_dev ? probs_dev + (size_t)row0 * Wo : nullptr;
        void* dZ = ws + g.delta_off[0];
        mpcnn_status st =
            net->bf16 ? run_forward<mpcnn::bf16>(net, g, image_dev, ws, lab, pw, pr, dZ, loss_dev, stream)
                      : run_forward<float>(net, g, image_dev, ws, lab, pw, pr, dZ, loss_dev, stream);
        net->last = gp; net->last_ws = ws_dev;
        if (st != MPCNN_OK) return st;
        st = net->bf16 ? run_backward<mpcnn::bf16>(net, g, image_dev, ws, stream)
                       : run_backward<float>(net, g, image_dev, ws, stream);
        if (st != MPCNN_OK) return st;
    }
    return MPCNN_OK;
}

// forward + summed loss, nothing kept (the workspace is a forward-only one)
static mpcnn_status loss_only(mpcnn_net* net, const Geom& g, const float* image_dev, const int32_t* labels_dev,
                              const float* pixw_dev, double* loss_dev, char* ws, hipStream_t st)
{
    mpcnn_status rc = net->bf16 ? run_forward<mpcnn::bf16>(net, g, image_dev, ws, labels_dev, pixw_dev, nullptr,
                                                           nullptr, loss_dev, st)
                                : run_forward<float>(net, g, image_dev, ws, labels_dev, pixw_dev, nullptr, nullptr,
                                                     loss_dev, st);
    if (rc != MPCNN_OK) return rc;
    if (net->loss_shares < 1) return fail(MPCNN_EINVAL, "no loss was computed");
    mpcnn::ReduceArgs ra{};
    mpcnn::ReduceSeg& sg = ra.seg[ra.n_seg++];
    sg.partial = (const float*)(ws + g.loss_partial_off);
    sg.out = (float*)loss_dev;
    sg.n = net->loss_shares; sg.tiled = 2; sg.items = 1; sg.block0 = 0;
    ra.total_blocks = 1;
    LAUNCH("reduce_all", -1, 0, 0, 8.0 * sg.n, mpcnn::reduce_all_kernel<<<1, 256, 0, st>>>(ra));
    HIP_TRY(hipGetLastError());
    return MPCNN_OK;
}

mpcnn_status mpcnn_seg_loss(mpcnn_net* net, const float* image_dev, const int32_t* labels_dev,
                            const float* pixw_dev, int B, int H, int W, double* loss_dev,
                            void* ws_dev, size_t ws_bytes, void* hip_stream)
{
    std::shared_ptr<const Geom> gp;
    mpcnn_status st = check_call(net, image_dev, B, H, W, ws_dev, ws_bytes, false, &gp);
    if (st != MPCNN_OK) return st;
    if (!labels_dev || !loss_dev) return fail(MPCNN_EINVAL, "null argument");
    return loss_only(net, *gp, image_dev, labels_dev, pixw_dev, loss_dev, (char*)ws_dev, (hipStream_t)hip_stream);
}

mpcnn_status mpcnn_armijo_step(mpcnn_net* net, const float* image_dev, const int32_t* labels_dev,
                               const float* pixw_dev, int B, int H, int W, double f0, float alpha0,
                               float grad_scale, float c, float beta, int max_trials, void* ws_dev,
                               size_t ws_bytes, void* hip_stream, float* alpha_host, double* loss_host,
                               int* trials_host)
{
    std::shared_ptr<const Geom> gp;
    mpcnn_status rc = check_call(net, image_dev, B, H, W, ws_dev, ws_bytes, false, &gp);
    if (rc != MPCNN_OK) return rc;
    const Geom& g = *gp;
    if (!labels_dev) return fail(MPCNN_EINVAL, "null labels_dev");
    if (!(alpha0 > 0.f) || !(beta > 0.f && beta < 1.f) || !(c >= 0.f && c < 1.f) || max_trials < 1)
        return fail(MPCNN_EINVAL, "alpha0 = %g, beta = %g, c = %g, max_trials = %d", alpha0, beta, c, max_trials);
    hipStream_t st = (hipStream_t)hip_stream;
    const long n = (long)net->n_params;
    if (!net->d_params0) HIP_TRY(hipMalloc((void**)&net->d_params0, sizeof(float) * n));
    if (!net->d_scalar) HIP_TRY(hipMalloc((void**)&net->d_scalar, 8 * sizeof(double)));
    HIP_TRY(hipMemcpyAsync(net->d_params0, net->d_params, sizeof(float) * n, hipMemcpyDeviceToDevice, st));
    mpcnn::sqnorm_kernel<<<1, 1024, 0, st>>>(net->d_grads, n, net->d_scalar);
    double both[2];           // |g|^2, and the loss of a trial: read back together, so that the host waits once per trial
    float alpha = alpha0;
    double f = f0;
    int trial = 0;
    bool ok = false;
    while (trial < max_trials) {
        ++trial;
        mpcnn::step_from_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(net->d_params, net->d_params0,
                                                                              net->d_grads, alpha * grad_scale, n);
        net->packs_stale = true; net->wread_stale = true;
        rc = loss_only(net, g, image_dev, labels_dev, pixw_dev, net->d_scalar + 1, (char*)ws_dev, st);
        if (rc != MPCNN_OK) break;
        HIP_TRY(hipMemcpyAsync(both, net->d_scalar, sizeof both, hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        f = both[1];
        if (f <= f0 - (double)c * (double)alpha * (double)grad_scale * both[0]) { ok = true; break; }
        alpha *= beta;
    }
    if (!ok) {   // also after an error: the parameters the call started from
        HIP_TRY(hipMemcpyAsync(net->d_params, net->d_params0, sizeof(float) * n, hipMemcpyDeviceToDevice, st));
        HIP_TRY(hipStreamSynchronize(st));
        net->packs_stale = true; net->wread_stale = true;
        alpha = 0.f; f = f0;
    }
    if (alpha_host) *alpha_host = alpha;
    if (loss_host) *loss_host = f;
    if (trials_host) *trials_host = trial;
    return rc;
}

mpcnn_status mpcnn_lbfgs_reset(mpcnn_net* net)
{
    if (!net) return fail(MPCNN_EINVAL, "null net");
    net->lb_head = net->lb_count = 0;
    net->lb_have_prev = false;
    return MPCNN_OK;
}

mpcnn_status mpcnn_lbfgs_step(mpcnn_net* net, const float* image_dev, const int32_t* labels_dev,
                              const float* pixw_dev, int B, int H, int W, double f0, int history,
                              float alpha0, float c, float beta, int max_trials, void* ws_dev,
                              size_t ws_bytes, void* hip_stream, float* alpha_host, double* loss_host,
                              int* trials_host, int* pairs_host)
{
    using namespace mpcnn;
    std::shared_ptr<const Geom> gp;
    mpcnn_status rc = check_call(net, image_dev, B, H, W, ws_dev, ws_bytes, false, &gp);
    if (rc != MPCNN_OK) return rc;
    const Geom& g = *gp;
    if (!labels_dev) return fail(MPCNN_EINVAL, "null labels_dev");
    if (!(alpha0 > 0.f) || !(beta > 0.f && beta < 1.f) || !(c >= 0.f && c < 1.f) || max_trials < 1 ||
        history < 1 || history > 64)
        return fail(MPCNN_EINVAL, "alpha0 = %g, beta = %g, c = %g, max_trials = %d, history = %d", alpha0, beta,
                    c, max_trials, history);
    hipStream_t st = (hipStream_t)hip_stream;
    const long n = (long)net->n_params;
    const size_t vec = sizeof(float) * n;
    if (net->lb_m != history) {   // first call, or another history length: start afresh
        lbfgs_free(net);
        HIP_TRY(hipMalloc((void**)&net->d_lb_S, vec * (history + 1)));
        HIP_TRY(hipMalloc((void**)&net->d_lb_Y, vec * (history + 1)));
        HIP_TRY(hipMalloc((void**)&net->d_lb_theta_prev, vec));
        HIP_TRY(hipMalloc((void**)&net->d_lb_g_prev, vec));
        HIP_TRY(hipMalloc((void**)&net->d_lb_p, vec));
        HIP_TRY(hipMalloc((void**)&net->d_lb_part, sizeof(double) * 5 * kLbBlocks));
        HIP_TRY(hipMalloc((void**)&net->d_lb_alpha, sizeof(double) * (history + 1)));
        net->lb_m = history;
        net->lb_sy.assign(history + 1, 0.0); net->lb_yy.assign(history + 1, 0.0);
    }
    if (!net->d_params0) HIP_TRY(hipMalloc((void**)&net->d_params0, vec));
    if (!net->d_scalar) HIP_TRY(hipMalloc((void**)&net->d_scalar, 8 * sizeof(double)));
    const int slots = net->lb_m + 1;
    double* part[2] = {net->d_lb_part, net->d_lb_part + kLbBlocks};

    // 1. the pair (theta - theta_prev, g - g_prev), kept if its curvature s.y is positive
    if (net->lb_have_prev) {
        const int slot = (net->lb_head + net->lb_count) % slots;
        lb_pair_kernel<<<kLbBlocks, 256, 0, st>>>(net->d_params, net->d_lb_theta_prev, net->d_grads, net->d_lb_g_prev,
                                                  net->d_lb_S + (size_t)slot * n, net->d_lb_Y + (size_t)slot * n,
                                                  net->d_lb_part + 2 * kLbBlocks, n);
        lb_sum_kernel<<<1, 256, 0, st>>>(net->d_lb_part + 2 * kLbBlocks, 3, net->d_scalar + 2);
        double r[3];
        HIP_TRY(hipMemcpyAsync(r, net->d_scalar + 2, sizeof(r), hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        if (r[0] > 1e-10 * std::sqrt(r[2] * r[1])) {
            net->lb_sy[slot] = r[0]; net->lb_yy[slot] = r[1];
            if (net->lb_count < net->lb_m) ++net->lb_count;
            else net->lb_head = (net->lb_head + 1) % slots;   // the oldest pair's slot becomes the free one
        }
    }

    // 2. p = -H g by the two-loop recursion, and the slope g.p
    double slope = 0.0;
    for (int attempt = 0; attempt < 2; ++attempt) {
        const int M = net->lb_count;
        auto slot_of = [&](int i) { return (net->lb_head + i) % slots; };   // i = 0 oldest
        LbArgs a{};
        a.q = net->d_lb_p; a.n = n; a.alpha = net->d_lb_alpha;
        int flip = 0;
        a.mode = 0; a.src = net->d_grads; a.part_out = part[flip];
        if (M == 0) { a.scale = -1.0; a.u = net->d_grads; }
        else { a.scale = 1.0; a.u = net->d_lb_S + (size_t)slot_of(M - 1) * n; }
        lb_update_kernel<<<kLbBlocks, 256, 0, st>>>(a);
        for (int i = M - 1; i >= 0; --i) {        // newest to oldest
            const int sl = slot_of(i);
            a.mode = 1; a.idx = i; a.rho = 1.0 / net->lb_sy[sl];
            a.v = net->d_lb_Y + (size_t)sl * n;
            a.part_in = part[flip]; flip ^= 1; a.part_out = part[flip];
            if (i > 0) { a.scale = 1.0; a.u = net->d_lb_S + (size_t)slot_of(i - 1) * n; }
            else {                                  // the turn: r = H_0 q
                const int nw = slot_of(M - 1);
                a.scale = net->lb_sy[nw] / net->lb_yy[nw];
                a.u = net->d_lb_Y + (size_t)slot_of(0) * n;
            }
            lb_update_kernel<<<kLbBlocks, 256, 0, st>>>(a);
        }
        for (int i = 0; i < M; ++i) {              // oldest to newest
            const int sl = slot_of(i);
            a.mode = 2; a.idx = i; a.rho = 1.0 / net->lb_sy[sl];
            a.v = net->d_lb_S + (size_t)sl * n;
            a.part_in = part[flip]; flip ^= 1; a.part_out = part[flip];
            if (i + 1 < M) { a.scale = 1.0; a.u = net->d_lb_Y + (size_t)slot_of(i + 1) * n; }
            else { a.scale = -1.0; a.u = net->d_grads; }
            lb_update_kernel<<<kLbBlocks, 256, 0, st>>>(a);
        }
        lb_sum_kernel<<<1, 256, 0, st>>>(part[flip], 1, net->d_scalar);
        HIP_TRY(hipMemcpyAsync(&slope, net->d_scalar, sizeof(double), hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        if (slope < 0.0 || M == 0) break;
        net->lb_count = 0;                         // not a descent direction: forget the pairs
    }
    const int used = net->lb_count;

    // 3. back-tracking along p
    HIP_TRY(hipMemcpyAsync(net->d_params0, net->d_params, vec, hipMemcpyDeviceToDevice, st));
    float alpha = alpha0;
    double f = f0;
    int trial = 0;
    bool ok = false;
    while (slope < 0.0 && trial < max_trials) {
        ++trial;
        step_from_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(net->d_params, net->d_params0, net->d_lb_p,
                                                                      -alpha, n);
        net->packs_stale = true; net->wread_stale = true;
        rc = loss_only(net, g, image_dev, labels_dev, pixw_dev, net->d_scalar + 1, (char*)ws_dev, st);
        if (rc != MPCNN_OK) break;
        HIP_TRY(hipMemcpyAsync(&f, net->d_scalar + 1, sizeof(double), hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        if (f <= f0 + (double)c * (double)alpha * slope) { ok = true; break; }
        alpha *= beta;
    }
    if (ok) {      // this iterate becomes the previous one
        std::swap(net->d_params0, net->d_lb_theta_prev);
        HIP_TRY(hipMemcpyAsync(net->d_lb_g_prev, net->d_grads, vec, hipMemcpyDeviceToDevice, st));
        HIP_TRY(hipStreamSynchronize(st));
        net->lb_have_prev = true;
    } else {       // also after an error: the parameters the call started from, no history
        HIP_TRY(hipMemcpyAsync(net->d_params, net->d_params0, vec, hipMemcpyDeviceToDevice, st));
        HIP_TRY(hipStreamSynchronize(st));
        net->packs_stale = true; net->wread_stale = true;
        net->lb_count = 0; net->lb_head = 0; net->lb_have_prev = false;
        alpha = 0.f; f = f0;
    }
    if (alpha_host) *alpha_host = alpha;
    if (loss_host) *loss_host = f;
    if (trials_host) *trials_host = trial;
    if (pairs_host) *pairs_host = used;
    return rc;
}

mpcnn_status mpcnn_sgd_step(mpcnn_net* net, float lr, float grad_scale, void* hip_stream)
{
    if (!net) return fail(MPCNN_EINVAL, "null net");
    if (!net->d_params) return fail(MPCNN_EINVAL, "parameters were never set");
    long n = (long)net->n_params;
    hipStream_t st = (hipStream_t)hip_stream;
    LAUNCH("sgd", -1, 8, 2.0 * n, 12.0 * n,
           mpcnn::sgd_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(net->d_params, net->d_grads,
                                                                          lr * grad_scale, n));
    HIP_TRY(hipGetLastError());
    net->packs_stale = true; net->wread_stale = true;
    return MPCNN_OK;
}

mpcnn_status mpcnn_get_activation(const mpcnn_net* net, int layer, float* host, size_t n)
{
    if (!net || !host) return fail(MPCNN_EINVAL, "null argument");
    if (!net->last_ws || !net->last || !net->last->training) return fail(MPCNN_EINVAL, "no backward call has been made");
    if (layer < 0 || layer >= (int)net->layers.size()) return fail(MPCNN_EINVAL, "layer %d out of range", layer);
    const Geom& g = *net->last;
    size_t elems = (size_t)g.B * g.rows[layer] * g.cols[layer] * net->layers[layer].cout;
    if (n != elems) return fail(MPCNN_EINVAL, "n = %zu, layer holds %zu elements", n, elems);
    HIP_TRY(hipSetDevice(net->device));
    HIP_TRY(hipDeviceSynchronize());
    const char* src = (const char*)net->last_ws + g.act_off[layer];
    if (!net->bf16) {
        HIP_TRY(hipMemcpy(host, src, sizeof(float) * elems, hipMemcpyDeviceToHost));
    } else {
        std::vector<uint16_t> tmp(elems);
        HIP_TRY(hipMemcpy(tmp.data(), src, sizeof(uint16_t) * elems, hipMemcpyDeviceToHost));
        for (size_t i = 0; i < elems; ++i) {
            const uint32_t bits = (uint32_t)tmp[i] << 16;   // bf16 = the upper half of an fp32
            memcpy(host + i, &bits, sizeof(float));
        }
    }
    return MPCNN_OK;
}

mpcnn_status mpcnn_get_argmax(const mpcnn_net* net, int layer, uint8_t* host, size_t n)
{
    if (!net || !host) return fail(MPCNN_EINVAL, "null argument");
    if (!net->last_ws || !net->last || !net->last->training) return fail(MPCNN_EINVAL, "no backward call has been made");
    if (layer < 0 || layer >= (int)net->layers.size() || net->layers[layer].kind != MPCNN_MP)
        return fail(MPCNN_EINVAL, "layer %d is not an MP layer", layer);
    const Geom& g = *net->last;
    size_t elems = (size_t)g.B * g.rows[layer] * g.cols[layer] * net->layers[layer].cout;
    if (n != elems) return fail(MPCNN_EINVAL, "n = %zu, layer holds %zu elements", n, elems);
    HIP_TRY(hipSetDevice(net->device));
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipMemcpy(host, (char*)net->last_ws + g.code_off[layer], elems, hipMemcpyDeviceToHost));
    return MPCNN_OK;
}

mpcnn_status mpcnn_profile_enable(mpcnn_net* net, int on)
{
    if (!net) return fail(MPCNN_EINVAL, "null net");
    net->prof_on = on != 0;
    return MPCNN_OK;
}

mpcnn_status mpcnn_profile_read(mpcnn_net* net, mpcnn_kernel_stat* out_host, int cap, int* n)
{
    if (!net || !n || (cap > 0 && !out_host)) return fail(MPCNN_EINVAL, "null argument");
    for (auto& p : net->pending) {
        HIP_TRY(hipEventSynchronize(p.e1));
        float ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&ms, p.e0, p.e1));
        net->sites[p.site].ms += ms;
        net->sites[p.site].launches += 1;
        net->pool.push_back(p.e0);
        net->pool.push_back(p.e1);
    }
    net->pending.clear();
    *n = (int)net->sites.size();
    for (int i = 0; i < *n && i < cap; ++i) {
        const ProfSite& s = net->sites[i];
        mpcnn_kernel_stat& o = out_host[i];
        memset(&o, 0, sizeof o);
        snprintf(o.name, sizeof o.name, "%s", s.name);
        o.layer = s.layer; o.step = s.step; o.launches = s.launches;
        o.ms_total = s.ms; o.flops = s.flops; o.bytes = s.bytes;
    }
    for (auto& s : net->sites) { s.ms = 0; s.launches = 0; }
    return MPCNN_OK;
}

}  // extern "C"
