// Convolution layer of the forward pass served on a gpu-let (paper Sec. 5; the
// models of Table 4): argument checks and the choice of kernel.  The kernels
// themselves live in conv_igemm.hip (implicit GEMM with gathered operands, the
// general case), conv_patch.hip (3x3 with the input patch in LDS), conv_stream.hip
// (1x1 with a short depth), conv_stem.hip (at most four input channels) and
// conv_pooled.hip (max pool fused into a 1x1 convolution); conv_common.h holds
// what they share.
#include <algorithm>
#include <atomic>

#include "conv_common.h"

namespace gpulet {

using namespace conv;

namespace {

// Off by default: the partial tiles cross dies through memory, which costs about 8 us per
// launch on MI355X and only pays for layers with very few tiles and a very long depth.
std::atomic<int> g_max_split_k{1};
std::atomic<int> g_pool_fusion{1};

std::atomic<int> g_tile_override{-1};

struct TileChoice {
    int id, bm, bn;
    float eff;  // relative MFMA efficiency of the tile shape (bigger tiles reuse LDS reads more)
};

// The gathering tiles in the order in which they are tried (on a tie the earlier one wins).
// 192x128 and 96x128 exist for the layers whose 128-pixel tiles just miss a whole number of
// rounds on a gpu-let (98 tiles on 96 CUs, 196 on 192): three row tiles per wavefront instead
// of two or four change the tile count enough to save a round.  32x32 is for launches whose 64x64
// tiles leave CUs idle: such a launch waits for the ~50 B/clk at which one CU takes transfers, so
// the rows a workgroup stages (64 instead of 128 per slice) set its time: 0.55 of a 64x64 round
// (1x1 2048 -> 512 on 7x7 at batch 1 6.6 us in 64x64, 4.7 in 32x32; 3x3/2 512 -> 512 on 14x14 12.8 and 8.5; with
// a second workgroup on every CU it is the slower one, 512 -> 1024 on 10x10 at batch 5 4.3 against 4.0,
// except for filters larger than 1x1 and depths from 18 slices on, see choose_kernel).
const TileChoice kTiles[] = {{6, 256, 128, 1.00f}, {12, 192, 128, 0.93f}, {0, 128, 128, 0.90f}, {13, 96, 128, 0.80f},
                             {2, 64, 128, 0.72f},  {1, 128, 64, 0.72f},   {3, 64, 64, 0.58f},   {5, 32, 128, 0.40f},
                             {4, 128, 32, 0.30f},  {14, 32, 32, 0.26f}};
constexpr int kNumTiles = static_cast<int>(sizeof(kTiles) / sizeof(kTiles[0]));

bool is_gathering_tile(int id) { return (id >= 0 && id <= 6) || (id >= 12 && id <= 14); }


}  // namespace

gpulet_status check_conv(const ConvArgs &a) {
    if (!a.x || !a.w || !a.y) return GPULET_EINVAL;
    if (a.N < 1 || a.C < 1 || a.H < 1 || a.W < 1 || a.K < 1 || a.R < 1 || a.S < 1 || a.stride < 1 ||
        a.pad < 0)
        return GPULET_EINVAL;
    if (a.P < 1 || a.Q < 1) return GPULET_EINVAL;
    if (a.y2) {
        if (a.k2 < 1 || a.k2 >= a.K || a.R != 1 || a.S != 1 || a.pad != 0 || a.residual || a.pre_pool)
            return GPULET_EINVAL;
        if (a.y2_ch_offset < 0 || a.y2_ch_offset + (a.K - a.k2) > a.y2_ch_stride) return GPULET_EINVAL;
        if (1LL * a.N * a.P * a.Q * a.y2_ch_stride >= (1LL << 30)) return GPULET_EINVAL;
    }
    if (a.y_ch_offset < 0 || a.y_ch_offset + (a.y2 ? a.k2 : a.K) > a.y_ch_stride) return GPULET_EINVAL;
    if (a.pool_y && (a.R != 1 || a.S != 1 || a.pad != 0 || a.pre_pool || a.C % 8 != 0 ||
                     (a.x_ch_stride != 0 && a.x_ch_stride != a.C)))
        return GPULET_EINVAL;
    if (a.post_pool2 != 0 && (a.post_pool2 != 2 || a.P % 2 != 0 || a.Q % 2 != 0 || a.residual || a.y2 || a.pool_y || a.pre_pool))
        return GPULET_EINVAL;
    if (a.pre_pool != 0 && (a.pre_pool != 3 || a.R != 1 || a.S != 1 || a.stride != 1 || a.pad != 0 || a.C % 8 != 0))
        return GPULET_EINVAL;
    const int ldx = a.x_ch_stride ? a.x_ch_stride : a.C;
    if (a.x_ch_offset < 0 || a.x_ch_offset + a.C > ldx) return GPULET_EINVAL;
    if (ldx != a.C && a.pre_pool) return GPULET_EINVAL;
    // Byte offsets are 32-bit with the top bit reserved as the out-of-range marker.
    const long long lim = 1LL << 30;
    const long long xe = 1LL * a.N * a.H * a.W * ldx;
    const long long we = 1LL * a.K * a.R * a.S * a.C;
    const long long ye = 1LL * a.N * a.P * a.Q * a.y_ch_stride;
    // The gather indexes from (h, w) = (-pad, -pad) and may step past the last tap.
    const long long slack = (1LL * (a.pad + a.R) * a.W + a.pad + a.S) * ldx + 64;
    if (xe + slack >= lim || we + 64 >= lim || ye >= lim) return GPULET_EINVAL;
    return GPULET_OK;
}

namespace {

// The kernel's parameter block for one layer (tile-dependent fields are filled in by the
// launchers) and whether its operands allow 16-byte gathers.
hipError_t make_params(const ConvArgs &a, const LaunchCtx &ctx, ConvParams &p, bool &vec) {
    p.ldx = a.x_ch_stride ? a.x_ch_stride : a.C;
    p.x = static_cast<const __bf16 *>(a.x) + a.x_ch_offset;
    p.w = static_cast<const __bf16 *>(a.w);
    p.b = a.b;
    p.y = static_cast<__bf16 *>(a.y);
    p.res = static_cast<const __bf16 *>(a.residual);
    p.N = a.N; p.C = a.C; p.H = a.H; p.W = a.W; p.K = a.K; p.R = a.R; p.S = a.S;
    p.stride = a.stride; p.pad = a.pad; p.relu = a.relu; p.P = a.P; p.Q = a.Q;
    p.M = a.N * a.P * a.Q;
    p.Kg = a.R * a.S * a.C;
    p.ldy = a.y_ch_stride;
    p.y_off = a.y_ch_offset;
    p.y2 = static_cast<__bf16 *>(a.y2);
    p.k2 = a.y2 ? a.k2 : a.K;
    p.ldy2 = a.y2_ch_stride;
    p.y2_off = a.y2_ch_offset;
    p.pool2 = p.pad4 = 0;
    p.stamps = static_cast<long long *>(a.stamps);
    p.tiles_n = p.n_tiles = p.tiles_per_xcd = 0;
    // up to the last channel the layer reads of the last pixel
    p.x_bytes = static_cast<unsigned>(2LL * ((1LL * a.N * a.H * a.W - 1) * p.ldx + a.C));
    p.w_bytes = static_cast<unsigned>(2LL * a.K * a.R * a.S * a.C);
    p.tap_inner = a.C % BK == 0 ? 1 : 0;
    p.vec_store = (a.y_ch_stride % 8 == 0 && a.y_ch_offset % 8 == 0 && reinterpret_cast<uintptr_t>(a.y) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(a.b) % 16 == 0 &&
                   (!a.residual || (a.K % 8 == 0 && reinterpret_cast<uintptr_t>(a.residual) % 16 == 0)) &&
                   (!a.y2 || (a.k2 % 8 == 0 && a.y2_ch_stride % 8 == 0 && a.y2_ch_offset % 8 == 0 &&
                              reinterpret_cast<uintptr_t>(a.y2) % 16 == 0)))
                      ? 1
                      : 0;
    p.split_k = 1;
    p.sps = 0;
    p.part = ctx.scratch;
    p.cnt = ctx.counters;
    p.tw = p.n_cb = p.th = p.tiles_img = 0;
    p.d_pq = make_fastdiv(a.P * a.Q);
    p.d_q = make_fastdiv(a.Q);
    p.d_p = make_fastdiv(a.P);
    p.d_c = make_fastdiv(a.C);
    p.d_s = make_fastdiv(a.S);
    p.d_tiles_n = p.d_split_k = p.d_tw = p.d_ncb = p.d_pwt = p.d_hp = make_fastdiv(1);

    vec = (a.C % CHUNK == 0) && (p.ldx % CHUNK == 0) && (reinterpret_cast<uintptr_t>(p.x) % 16 == 0) &&
                     (reinterpret_cast<uintptr_t>(a.w) % 16 == 0);
    if (a.y2 && !vec) return hipErrorInvalidValue;  // only the 16-byte gathering kernels store to two tensors
    p.side_blocks = 0;
    p.side_pool = PoolParams{};
    if (a.pool_y) {
        if (!vec || reinterpret_cast<uintptr_t>(a.pool_y) % 16 != 0) return hipErrorInvalidValue;
        PoolParams &sp = p.side_pool;
        sp.x = static_cast<const __bf16 *>(a.x);
        sp.y = static_cast<__bf16 *>(a.pool_y);
        sp.N = a.N; sp.C = a.C; sp.H = a.H; sp.W = a.W; sp.P = a.H; sp.Q = a.W; sp.k = 3; sp.stride = 1; sp.pad = 1;
        sp.total = a.N * a.H * a.W * (a.C / 8);
        sp.d_cv = make_fastdiv(a.C / 8);
        sp.d_q = make_fastdiv(a.W);
        sp.d_p = make_fastdiv(a.H);
    }
    return hipSuccess;
}

// Which kernel runs a layer: 0..6 and 12..14 a gathering tile (with `split` workgroups per tile), 7
// the patch kernel (column block `tw`, tile `patch_tile`), 8 the streaming 1x1 kernel, 9 the stem
// kernel, 10 the resident-weight kernel (column block `tw64`), 11 the tall tile (`th11` x `tw11`).
struct Choice {
    int best, split, tw, tw64, th11, tw11, patch_tile;
    double cost;   // of `best` in the cost model's units when it is a gathering tile or the tall tile, else 0
};

// Cost of a layer on the tall tile in the units of choose_kernel: rounds on the busiest CU x tile
// area / efficiency relative to the 256x128 gathering tile.  The efficiency is fitted to
// measurements on MI355X (3x3 layers of 128..512 channels on 14..112 pixel maps at batch 16 and
// 32, on 64, 128 and 256 CUs): 0.95 when every tile row is a pixel and the depth is long, less a
// share of the rows that are not pixels (they are already in the tile count; what remains is that
// the epilogue and the patch do not shrink with them) and the first loads and the epilogue that
// a short depth does not amortise.
double tall_cost(const ConvParams &p, int th, int tw, double geo, int n_cu) {
    const double eff = 0.95 - 0.35 * (1.0 - geo) - 0.04 / (p.C / BK);
    return static_cast<double>((tall_tiles(p, th, tw) + n_cu - 1) / n_cu) * 224 * 128 / eff;
}

// Loading 144 registers of weights per consumer (about 2.5 us) wants three pixel tiles per workgroup, and 4.5 where several
// filter tiles share a gathered pixel tile.
bool c64_enough_tiles(const C64Grid &g, int n_cu) {
    return 2LL * g.tiles_m >= (g.tiles_n == 1 ? 6LL : 9LL) * std::max(1, n_cu / g.tiles_n);
}

Choice choose_kernel(const ConvParams &p, bool vec, const LaunchCtx &ctx) {
    // Pick the tile and the split of the depth that minimise
    //   (work items on the busiest CU) x (tile area) x (share of the depth + fixed cost of a split) / efficiency.
    // The efficiencies are measured throughput ratios on MI355X (large layers, all CUs busy);
    // on a tie the earlier entry wins.  A split needs the gpu-let's scratch, at least four
    // slices per workgroup, and pays for parking and re-reading fp32 partial tiles.
    const int nk = (p.Kg + BK - 1) / BK;
    const int forced = g_tile_override.load();
    const int max_split = (vec && ctx.scratch && forced < 0) ? g_max_split_k.load() : 1;
    int best = 0, best_split = 1;
    double best_cost = 0.0;
    const int n_cu = ctx.n_cu < 1 ? 1 : ctx.n_cu;
    for (int o = 0; o < kNumTiles; ++o) {
        const TileChoice &t = kTiles[o];
        const int i = t.id;
        const long long tiles = 1LL * ((p.M + t.bm - 1) / t.bm) * ((p.K + t.bn - 1) / t.bn);
        for (int sk = 1; sk <= max_split; ++sk) {
            if (sk > 1) {
                const int sps = (nk + sk - 1) / sk;
                if (sps < 4 || (sk - 1) * sps >= nk) continue;                         // too thin, or an empty split
                if (tiles > ctx.n_counters) continue;
                if (static_cast<size_t>(tiles) * sk * t.bm * t.bn * 4 > ctx.scratch_bytes) continue;
            }
            const long long per_cu = (tiles * sk + n_cu - 1) / n_cu;
            const double share = 1.0 / sk + (sk > 1 ? 0.06 + 0.02 * sk : 0.0);
            double eff = t.eff;
            // 128x128 runs two workgroups per CU when there are more tiles than CUs (see the
            // launch below); the overlap of one's loads with the other's epilogue weighs more
            // the shorter the depth (measured against 256x128 at 9 .. 72 slices).
            // (filters larger than 1x1 gain less: 0.92-0.95 measured at 18 and 36 slices)
            // Two workgroups of 32x32 per CU against one of 64x64: 3x3 512 -> 512 on 14x14 at batch 5 15 against
            // 19 us, 128 -> 128 on 28x28 even.
            if (i == 14 && p.R * p.S > 1 && nk >= 18) eff = 0.30;
            if (i == 0 && sk == 1 && tiles > n_cu) eff = std::min(1.2, 0.90 + (p.R * p.S == 1 ? 3.0 : 0.6) / nk);
            const double cost = static_cast<double>(per_cu) * t.bm * t.bn * share / eff;
            if ((o == 0 && sk == 1) || cost < best_cost) {
                best = i;
                best_split = sk;
                best_cost = cost;
            }
        }
    }
    if (forced >= 0 && forced < GPULET_CONV_TILES) {
        best = forced;
        best_split = 1;
    }
    // The tall tile (224 pixels of one image x 128 filters, input patch in LDS) against the best
    // gathering tile, in the same units (tall_cost).
    int th11 = 0, tw11 = 0;
    double geo11 = 0.0;
    const bool tall_ok = tall_eligible(p, vec, &th11, &tw11, &geo11);
    if (forced < 0 && tall_ok && p.C >= 2 * BK) {
        const double cost = tall_cost(p, th11, tw11, geo11, n_cu);
        if (cost < best_cost) {
            best = 11;
            best_split = 1;
            best_cost = cost;
        }
    }
    int tw = 0;
    const bool patch_ok = patch_eligible(p, vec, &tw);
    if (best == 7 && !patch_ok) best = 1;  // the patch kernel does not apply: same tile shape, gathered
    // The patch kernel runs one workgroup per CU.  Measured on MI355X it beats the gathering
    // tiles whenever all of its 128x64 workgroups are resident at once (a second round doubles its
    // time), from a single block of 64 channels on: 3x3 64 -> 64 on 56x56 at batch 8 5.5 against
    // 6.2 us, 128 -> 256 on 14x14 at batch 32 6.9 against 7.8, 192 -> 384 on 7x7 7.9 against 10.0.
    // patch_variant() then says whether smaller tiles spread it better.
    int patch_tile = 0;
    if (forced < 0 && patch_ok) {
        bool one_round = false;
        const int v = patch_variant(p, tw, n_cu, &one_round);
        if (one_round) {
            best = 7;
            best_split = 1;
            patch_tile = v;
        }
    }
    if (best == 8 && !stream_applicable(p, vec)) best = 2;  // same tile shape, one tile per workgroup
    if (forced < 0 && stream_eligible(p, vec, n_cu)) best = 8;
    int tw64 = 0;
    const bool c64_ok = c64_applicable(p, vec, &tw64);
    if (best == 10 && !c64_ok) best = 1;
    // The resident-weight kernel takes 4.2 us and 2.1 to 2.4 per pixel tile of its busiest workgroup, the best gathering
    // tile 2.4 us and 2.0 to 2.2 per 128x64 of the cost above.  In 1454 layers (8 to 320 filters, maps of 14 to 224, batch
    // 1 to 64, 64 to 256 CUs) the second condition picks the slower one in nine, by 4 % at most: 64 -> 64 on 56x56 at batch 32 on
    // 256 CUs (4 tiles) 15.0 us gathered and 14.3, 64 -> 192 there (10 tiles) 34.3 and 27.8, but 64 -> 128 on 64 CUs
    // (25 tiles) 53.6 and 57.7, 64 -> 256 on 20x20 on 128 CUs (columns of 16 in rows of 20, 5 tiles) 11.3 and 15.7.
    // The tiles' efficiencies hold for long depths: at nine slices those over 64 rows x 128 filters are 8 % dearer, and 128x128
    // is 5 % cheaper unless all CUs draw on memory.
    if (forced < 0 && c64_ok) {
        const C64Grid g = c64_grid(p, tw64, n_cu);
        const bool large = best == 6 || best == 12 || best == 13;
        const double nine = large ? 1.08 : best == 0 && n_cu <= 192 ? 0.95 : 1.0;
        if (c64_enough_tiles(g, n_cu) && (g.rounds + 1.0) * PATCH_BM * 64 <= nine * best_cost) best = 10;
    }
    if (best == 9 && !stem_applicable(p)) best = 1;
    if (forced < 0 && stem_applicable(p)) best = 9;  // by shape alone: the same bits in every batch and gpu-let
    if (best == 11 && !tall_ok) best = 1;
    return Choice{best, best_split, tw, tw64, th11, tw11, patch_tile, (is_gathering_tile(best) || best == 11) ? best_cost : 0.0};
}

// Only the gathering tiles split.
bool splits_depth(const Choice &c) { return is_gathering_tile(c.best) && c.split > 1; }

}  // namespace

hipError_t launch_conv(const ConvArgs &a, const LaunchCtx &ctx, hipStream_t stream) {
    ConvParams p;
    bool vec = false;
    const hipError_t st = make_params(a, ctx, p, vec);
    if (st != hipSuccess) return st;
    if (a.pre_pool) {
        // checked by check_conv: 3x3 window, 1x1 filter, stride 1, no padding, C % 8 == 0; the
        // callers check the 16-byte alignment of x and w
        if (!vec || p.ldx != a.C) return hipErrorInvalidValue;
        return launch_pooled_conv(p, stream);
    }

    if (a.post_pool2) {
        // the two kernels with a pooled epilogue: weights in registers for 64 input channels, else the tall tile
        int th = 0, tw = 0;
        double geo = 0.0;
        if (a.post_pool2 != 2 || a.y2 || a.pool_y) return hipErrorInvalidValue;
        if (c64_applicable(p, vec, &tw, true)) return launch_c64(p, tw, ctx.n_cu < 1 ? 1 : ctx.n_cu, true, stream);
        if (!tall_eligible(p, vec, &th, &tw, &geo, true)) return hipErrorInvalidValue;
        return launch_tall(p, th, tw, true, stream);
    }
    const Choice c = choose_kernel(p, vec, ctx);
    const int n_cu = ctx.n_cu < 1 ? 1 : ctx.n_cu;
    switch (c.best) {
        case 11: return launch_tall(p, c.th11, c.tw11, false, stream);
        case 10: return launch_c64(p, c.tw64, n_cu, false, stream);
        case 9: return launch_stem(p, n_cu, stream);
        case 8: return launch_stream(p, n_cu, stream);
        case 7: return launch_patch(p, c.tw, c.patch_tile, stream);
        default: {
            const long long tiles128 = 1LL * ((p.M + 127) / 128) * ((p.K + 127) / 128);
            // 16x16 tiles where they still all start at once: a CU takes operands that are in no nearby cache
            // at about 60 KB/us, however many of them it has requested (a ring of 8 stages instead of 3 made 32x32
            // tiles 2 % slower), so what counts is how many CUs share the operands' transfer.  1x1 2048 -> 512 on 7x7 at
            // batch 1 4.6 us in 32x32, 3x3/2 512 -> 512 on 14x14 9.0 and 7.8, 3x3/2 256 -> 256 on 28x28 6.0 and 5.4;
            // with a second workgroup on a CU they lose.  Filters larger than 1x1 on other channel counts than multiples of
            // 64, whose producers work out every chunk's tap, have two producers for it instead of four and lose
            // too until the depth is long (3x3/2 8 -> 24 on 14x14 4.7 and 7.0, 5x5 16 -> 96 5.4 and 5.9; 388 such layers
            // of fewer than 28 slices 14 % slower, the other 1112 measured 6 % faster).
            int tile = c.best;
            const long long tiles16 = 1LL * ((p.M + 15) / 16) * ((p.K + 15) / 16);
            const bool plain = p.R * p.S == 1 || p.C % BK == 0 || p.Kg >= 28 * BK;
            if (tile == 14 && vec && c.split == 1 && g_tile_override.load() < 0 && plain && tiles16 <= n_cu) tile = kTile16;
            return launch_igemm(p, vec, tile, c.split, tiles128 > n_cu, stream);
        }
    }
}

// The pooled epilogue saves the layer's full-size store and the pool kernel's pass over it (at
// least a sixth of the pair's time on the layers it applies to), so the tall tile may cost up to
// 15 % more than the kernel the layer would get by itself.  Layers that a specialised kernel takes
// (all workgroups of the patch kernel resident, 64 input channels) keep it and their pool kernel.
bool conv_pool2_fusable(const ConvArgs &a, const LaunchCtx &ctx) {
    if (!conv_fusion_allowed()) return false;
    if (a.pre_pool || a.y2 || a.pool_y || a.residual || !a.relu) return false;
    ConvParams p;
    bool vec = false;
    if (make_params(a, ctx, p, vec) != hipSuccess) return false;
    int th = 0, tw = 0;
    double geo = 0.0;
    const Choice c = choose_kernel(p, vec, ctx);
    if (splits_depth(c)) return false;   // partial sums: other bits than the pooled epilogue's
    if (c.best == 10) return c64_applicable(p, vec, &tw, true);   // the same kernel with another epilogue
    // With the pool it also pays where it does not alone: in 343 pairs (16 to 256 filters, maps of 14 to 224, batch 1 to
    // 64, 64 to 256 CUs) by 7 % at least.
    if (c64_applicable(p, vec, &tw, true)) {
        const int n_cu = std::max(1, ctx.n_cu);
        return c64_enough_tiles(c64_grid(p, tw, n_cu), n_cu);
    }
    if (p.C < 2 * BK || !tall_eligible(p, vec, &th, &tw, &geo, true)) return false;
    if (c.cost <= 0.0) return false;
    return tall_cost(p, th, tw, geo, ctx.n_cu < 1 ? 1 : ctx.n_cu) <= 1.15 * c.cost;
}

bool conv_splits_depth(const ConvArgs &a, const LaunchCtx &ctx) {
    if (g_max_split_k.load() <= 1) return false;
    ConvParams p;
    bool vec = false;
    return make_params(a, ctx, p, vec) == hipSuccess && splits_depth(choose_kernel(p, vec, ctx));
}

// Independent layers in one launch.  Every member must be a layer the gathering kernel would
// run anyway, unsplit: 16-byte gathers, no fused pool, one output, and none of the specialised
// kernels chosen for its shape; otherwise the members are launched one after the other.  The
// tile shared by all members minimises the work of the busiest CU (slices and a fixed part per
// round) over the members' tiles together.  Results are those of separate launches, bit for bit.
hipError_t launch_conv_group(const ConvArgs *a, int n, const LaunchCtx &ctx, hipStream_t stream, int *launches) {
    ConvParams p[MAX_GROUP];
    bool together = n >= 2 && n <= MAX_GROUP;
    const int forced = g_tile_override.load();
    for (int j = 0; j < n && together; ++j) {
        bool vec = false;
        if (make_params(a[j], ctx, p[j], vec) != hipSuccess || !vec || a[j].pre_pool || a[j].y2 || a[j].pool_y) {
            together = false;
            break;
        }
        const Choice c = choose_kernel(p[j], vec, ctx);
        if (!is_gathering_tile(c.best) || splits_depth(c)) together = false;
    }
    if (launches) *launches = together ? 1 : n;
    if (!together) {
        for (int j = 0; j < n; ++j) {
            const hipError_t st = launch_conv(a[j], ctx, stream);
            if (st != hipSuccess) return st;
        }
        return hipSuccess;
    }
    const int n_cu = ctx.n_cu < 1 ? 1 : ctx.n_cu;
    long long tiles128 = 0, slices128 = 0;
    for (int j = 0; j < n; ++j) {
        const long long tj = 1LL * ((p[j].M + 127) / 128) * ((p[j].K + 127) / 128);
        tiles128 += tj;
        slices128 += tj * ((p[j].Kg + BK - 1) / BK);
    }
    // The deepest member first: its workgroups start first, and a CU's second one is then a shallower one.
    std::stable_sort(p, p + n, [](const ConvParams &a, const ConvParams &b) { return a.Kg > b.Kg; });
    int best = 0;
    double best_cost = 0.0;
    for (int o = 0; o < kNumTiles; ++o) {
        const TileChoice &t = kTiles[o];
        // Work of the busiest CU, the one that takes workgroups 0, n_cu, 2 n_cu, ...  With members of
        // different depths a round costs the slices of its deepest workgroup (4d at batch 1 on 64
        // CUs 7.1 us in 32x32, 7.6 in 64x64) and, whatever the depth, what fetching the arguments, the
        // first transfers and the epilogue take: as much as 7 to 9 slices, fitted over every tile of
        // 432 groups (inception blocks, ResNet shortcuts, detection heads; batch 1 to 32 on 64 to 256
        // CUs).  Without that part a tile with a shallow second round looks too cheap (4a at batch 32 on
        // 192 CUs: 196 tiles of 128x128 12.6 us, 294 of 128x64 12.0).
        constexpr int kFixedSlices = 8;
        long long tiles = 0, slices = 0;
        for (int j = 0; j < n; ++j) {
            const long long first = (tiles + n_cu - 1) / n_cu;   // this member's first round
            tiles += 1LL * ((p[j].M + t.bm - 1) / t.bm) * ((p[j].K + t.bn - 1) / t.bn);
            slices += ((tiles + n_cu - 1) / n_cu - first) * ((p[j].Kg + BK - 1) / BK);
        }
        double eff = t.eff;
        // The same bonus as in a single launch for 128x128 with two workgroups per CU, at the
        // members' mean depth (inception 3a's group at batch 32: 18.0 -> 15.8 us), but no more than
        // 1.1: a second, shallower member fills less (3b at batch 32 on 256 CUs 30.4 us, 28.7 in 128x64).
        if (t.id == 0 && tiles128 > n_cu) eff = std::min(1.1, 0.90 + 3.0 * tiles128 / slices128);
        const long long rounds = (tiles + n_cu - 1) / n_cu;
        const double cost = static_cast<double>(slices + kFixedSlices * rounds) * t.bm * t.bn / eff;
        if (o == 0 || cost < best_cost) {
            best = t.id;
            best_cost = cost;
        }
    }
    if (is_gathering_tile(forced)) best = forced;
    return launch_igemm_group(p, n, best, tiles128 > n_cu, stream);
}

void set_conv_split_k(int max_split) { g_max_split_k.store(max_split); }

bool conv_fusion_allowed() { return g_pool_fusion.load() && g_tile_override.load() < 0; }

void set_conv_pool_fusion(int on) { g_pool_fusion.store(on ? 1 : 0); }

void set_conv_tile(int tile) { g_tile_override.store(tile); }

}  // namespace gpulet
