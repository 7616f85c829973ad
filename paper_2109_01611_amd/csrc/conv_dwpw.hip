// A depthwise 3x3 convolution (stride 1, pad 1) and the 1x1 convolution behind it as one launch (the blocks of
// SSD-MobileNet, paper Table 4).
//
// As two launches the depthwise output makes a round trip, and at small batches both are little more than fixed
// cost.  Here a workgroup computes the depthwise output of its pixels for all channels into LDS (and copies it to
// its own buffer where somebody may want it), and multiplies it by the pointwise filters from there.
//
// A tile's pixels come in blocks of 4 x 2 pixels of one image, the patch a thread of the depthwise part owns
// (4 channels of it: see dwconv.hip); a block's eight pixels are eight rows of the product, those of a ragged
// edge are computed and not stored.  The product is taken as filters x pixels, which leaves a lane with four
// consecutive channels of one pixel: bias, ReLU, rounding and an 8-byte store, no staging.
//
// Two kernels:
//  * dwpw_small (32 or 128 channels: large maps, bound by memory): 256 threads, a tile's filters resident in LDS,
//    three or four workgroups per CU so that one's loads overlap another's arithmetic;
//  * dwpw_deep (192 to 512 channels): 12 wavefronts, all in the depthwise part (instruction issue and load latency:
//    3-5 us for 32 pixels of 512 channels), then 8 that multiply and 4 that bring the filters through a ring of three
//    stages, as in conv_igemm.hip.  The two parts do not overlap, so this pays for launches of one round only.
// At stride 2 the patches overlap less and the two launches are the faster way (64 -> 128 channels on 150x150 at batch
// 32 31.0 us, as one launch 38.7), and so they are with 64 channels (25.3 and 30.5) and with 1024 (17.1 and 27.0).
// Where it applies is in dwpw_applicable.
//
// Sums run in the order of the separate kernels (depthwise: bias, then taps ascending; pointwise: channels
// ascending), so the bits are theirs.
#include <algorithm>

#include "conv_common.h"

namespace gpulet {

using namespace conv;

namespace {

struct DwPwParams {
    const __bf16 *x, *wd, *w;
    const float *bd, *b;
    __bf16 *yd, *y;                      // yd: the depthwise output, or null
    int H, W, C, P, Q, K, relu_d, relu;
    int qb, n_blocks;                    // blocks per row of blocks, blocks in all
    int tiles, n_split, per_die;         // tiles of pixels, workgroups per tile, workgroups per die
    unsigned x_bytes, w_bytes;
    FastDiv d_qb, d_pb, d_split;         // by qb, blocks of rows per image, n_split
};

__device__ __forceinline__ void fetch(const DwPwParams &p) {
    asm volatile("" ::"s"(p.x), "s"(p.wd), "s"(p.w), "s"(p.bd), "s"(p.b), "s"(p.yd), "s"(p.y), "s"(p.H), "s"(p.W), "s"(p.C),
                 "s"(p.P), "s"(p.Q), "s"(p.K), "s"(p.relu_d), "s"(p.relu), "s"(p.qb), "s"(p.n_blocks), "s"(p.tiles),
                 "s"(p.n_split), "s"(p.per_die), "s"(p.x_bytes), "s"(p.w_bytes), "s"(p.d_qb.mul), "s"(p.d_qb.shift),
                 "s"(p.d_pb.mul), "s"(p.d_pb.shift), "s"(p.d_split.mul), "s"(p.d_split.shift));
}

// First pixel of a block.
struct Block {
    int n, p0, q0;
    __device__ __forceinline__ Block(const DwPwParams &p, int bi) {
        const int t = fdiv(bi, p.d_qb);
        q0 = (bi - t * p.qb) * 4;
        n = fdiv(t, p.d_pb);
        p0 = (t - n * ((p.P + 1) >> 1)) * 2;
    }
};

__device__ __forceinline__ void unpack4(const uint2 v, float (&f)[4]) {
    f[0] = __uint_as_float(v.x << 16);
    f[1] = __uint_as_float(v.x & 0xFFFF0000u);
    f[2] = __uint_as_float(v.y << 16);
    f[3] = __uint_as_float(v.y & 0xFFFF0000u);
}

// Depthwise output (stride 1) of channels c .. c+3 of one block: put(row 0..7 of the block, four bf16).  Pixels past
// the image's edge get values too.
template <typename Put>
__device__ __forceinline__ void depthwise_block(const DwPwParams &p, const Block &b, int c, Put put) {
    constexpr int SPAN = 6, ROWS = 4;   // input columns and rows of the block
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16 *>(p.x), 0, p.x_bytes, RSRC_FLAGS);
    const int h0 = b.p0 - 1, w0 = b.q0 - 1;
    uint2 xr[ROWS][SPAN];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        const bool h_ok = static_cast<unsigned>(h0 + i) < static_cast<unsigned>(p.H);
        const int row = (((b.n * p.H + h0 + i) * p.W + w0) * p.C + c) * 2;
#pragma unroll
        for (int u = 0; u < SPAN; ++u) {
            const bool ok = h_ok && static_cast<unsigned>(w0 + u) < static_cast<unsigned>(p.W);
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(rx, ok ? static_cast<unsigned>(row + u * (p.C * 2)) : OOB, 0, 0);
            xr[i][u] = make_uint2(v[0], v[1]);
        }
    }
    uint2 wr[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) wr[k] = *reinterpret_cast<const uint2 *>(p.wd + k * p.C + c);
    float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
    if (p.bd) bias = *reinterpret_cast<const float4 *>(p.bd + c);
    const unsigned limit = relu_limit(p.relu_d);
    float wt[9][4];
#pragma unroll
    for (int k = 0; k < 9; ++k) unpack4(wr[k], wt[k]);
    float acc[2][4][4];
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            acc[o][j][0] = bias.x;
            acc[o][j][1] = bias.y;
            acc[o][j][2] = bias.z;
            acc[o][j][3] = bias.w;
        }
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
#pragma unroll
        for (int u = 0; u < SPAN; ++u) {
            float xv[4];
            unpack4(xr[i][u], xv);
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const int r = i - o;
                if (r < 0 || r >= 3) continue;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int s = u - j;   // input column u is tap s of pixel j
                    if (s < 0 || s >= 3) continue;
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[o][j][e] = fmaf(xv[e], wt[r * 3 + s][e], acc[o][j][e]);
                }
            }
        }
        if (i >= 2) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                put((i - 2) * 4 + j, make_uint2(relu_or_pass(pack_bf16(acc[i - 2][j][0], acc[i - 2][j][1]), limit),
                                                relu_or_pass(pack_bf16(acc[i - 2][j][2], acc[i - 2][j][3]), limit)));
        }
    }
}

// LDS element of 16-byte chunk `chunk` of row `row`, ROWS rows of C channels: blocks of 64 channels, each
// swizzled like the stages of conv_igemm.hip; 32 channels are rows of 64 bytes, swizzled so that 16 rows at one
// chunk touch 16 different groups of banks.
template <int C>
__device__ __forceinline__ int tile_pos(int rows, int row, int chunk) {
    if (C == 32) return row * 32 + ((chunk ^ ((row >> 2) & 3)) * CHUNK);
    return (chunk >> 3) * (rows * BK) + lds_pos(row, chunk & 7);
}

// The depthwise part of a tile: BM / 8 blocks, all channels, into LDS at sA (tile_pos) and, for the first of the
// workgroups that share the tile, to memory.
template <int C_LAYOUT, int BM, int NTHR>
__device__ __forceinline__ void depthwise_tile(const DwPwParams &p, __bf16 *sA, int tile, bool to_memory, const FastDiv d_c4) {
    const int c4 = p.C >> 2, items = (BM / 8) * c4;
    for (int it = threadIdx.x; it < items; it += NTHR) {
        const int blk = C_LAYOUT == 0 ? fdiv(it, d_c4) : it / (C_LAYOUT >> 2);
        const int c = (it - blk * c4) * 4, bi = tile * (BM / 8) + blk;
        const bool live = bi < p.n_blocks;
        const Block b(p, live ? bi : 0);
        __bf16 *yd = p.yd + (((b.n * p.P + b.p0) * p.Q + b.q0) * p.C + c);
        depthwise_block(p, b, c, [&](int row, const uint2 v) {
            const int o = row >> 2, j = row & 3;
            *reinterpret_cast<uint2 *>(&sA[tile_pos<C_LAYOUT == 32 ? 32 : 64>(BM, blk * 8 + row, c >> 3) + (c & 7)]) = v;
            if (to_memory && live && b.p0 + o < p.P && b.q0 + j < p.Q)
                *reinterpret_cast<uint2 *>(yd + (o * p.Q + j) * p.C) = v;
        });
    }
}

// Where a lane's pixel of a tile goes: element offset of its channel 0 in y, or -1.
template <int BM>
__device__ __forceinline__ int out_offset(const DwPwParams &p, int tile, int row) {
    const int bi = tile * (BM / 8) + (row >> 3);
    if (bi >= p.n_blocks) return -1;
    const Block b(p, bi);
    const int pp = b.p0 + ((row >> 2) & 1), qq = b.q0 + (row & 3);
    return pp < p.P && qq < p.Q ? ((b.n * p.P + pp) * p.Q + qq) * p.K : -1;
}

typedef Mma<16> MM;

__device__ __forceinline__ void store4(const DwPwParams &p, int at, int k, const f32x4 acc, const float4 bias, unsigned limit) {
    if (at < 0) return;
    *reinterpret_cast<uint2 *>(p.y + (at + k)) = make_uint2(relu_or_pass(pack_bf16(acc[0] + bias.x, acc[1] + bias.y), limit),
                                                            relu_or_pass(pack_bf16(acc[2] + bias.z, acc[3] + bias.w), limit));
}

// 32 or 128 channels: 8192 / C pixels x BN filters per workgroup of four wavefronts (WM x WN).
template <int C, int BN, int WM, int WN>
__global__ __launch_bounds__(256, C == 32 ? 4 : 3) void dwpw_small(const DwPwParams p) {
    constexpr int BM = 8192 / C, MT = BM / WM / 16, NT = BN / WN / 16, KS = C / 32;
    static_assert(WM * WN == 4 && MT >= 1 && NT >= 1, "four wavefronts");
    __shared__ __attribute__((aligned(1024))) __bf16 sA[BM * C];
    __shared__ __attribute__((aligned(1024))) __bf16 sB[BN * C];
    fetch(p);
    const int item = die_block(p.per_die, blockIdx.x);
    if (item >= p.tiles * p.n_split) return;
    const int tile = fdiv(item, p.d_split), ns = item - tile * p.n_split, n0 = ns * BN;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    {   // the filters: 1 KB per transfer
        const i32x4 rw = make_rsrc(p.w, p.w_bytes);
        constexpr int CPR = C == 32 ? 4 : 8;             // chunks per row of a block
        constexpr int ROWS = 64 / CPR, PER = BN / ROWS;  // rows per transfer, transfers per block of channels
        const int r = lane / CPR;
        for (int t = wave; t < PER * (C == 32 ? 1 : C / 64); t += 4) {
            const int cb = t / PER, row = (t - cb * PER) * ROWS + r;
            const int chunk = C == 32 ? (lane & 3) ^ ((row >> 2) & 3) : (lane & 7) ^ ((row >> 1) & 7);
            dma16(rw, lds_addr(sB) + t * 1024, static_cast<unsigned>(((n0 + row) * C + cb * 64 + chunk * CHUNK) * 2));
        }
    }
    depthwise_tile<C, BM, 256>(p, sA, tile, p.yd && ns == 0, FastDiv{});
    const int wy = wave / WN, wx = wave - wy * WN, sub = lane & 15, kq = lane >> 4;
    int at[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) at[i] = out_offset<BM>(p, tile, wy * (BM / WM) + i * 16 + sub);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();

    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        bf16x8 fx[MT], fw[NT];
#pragma unroll
        for (int i = 0; i < MT; ++i)
            fx[i] = *reinterpret_cast<const bf16x8 *>(&sA[tile_pos<C>(BM, wy * (BM / WM) + i * 16 + sub, ks * 4 + kq)]);
#pragma unroll
        for (int j = 0; j < NT; ++j)
            fw[j] = *reinterpret_cast<const bf16x8 *>(&sB[tile_pos<C>(BN, wx * (BN / WN) + j * 16 + sub, ks * 4 + kq)]);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = MM::mul(fw[j], fx[i], acc[i][j]);
    }
    const unsigned limit = relu_limit(p.relu);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int k = n0 + wx * (BN / WN) + j * 16 + kq * 4;
        float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
        if (p.b) bias = *reinterpret_cast<const float4 *>(p.b + k);
#pragma unroll
        for (int i = 0; i < MT; ++i) store4(p, at[i], k, acc[i][j], bias, limit);
    }
}

// Many channels: BM pixels, BN filters at a time, K / (BN * n_split) times per workgroup.  Eight wavefronts
// multiply (BM pixels x BN / 8 filters each), four bring the filters.
constexpr int kDeepLds = 156 * 1024, kDeepStages = 3;
template <int BM, int BN>
__global__ __launch_bounds__(768) void dwpw_deep(const DwPwParams p, const int passes, const FastDiv d_c4) {
    constexpr int MT = BM / 16, NT = BN / 8 / 16, STAGE = BN * BK, BINS = BN / 32;
    static_assert(NT >= 1 && BINS * (kDeepStages - 1) <= 63, "tile shape");
    __shared__ __attribute__((aligned(1024))) __bf16 lds[kDeepLds / 2];
    __bf16 *ring = lds, *sA = lds + kDeepStages * STAGE;
    fetch(p);
    const int item = die_block(p.per_die, blockIdx.x);
    if (item >= p.tiles * p.n_split) return;
    const int tile = fdiv(item, p.d_split), ns = item - tile * p.n_split, n0 = ns * passes * BN;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nk = p.C / BK, steps = passes * nk;

    // producers: transfer u of a stage fills filter rows u * 32 + pw * 8 .. + 8
    const int pw = wave - 8, lrow = pw * 8 + (lane >> 3), chunk = (lane & 7) ^ ((lrow >> 1) & 7);
    const i32x4 rw = make_rsrc(p.w, p.w_bytes);
    const unsigned voff = static_cast<unsigned>((lrow * p.C + chunk * CHUNK) * 2);
    int pass_off = n0 * p.C * 2, k_off = 0, left = steps;   // byte offsets of the next stage's filters and depth
    auto issue = [&](int stage) {
        const unsigned base = lds_addr(ring) + pw * 1024 + stage * (STAGE * 2);
        const int soff = left > 0 ? pass_off + k_off : 0;    // past the last step: something harmless that nobody reads
#pragma unroll
        for (int u = 0; u < BINS; ++u) dma16(rw, base, u * 4096, voff + static_cast<unsigned>(u * 32 * p.C * 2), soff);
        --left;
        k_off += BK * 2;
        if (k_off == p.C * 2) {
            k_off = 0;
            pass_off += BN * p.C * 2;
        }
    };
    if (wave >= 8) {
#pragma unroll
        for (int i = 0; i < kDeepStages - 1; ++i) issue(i);
    }
    depthwise_tile<0, BM, 768>(p, sA, tile, p.yd && ns == 0, d_c4);
    __syncthreads();

    if (wave >= 8) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // the depthwise stores are behind the first stages
        int stage = kDeepStages - 1;
        for (int t = 0; t < steps; ++t) {
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(BINS * (kDeepStages - 2)));
            __syncthreads();
            issue(stage);
            stage = stage + 1 == kDeepStages ? 0 : stage + 1;
        }
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        return;
    }
    const int sub = lane & 15, kq = lane >> 4;
    int at[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) at[i] = out_offset<BM>(p, tile, i * 16 + sub);
    const unsigned limit = relu_limit(p.relu);
    int stage = 0;
    for (int pass = 0; pass < passes; ++pass) {
        const int k0 = n0 + pass * BN + wave * (BN / 8) + kq * 4;
        float4 bias[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            bias[j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (p.b) bias[j] = *reinterpret_cast<const float4 *>(p.b + k0 + j * 16);
        }
        f32x4 acc[MT][NT];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < nk; ++s) {
            __syncthreads();
            const __bf16 *a = sA + s * (BM * BK), *b = ring + stage * STAGE;
            bf16x8 fx[2][MT], fw[2][NT];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    fw[ks][j] = *reinterpret_cast<const bf16x8 *>(&b[lds_pos(wave * (BN / 8) + j * 16 + sub, ks * 4 + kq)]);
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    fx[ks][i] = *reinterpret_cast<const bf16x8 *>(&a[lds_pos(i * 16 + sub, ks * 4 + kq)]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j) acc[i][j] = MM::mul(fw[ks][j], fx[ks][i], acc[i][j]);
            stage = stage + 1 == kDeepStages ? 0 : stage + 1;
        }
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int i = 0; i < MT; ++i) store4(p, at[i], k0 + j * 16, acc[i][j], bias[j], limit);
    }
}

// Which kernel and tile a pair gets.
struct DwPwPlan {
    int bm = 0, bn = 0, n_split = 1, passes = 1;   // bn 0: none
    long long tiles = 0;
    bool deep = false;
};

DwPwPlan plan_pair(const DwPwArgs &a, int n_cu) {
    DwPwPlan r;
    const long long rows = 8LL * a.N * ((a.P + 1) / 2) * ((a.Q + 3) / 4);
    if (a.C == 32 || a.C == 128) {
        const int bn = a.C == 32 ? 64 : 128;
        if (a.K % bn != 0) return r;
        r.bn = bn;
        r.bm = 8192 / a.C;
        r.n_split = a.K / bn;
        r.tiles = (rows + r.bm - 1) / r.bm;
        return r;
    }
    if (a.C % BK != 0 || a.C < 192 || a.C > 512 || a.K % 128 != 0) return r;
    r.deep = true;
    // 48 pixels and all filters per workgroup; fewer pixels, then fewer filters, while that leaves CUs without work
    r.bm = (rows + 31) / 32 <= n_cu ? 32 : 48;
    r.tiles = (rows + r.bm - 1) / r.bm;
    r.bn = a.K % 256 == 0 && r.tiles * (a.K / 128) > n_cu ? 256 : 128;
    const int n_tiles = a.K / r.bn;
    for (int s = 1; s <= n_tiles; ++s)
        if (n_tiles % s == 0 && (s == 1 || r.tiles * s <= n_cu)) r.n_split = s;
    r.passes = n_tiles / r.n_split;
    return r;
}

}  // namespace

bool dwpw_applicable(const DwPwArgs &a, int n_cu) {
    if (a.N < 1 || a.stride != 1) return false;
    auto aligned = [](const void *q) { return reinterpret_cast<uintptr_t>(q) % 16 == 0; };
    if (!aligned(a.x) || !aligned(a.wd) || !aligned(a.w) || !aligned(a.bd) || !aligned(a.b) || !aligned(a.yd) || !aligned(a.y)) return false;
    // 32-bit offsets with the top bit as the out-of-range marker; a block may reach past a row and an image
    const long long lim = 1LL << 30, slack = 8LL * (a.W + 8) * a.C;
    if (1LL * a.N * a.H * a.W * a.C + slack >= lim || 1LL * a.N * a.P * a.Q * std::max(a.C, a.K) + slack >= lim || 1LL * a.K * a.C >= lim)
        return false;
    const int cus = n_cu < 1 ? 1 : n_cu;
    const DwPwPlan r = plan_pair(a, cus);
    if (r.bn == 0) return false;
    // Against two launches (us, two and one):
    // 32 channels, 150x150: 9.3/7.7 at batch 1 on 160 CUs, 16.1/11.1 at batch 4 on 256 (all workgroups resident); with more
    // rounds the pair alone gains (52/47 at batch 32) and whole SSD-MobileNet loses (435 and 442 us).  Its launch takes 7.2 us
    // however small, the two together 5.5 to 7.9 below one workgroup for three CUs (102 of 119 pairs 3 % slower and
    // more, 7 % in the mean), and several workgroups per tile want one round (128 filters: 8.5/7.8 with 0.96 workgroups per
    // CU, 9.9/10.0 with 1.2); between these lines 52 pairs gain 4.5 % in the mean.
    // 128 channels, 75x75: 8.0/6.8 at batch 1, 37.2/35.9 at batch 32 on 256 CUs (11 tiles per CU); on 64 CUs at batch 16
    // (23 per CU) 60.7/61.4.  With two workgroups per tile, each doing the depthwise part (38x38 to 256): 8.5/7.1 at
    // batch 4 (0.75 workgroups per CU), 9.3/9.2 at batch 8, 12.7/14.2 at batch 16.
    // Deep: 256 channels on 38x38 7.7/5.8 at batch 1, 11.3/9.7 at batch 8 (254 tiles on 256 CUs), 16.3/17.2 at batch 16;
    // 512 on 19x19 8.2/7.6 and 10.4/9.5 at batch 1 and 8, where a workgroup has one pass over the filters, 12.8/13.1 at
    // batch 16 with two.  One workgroup fills a CU, so a second round costs as much as the first.  Other channel counts lie
    // between: 187 pairs of 192 to 512 channels (maps of 2x2 to 80x80, batch 1 to 32, 64 to 256 CUs) take 9 to 31 % less in
    // the mean of a channel count, 88 with 128 channels 18 %, and none takes 0.5 % more.
    if (r.deep) return r.passes == 1 && r.tiles * r.n_split <= cus;
    const long long wgs = r.tiles * r.n_split;
    if (a.C == 32) return 3 * wgs >= cus && wgs <= (r.n_split > 1 ? 1LL : 4LL) * cus;
    return r.n_split > 1 ? 4 * wgs <= 5LL * cus : wgs <= 14LL * cus;
}

hipError_t launch_dwpw(const DwPwArgs &a, int n_cu, hipStream_t stream) {
    if (!dwpw_applicable(a, n_cu)) return hipErrorInvalidValue;
    const DwPwPlan r = plan_pair(a, n_cu < 1 ? 1 : n_cu);
    DwPwParams p;
    p.x = static_cast<const __bf16 *>(a.x);
    p.wd = static_cast<const __bf16 *>(a.wd);
    p.w = static_cast<const __bf16 *>(a.w);
    p.bd = a.bd;
    p.b = a.b;
    p.yd = static_cast<__bf16 *>(a.yd);
    p.y = static_cast<__bf16 *>(a.y);
    p.H = a.H; p.W = a.W; p.C = a.C; p.P = a.P; p.Q = a.Q; p.K = a.K; p.relu_d = a.relu_d; p.relu = a.relu;
    const int pb = (a.P + 1) / 2;
    p.qb = (a.Q + 3) / 4;
    p.n_blocks = a.N * pb * p.qb;
    p.tiles = static_cast<int>(r.tiles);
    p.n_split = r.n_split;
    p.per_die = (p.tiles * r.n_split + 7) / 8;
    p.x_bytes = static_cast<unsigned>(2LL * a.N * a.H * a.W * a.C);
    p.w_bytes = static_cast<unsigned>(2LL * a.K * a.C);
    p.d_qb = make_fastdiv(p.qb);
    p.d_pb = make_fastdiv(pb);
    p.d_split = make_fastdiv(r.n_split);
    const dim3 grid(static_cast<unsigned>(8 * p.per_die));
    const FastDiv d_c4 = make_fastdiv(a.C / 4);
    auto small = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, p); };
    auto deep = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(768), 0, stream, p, r.passes, d_c4); };
    if (!r.deep) {
        a.C == 32 ? small(dwpw_small<32, 64, 4, 1>) : small(dwpw_small<128, 128, 2, 2>);
    } else if (r.bn == 256) {
        r.bm == 48 ? deep(dwpw_deep<48, 256>) : deep(dwpw_deep<32, 256>);
    } else {
        r.bm == 48 ? deep(dwpw_deep<48, 128>) : deep(dwpw_deep<32, 128>);
    }
    return hipGetLastError();
}

}  // namespace gpulet
