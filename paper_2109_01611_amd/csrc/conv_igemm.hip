// Convolution layer of the forward pass served on a gpu-let (paper Sec. 5; the
// models of Table 4), as an implicit GEMM on gfx950 matrix cores:
//
//   rows    m = (n, p, q)   output pixels          M  = N*P*Q
//   columns k               output channels        Ng = K
//   depth   g = (r, s, c)   filter taps x channels Kg = R*S*C
//
// x is NHWC and w is KRSC, so both operands are contiguous along the depth
// and neither the im2col matrix nor a transposed weight is ever built.
//
// One workgroup owns a BM x BN output tile and walks the depth in slices of 64.
// Its wavefronts are specialised.  Producer wavefronts only compute addresses
// and issue 16-byte buffer loads (8 channels of one tap) that land directly in
// LDS without passing through registers; the hardware range check of the
// buffer descriptor returns zeros for padding taps and ragged edges, so the
// gather has no branches.  Consumer wavefronts only read 8-element fragments
// back from the XOR-swizzled LDS tile with ds_read_b128 and feed
// v_mfma_f32_32x32x16_bf16; accumulators stay in registers for the whole
// depth.  Slices travel through a ring of three LDS stages, two loads ahead of
// the one being multiplied, with one workgroup barrier per slice.  When the
// channel count is a multiple of 64 the depth is walked with the filter taps
// innermost, so a producer's lane keeps its channel offset and only steps the
// tap.  The epilogue parks the fp32 tile in the idle ring, adds bias and the
// optional residual, applies ReLU, rounds once to bf16 and writes 16-byte
// rows, optionally at a channel offset inside a wider (concatenated) tensor.
// Optionally several workgroups share a tile by splitting the depth; partial
// tiles meet in device scratch and the last one to arrive reduces them in a
// fixed order.
//
// Channel counts that are not multiples of 8 (image stems, LeNet) take a
// scalar-gather variant of the same tiling with four wavefronts.
#include <climits>

#include "conv_common.h"

namespace gpulet {
namespace conv {

namespace {

// Epilogue shared by both kernels.  Accumulator register v of a lane holds row
// 8*(v/4) + 4*(lane/32) + v%4 and column lane%32 of its 32x32 tile.
template <int MT, int NT>
__device__ __forceinline__ void store_tile(const ConvParams &p, const f32x16 (&acc)[MT][NT], int m_base,
                                           int n_base, int lane) {
    const int frow = lane & 31, fhalf = lane >> 5;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int k = n_base + j * 32 + frow;
        if (k >= p.K) continue;
        const float bias = p.b ? p.b[k] : 0.f;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = m_base + i * 32 + 8 * (v >> 2) + 4 * fhalf + (v & 3);
                if (m >= p.M) continue;
                float val = acc[i][j][v] + bias;
                if (p.res) val += static_cast<float>(p.res[m * p.K + k]);
                if (p.relu) val = val > 0.f ? val : 0.f;
                p.y[m * p.ldy + p.y_off + k] = static_cast<__bf16>(val);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Main kernel: C % 8 == 0.  How an instance walks the depth (Depth): POINT = 1x1 filter
// without padding (no bounds tests at all; a strided 1x1 is pointwise too); TAPS = 64-channel
// blocks with the filter taps inside; LINEAR = (r, s, c), any C; MIXED = TAPS or LINEAR as the
// layer asks (launch groups).
//
// Staging uses buffer loads that write straight into LDS (no registers, no
// ds_write): one wavefront instruction moves 64 x 16 bytes into a contiguous
// 1 KB span = 8 tile rows of 128 bytes, lane i landing at byte 16*i.  The XOR
// swizzle is therefore applied on the global side: the lane that fills
// physical chunk q of row t fetches logical chunk q ^ swizzle(t).  Offsets
// past the buffer make the hardware write zeros (padding, ragged edges).
// NS LDS stages form a ring: while slice j is multiplied, slices j+1 .. j+NS-1
// are in flight.
// ---------------------------------------------------------------------------

enum class Depth { POINT, TAPS, LINEAR, MIXED };

// LDS elements of an instance: the ring, or the fp32 tile of the epilogue (rows padded by 8 floats).
constexpr int ring_elems(int bm, int bn, int ns, int spb) {
    return std::max(ns * spb * (bm + bn) * BK, bm * (bn + 8) * 2);
}
// Wavefronts per SIMD that the registers must leave room for: as many workgroups as LDS holds.  (At 84
// registers instead of 80 a CU held one 128x64 workgroup instead of two: 3x3 64 -> 64 on 56x56 at
// batch 32 19 -> 22.7 us.)
constexpr int waves_per_simd(int bm, int bn, int ns, int spb, int waves) {
    return std::min(8, std::max(1, 160 * 1024 / (ring_elems(bm, bn, ns, spb) * 2 + 512)) * waves / 4);
}

// Wavefronts are specialised.  The first CWM x CWN wavefronts ("consumers")
// only read LDS and issue MFMAs; the last NPROD wavefronts ("producers") only
// compute addresses and issue transfers.  A wavefront blocked on a saturated
// memory pipeline therefore never holds back matrix instructions.  Every ring
// step has one workgroup barrier: before it a producer waits for its own
// transfers of slice j, after it the stage slice j-1 occupied is free again.
// EXTRA: the layer has a second destination or a pooling side job (1x1 layers only); layers
// without either run the instance that knows of neither.
// SPLIT: the layer's depth is split over workgroups.
// MF: edge of the matrix instruction's tile.  SPB: depth slices per ring stage and barrier.  Launches
// whose tiles do not even fill the CUs are bound by the step from one barrier to the next, not by
// the matrix pipeline: the 32x32 tile takes two slices per barrier.
template <int BM, int BN, int CWM, int CWN, int NPROD, int NS, Depth DEPTH, bool EXTRA, bool SPLIT, int MF, int SPB>
__device__ __forceinline__ void conv_igemm_body(const ConvParams &p, const int bid) {
    constexpr int NCONS = CWM * CWN;
    constexpr int WM = BM / CWM, WN = BN / CWN;  // consumer wavefront tile
    constexpr int MT = WM / MF, NT = WN / MF;    // MFMA tiles per consumer
    static_assert(MT >= 1 && NT >= 1 && WM % MF == 0 && WN % MF == 0, "tile shape");
    typedef Mma<MF> MM;
    static_assert(NPROD == 2 || NPROD == 4, "swizzle key must not depend on the instruction index");
    constexpr int PROWS = NPROD * 8;                       // tile rows one round of producer instructions fills
    constexpr int AINS = BM / PROWS, BINS = BN / PROWS;    // transfers per producer lane and slice
    static_assert(BM % PROWS == 0 && BN % PROWS == 0, "tile rows per producer round");
    constexpr int SLICE = (BM + BN) * BK;                  // elements per depth slice: A rows, then B rows
    constexpr int STAGE = SLICE * SPB;                     // elements per LDS stage
    static_assert(NS >= 2 && (AINS + BINS) * SPB * (NS - 2) <= 63, "ring depth vs the 6-bit transfer counter");

    constexpr int LDT = BN + 8;  // padded row of the fp32 epilogue tile that reuses the ring
    __shared__ __attribute__((aligned(1024))) __bf16 ring[ring_elems(BM, BN, NS, SPB)];

    // Split-K: consecutive work items share an output tile and each takes a
    // contiguous range of depth slices.
    // Workgroups past the tiles carry the layer's side job, if it has one: a max pool of the same
    // input, which would otherwise be a launch of its own with nothing but fixed cost to it.
    // They are told apart inside the early exit that idle workgroups take anyway, so that a
    // workgroup with a tile does not wait for one more field of the argument block first.
    fetch_params(p);
    const int item = tile_of_block(p, bid);
    if (item >= p.n_tiles * (SPLIT ? p.split_k : 1) || bid >= p.tiles_per_xcd * 8) {
        if (EXTRA && bid >= p.tiles_per_xcd * 8 && p.side_blocks > 0) {
            const int idx = (bid - p.tiles_per_xcd * 8) * ((CWM * CWN + NPROD) * 64) + static_cast<int>(threadIdx.x);
            if (idx < p.side_pool.total) pool_max_item<3>(p.side_pool, idx);
        }
        return;
    }
    const int tile = SPLIT ? fdiv(item, p.d_split_k) : item, ks = SPLIT ? item - tile * p.split_k : 0;
    const int tm = fdiv(tile, p.d_tiles_n), tn = tile - tm * p.tiles_n;
    const int m0 = tm * BM, n0 = tn * BN;
    const BiasRegs bias_regs = load_bias<BN, (CWM * CWN + NPROD) * 64>(p, n0);
    // Small tiles, and tiles of which a CU holds only one workgroup, request the residual now as well.
    constexpr bool EARLY_RES = DEPTH == Depth::POINT && !EXTRA && !SPLIT &&
                               (BM * BN <= 64 * 64 || waves_per_simd(BM, BN, NS, SPB, CWM * CWN + NPROD) == (CWM * CWN + NPROD) / 4);
    auto pixel_of = [&](int row) { return m0 + row < p.M ? m0 + row : -1; };
    uint4 early[TileItems<BM, BN, (CWM * CWN + NPROD) * 64>::ITEMS];
    if constexpr (EARLY_RES) load_residual<BM, BN, (CWM * CWN + NPROD) * 64>(p, n0, early, pixel_of);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nk_all = (p.Kg + BK - 1) / BK;
    const int k_first = SPLIT ? ks * p.sps : 0;                      // first slice of this workgroup
    const int nk = SPLIT ? max(0, min(nk_all, k_first + p.sps) - k_first) : nk_all;  // slices of this workgroup
    const int nst = (nk + SPB - 1) / SPB;                            // ring stages they fill

    typename MM::Acc acc[MT][NT];  // consumers only

    if (wave >= NCONS) {
        // ------------------------------------------------------------ producer
        const int pw = wave - NCONS;
        const i32x4 rw = make_rsrc(p.w, p.w_bytes);
        const unsigned ring_lds = lds_addr(ring);

        // Instruction u of this wavefront fills tile rows u*PROWS + pw*8 .. +8;
        // this lane fills physical chunk lane&7 of row u*PROWS + lrow, i.e.
        // fetches logical chunk cc (the same for every u).
        const int lrow = pw * 8 + (lane >> 3);
        const int cc = (lane & 7) ^ ((lrow >> 1) & 7);

        // Byte offset of tap (0, 0) of each pixel row, counted from `before` bytes in front of x so
        // that it is never negative, and the pixel's top-left corner.
        const int before = ((p.pad * p.W + p.pad) * p.ldx * 2 + 255) & ~255;
        int a_off[AINS], a_h0[AINS], a_w0[AINS];
#pragma unroll
        for (int i = 0; i < AINS; ++i) {
            const int m = m0 + lrow + PROWS * i;
            if (m < p.M) {
                const int n = fdiv(m, p.d_pq);
                const int pq = m - n * (p.P * p.Q);
                const int pp = fdiv(pq, p.d_q), qq = pq - pp * p.Q;
                a_h0[i] = pp * p.stride - p.pad;
                a_w0[i] = qq * p.stride - p.pad;
                a_off[i] = (((n * p.H + a_h0[i]) * p.W + a_w0[i]) * p.ldx) * 2 + before;
            } else {
                a_h0[i] = -(1 << 28);  // fails every bounds test
                a_w0[i] = -(1 << 28);
                a_off[i] = static_cast<int>(OOB);
            }
        }
        unsigned b_off[BINS];
#pragma unroll
        for (int i = 0; i < BINS; ++i) {
            const int k = n0 + lrow + PROWS * i;
            b_off[i] = k < p.K ? static_cast<unsigned>((k * p.Kg + cc * CHUNK) * 2) : OOB;
        }

        // The transfers of one depth slice: lane offsets into x and w, the scalar offsets added to
        // them, the buffers.
        struct Slice {
            unsigned a[AINS], b[BINS];
            int xs, ws;
            i32x4 rx, rw;
        };
        // Starts the transfers of a slice into the LDS stage `at` bytes behind `base`.
        auto transfer = [&](const Slice &sl, unsigned base, const int at) {
#pragma unroll
            for (int i = 0; i < AINS; ++i) dma16(sl.rx, base, at + i * PROWS * (BK * 2), sl.a[i], sl.xs);
#pragma unroll
            for (int i = 0; i < BINS; ++i) dma16(sl.rw, base, at + (BM + i * PROWS) * (BK * 2), sl.b[i], sl.ws);
        };
        // Keeps the compiler from moving the computation of a slice behind the next barrier.
        auto settle = [&](Slice &sl) {
            asm volatile("" : "+s"(sl.xs), "+s"(sl.ws));
#pragma unroll
            for (int i = 0; i < AINS; ++i) asm volatile("" : "+v"(sl.a[i]));
        };
        // Walks the depth.  next(slice) works out the transfers of the next slice and advances the
        // depth position; slices past the end of the workgroup's share transfer zeros: they change no
        // sum (the second half of a stage of two slices), or nobody reads them.  Step j waits for
        // this lane's transfers of stage j (those of the NS-2 later stages may stay in flight),
        // meets everybody, and refills the LDS stage j-1 was read from with stage j+NS-1.  What it
        // refills with is worked out in front of the barrier, so that the transfers follow the
        // barrier at once; with two slices per barrier the consumers' reads of the stage want that
        // time (3x3 512 -> 512, 14x14, stride 2, batch 1: 8.5 us so, 8.8 the other way).
        //
        // Up to six transfers per lane and slice the loop is not unrolled: such tiles serve small
        // launches, which start with cold instruction caches and want short code.  From seven on
        // (128x128, 256x128, 192x128, 96x128, 128x32, 32x128) the producers' instructions count,
        // and the ring position is a compile-time constant in an unrolled body.  Rolled and unrolled:
        // 1x1 64 -> 256, 56x56, batch 32 in 96x128 26.0 and 25.6 us, in 128x128 17.1 and 17.0; 3x3
        // 256 -> 256, 56x56, batch 4 on 96 CUs in 96x128 37.9 and 37.6; 1x1 480 -> 24, 14x14, batch 32 in
        // 128x32 4.6 and 4.4; 1x1 1024 -> 256, 7x7, batch 5 in 32x128 5.4 and 5.0.
        auto run = [&](auto &&next) {
            unsigned base = ring_lds + pw * 8 * (BK * 2);
            Slice sl;
            if constexpr (AINS + BINS >= 7) {
                static_assert(SPB == 1, "the unrolled walk takes one slice per stage");
                auto issue = [&](int stage) {
                    transfer(sl, base, stage * STAGE * 2);
                    next(sl);
                };
                auto step = [&](int refill) {
                    settle(sl);
                    __builtin_amdgcn_s_waitcnt(vmcnt_imm((AINS + BINS) * (NS - 2)));
                    __syncthreads();
                    issue(refill);
                };
                next(sl);
#pragma unroll
                for (int i = 0; i < NS - 1; ++i) issue(i);
                int kt = 0;
                for (; kt + NS <= nst; kt += NS) {
#pragma unroll
                    for (int u = 0; u < NS; ++u) step((u + NS - 1) % NS);
                }
#pragma unroll
                for (int u = 0; u < NS - 1; ++u)
                    if (kt + u < nst) step((u + NS - 1) % NS);
            } else {
                constexpr bool EARLY = SPB == 1;
                const unsigned end = base + NS * STAGE * 2;
                if (EARLY) next(sl);
#pragma unroll 1
                for (int j = 1 - NS; j < nst; ++j) {
                    if (EARLY) {
                        settle(sl);
                        asm volatile("" : "+s"(base));
                    }
                    if (j >= 0) {
                        __builtin_amdgcn_s_waitcnt(vmcnt_imm((AINS + BINS) * SPB * (NS - 2)));
                        __syncthreads();
                    }
#pragma unroll
                    for (int h = 0; h < SPB; ++h) {
                        if (!EARLY) next(sl);
                        transfer(sl, base, h * SLICE * 2);
                        if (EARLY) next(sl);
                    }
                    base += STAGE * 2;
                    if (base == end) base -= NS * STAGE * 2;
                }
            }
        };

        // Whether tap t of a row lies outside the image: bit t of a mask, made once by repeating the
        // mask of valid filter columns for every valid filter row with one multiplication.  For
        // filters of up to 31 taps; bit 31 is always set.
        auto taps_outside = [&](unsigned (&out)[AINS]) {
            unsigned rows = 0;   // bit r * S of every filter row r
            for (int i = 0; i < p.R; ++i) rows |= 1u << (i * p.S);
#pragma unroll
            for (int i = 0; i < AINS; ++i) {
                const int r_lo = max(0, -a_h0[i]), r_hi = min(p.R, p.H - a_h0[i]);
                const int s_lo = max(0, -a_w0[i]), s_hi = min(p.S, p.W - a_w0[i]);
                unsigned in = 0;
                if (r_lo < r_hi && s_lo < s_hi && a_h0[i] > -(1 << 28))
                    in = ((1u << s_hi) - (1u << s_lo)) * (((rows & ((1u << (r_hi * p.S)) - 1u)) >> (r_lo * p.S)) << (r_lo * p.S));
                out[i] = ~in;
            }
        };

        // Depth orders.  Linear: (r, s, c) as the weights are stored.  Tap-inner (C a multiple of 64):
        // for each block of 64 channels all taps follow one another, so the image rows a workgroup
        // just fetched for one tap are fetched again for the next while they are still in the
        // nearest cache.  Both operands use the same order, so only the summation order of the
        // result changes.
        //
        // Tap-inner and 1x1: the depth position is the same for all lanes, so it travels as the
        // transfers' scalar offset and a lane's own offsets never change.  That leaves two vector
        // instructions per pixel row (one for 1x1, none per filter row) next to the transfer; with
        // one wavefront per SIMD these instructions bound small tiles (per-lane depth positions:
        // 0.15 us per slice of a 32x32 tile on 3x3 512 -> 512, 14x14, stride 2, against 0.06 for 1x1).
        if (DEPTH == Depth::POINT) {
            const i32x4 rx = make_rsrc(p.x, p.x_bytes);
            // Channels of this workgroup's slices: its share of a split depth ends before the layer's depth does.
            int left = SPLIT ? min(p.C - k_first * BK, nk * BK) : p.C;
            int soff = k_first * BK * 2;
            const int cc8 = cc * CHUNK;
            run([&](Slice &sl) {
                // lanes past the last channel, and all lanes past this workgroup's last slice, transfer zeros
                const unsigned past = cc8 < left ? 0u : OOB;
                sl.rx = rx;
                sl.rw = rw;
                sl.xs = sl.ws = left > 0 ? soff : 0;
#pragma unroll
                for (int i = 0; i < AINS; ++i) sl.a[i] = static_cast<unsigned>(a_off[i] + cc8 * 2) | past;
#pragma unroll
                for (int i = 0; i < BINS; ++i) sl.b[i] = b_off[i] | past;
                left -= BK;
                soff += BK * 2;
            });
        } else if (DEPTH == Depth::TAPS || (DEPTH == Depth::MIXED && p.tap_inner)) {
            // The hardware may subtract the scalar offset from the size before it compares: the size
            // covers the largest one (lanes whose tap is inside the image stay inside x by the mask).
            const unsigned x_size = p.x_bytes + before + (((p.R - 1) * p.W + p.S - 1) * p.ldx + p.C) * 2;
            const i32x4 rx = make_rsrc(reinterpret_cast<const char *>(p.x) - before, x_size);
            const int rs = p.R * p.S;
            const int cb = k_first / rs;
            int t = k_first - cb * rs, r = fdiv(t, p.d_s), s = t - r * p.S, c2 = cb * BK * 2;
            int xo = (r * p.W + s) * p.ldx * 2 + c2, wo = t * p.C * 2 + c2, left = nk;
#pragma unroll
            for (int i = 0; i < AINS; ++i) a_off[i] += cc * (CHUNK * 2);
            // offset(i): the offset of this lane's pixel row i, with the OOB bit where the tap lies outside
            auto walk = [&](auto &&offset) {
                run([&](Slice &sl) {
                    const bool ok = left > 0;
                    sl.rx = rx;
                    sl.rw = rw;
                    sl.rx[2] = ok ? static_cast<int>(x_size) : 0;   // past the last slice everything is out of range
                    sl.rw[2] = ok ? static_cast<int>(p.w_bytes) : 0;
                    sl.xs = ok ? xo : 0;
                    sl.ws = ok ? wo : 0;
#pragma unroll
                    for (int i = 0; i < AINS; ++i) sl.a[i] = offset(i);
#pragma unroll
                    for (int i = 0; i < BINS; ++i) sl.b[i] = b_off[i];
                    --left;
                    ++t;
                    wo += p.C * 2;
                    xo += p.ldx * 2;
                    if (++s == p.S) {
                        s = 0;
                        xo += (p.W - p.S) * p.ldx * 2;
                        if (++r == p.R) {
                            r = t = 0;
                            c2 += BK * 2;
                            xo = wo = c2;
                        }
                    }
                });
            };
            // The mask walk is laid out first (the other way round 3x3 512 -> 512, 14x14, stride 2, batch 1
            // takes 9.3 us instead of 9.0).  7x7 64 -> 64 on 28x28 at batch 8 with both tests 10.2 us, in the
            // order of the stored weights 11.0.
            if (__builtin_expect(rs < 32, 1)) {
                unsigned out[AINS];
                taps_outside(out);
                walk([&](int i) { return ((out[i] << (31 - t)) & OOB) | static_cast<unsigned>(a_off[i]); });
            } else {
                // more taps than a mask holds: both bounds tests for every tap
                walk([&](int i) {
                    const bool in = ((unsigned)(a_h0[i] + r) < (unsigned)p.H) & ((unsigned)(a_w0[i] + s) < (unsigned)p.W);
                    return in ? static_cast<unsigned>(a_off[i]) : OOB;
                });
            }
        } else {
            // Depth position of the chunk this lane fetches next: element index g, its filter tap
            // (r, s), channel c, and the tap's byte offset inside the image.  With dense pixels
            // (ldx == C) advancing s by one and c by -C leaves the address unchanged (a filter row
            // covers a contiguous span of the image row), so the offset only jumps when the filter
            // moves to its next row; when the layer reads a channel slice of wider pixels it also
            // skips ldx - C elements from one pixel to the next.
            const i32x4 rx = make_rsrc(p.x, p.x_bytes);
            int g = k_first * BK + cc * CHUNK, issued = 0;
            const int t = fdiv(g, p.d_c);
            int c = g - t * p.C, r = fdiv(t, p.d_s), s = t - r * p.S;
            int tap = ((r * p.W + s) * p.ldx + c) * 2 - before;
            auto issue_slice = [&](unsigned base) {
                const bool g_ok = issued < nk && g < p.Kg;
                base += pw * 8 * (BK * 2);
#pragma unroll
                for (int i = 0; i < AINS; ++i) {
                    const bool ok = g_ok & ((unsigned)(a_h0[i] + r) < (unsigned)p.H) & ((unsigned)(a_w0[i] + s) < (unsigned)p.W);
                    dma16(rx, base + i * PROWS * (BK * 2), ok ? static_cast<unsigned>(a_off[i] + tap) : OOB);
                }
                base += BM * (BK * 2);
#pragma unroll
                for (int i = 0; i < BINS; ++i) {
                    const unsigned off = g_ok ? b_off[i] + static_cast<unsigned>(g - cc * CHUNK) * 2u : OOB;
                    dma16(rw, base + i * PROWS * (BK * 2), off);
                }
                ++issued;
                g += BK;
                c += BK;
                tap += BK * 2;
                while (c >= p.C) {
                    c -= p.C;
                    tap += (p.ldx - p.C) * 2;  // nothing when the pixels are dense
                    if (++s == p.S) {
                        s = 0;
                        ++r;
                        tap += (p.W - p.S) * p.ldx * 2;
                    }
                }
            };
            // The ring position is a compile-time constant inside the unrolled body (rolled up like the
            // other orders, this one lost a fifth on 3x3 160 -> 320, 14x14, batch 32).
            auto issue_stage = [&](int stage) {
#pragma unroll
                for (int i = 0; i < SPB; ++i) issue_slice(ring_lds + (stage * STAGE + i * SLICE) * 2);
            };
#pragma unroll
            for (int i = 0; i < NS - 1; ++i) issue_stage(i);
            auto step = [&](int refill) {
                __builtin_amdgcn_s_waitcnt(vmcnt_imm((AINS + BINS) * SPB * (NS - 2)));
                __syncthreads();
                issue_stage(refill);
            };
            int kt = 0;
            for (; kt + NS <= nst; kt += NS) {
#pragma unroll
                for (int u = 0; u < NS; ++u) step((u + NS - 1) % NS);
            }
#pragma unroll
            for (int u = 0; u < NS - 1; ++u)
                if (kt + u < nst) step((u + NS - 1) % NS);
        }
        // Every transfer has landed before the ring is reused by the epilogue.
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    } else {
    // ---------------------------------------------------------------- consumer
    const int wy = wave / CWN, wx = wave - wy * CWN;
    const int frow = lane & (MF - 1);  // row of an MFMA operand this lane supplies
    const int fpart = lane / MF;       // which 8 of the depth elements of a step

#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int v = 0; v < MM::NV; ++v) acc[i][j][v] = 0.f;

    auto step = [&](int cur) {
        __syncthreads();
        constexpr int KS = BK / MM::KSTEP, CPS = MM::KSTEP / CHUNK;   // depth steps of a slice, chunks of a step
        if constexpr (MT * NT == 1) {
            // One matrix instruction per pair of fragment reads: the wavefront would wait out the
            // LDS latency before each of them.  All reads of the stage are issued first, and the
            // scheduling barrier keeps them there; each matrix instruction then waits only for its
            // own operands, and the compiler moves the next stage's barrier and reads up between
            // this stage's last matrix instructions.  (With more accumulators per wavefront the
            // extra fragment registers cost more than the latency: measured slower.)
            bf16x8 fa[SPB * KS], fb[SPB * KS];
#pragma unroll
            for (int i = 0; i < SPB * KS; ++i) {
                const __bf16 *sA = ring + cur * STAGE + (i / KS) * SLICE, *sB = sA + BM * BK;
                fa[i] = *reinterpret_cast<const bf16x8 *>(&sA[lds_pos(wy * WM + frow, (i % KS) * CPS + fpart)]);
                fb[i] = *reinterpret_cast<const bf16x8 *>(&sB[lds_pos(wx * WN + frow, (i % KS) * CPS + fpart)]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < SPB * KS; ++i) acc[0][0] = MM::mul(fa[i], fb[i], acc[0][0]);
        } else {
            static_assert(SPB == 1, "several slices per barrier: one accumulator tile per wavefront");
            const __bf16 *sA = ring + cur * STAGE, *sB = sA + BM * BK;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                bf16x8 fa[MT], fb[NT];
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    fa[i] = *reinterpret_cast<const bf16x8 *>(&sA[lds_pos(wy * WM + i * MF + frow, ks * CPS + fpart)]);
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    fb[j] = *reinterpret_cast<const bf16x8 *>(&sB[lds_pos(wx * WN + j * MF + frow, ks * CPS + fpart)]);
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j) acc[i][j] = MM::mul(fa[i], fb[j], acc[i][j]);
            }
        }
    };
    int kt = 0;
    for (; kt + NS <= nst; kt += NS) {
#pragma unroll
        for (int u = 0; u < NS; ++u) step(u);
    }
#pragma unroll
    for (int u = 0; u < NS - 1; ++u)
        if (kt + u < nst) step(u);

    }

    // ------------------------------------------------------------------ epilogue
    // The accumulators hold one column (channel) and 16 scattered rows per lane,
    // which would mean 2-byte stores.  They go through LDS instead: consumers
    // drop acc + bias as fp32 into the (now idle) ring, then every wavefront of
    // the workgroup picks up 8 consecutive channels of a pixel, adds the
    // residual, applies ReLU, rounds once to bf16 and stores 16 bytes.
    // Rows are padded by 8 floats so that lanes 32..63 (4 rows further down) use
    // the other half of the banks.
    float *stg = reinterpret_cast<float *>(ring);
    __syncthreads();  // all LDS reads of the main loop are done, all transfers have landed
    if (wave < NCONS) {
        const int wy = wave / CWN, wx = wave - wy * CWN;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int col = wx * WN + j * MF + (lane & (MF - 1));
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int v = 0; v < MM::NV; ++v) {
                    const int row = wy * WM + i * MF + MM::row(v, lane);
                    stg[row * LDT + col] = acc[i][j][v];
                }
        }
    }
    __syncthreads();
    constexpr int NTHR = (NCONS + NPROD) * 64;
    constexpr int VPR = BN / 8;  // 8-channel groups per tile row

    // Split-K: every workgroup but the last to arrive parks its partial tile in
    // scratch and leaves; the last one adds the others' tiles to its own, always
    // in split order so the sum does not depend on who came last.  Arrival is
    // counted with one atomic per workgroup; nobody ever waits.
    //
    // The dies' L2 caches are not coherent with one another, and a device-wide
    // fence would write back and invalidate a whole L2.  So the partial tiles and
    // the counter are accessed with device-scope (cache-bypassing) loads and
    // stores only, and a workgroup waits for its own stores to be acknowledged
    // before it counts itself in.
    if constexpr (SPLIT) {
        constexpr int DEVICE_SCOPE = 16;  // cache policy sc1: device scope, bypasses the die-local caches
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
            p.part, 0, p.n_tiles * p.split_k * (BM * BN * 4), RSRC_FLAGS);
        const int mine = (tile * p.split_k + ks) * (BM * BN * 4);  // byte offset of this workgroup's tile
        for (int it = threadIdx.x; it < BM * VPR; it += NTHR) {
            const int row = it / VPR, cv = it - row * VPR;
            const u32x4 lo = *reinterpret_cast<const u32x4 *>(&stg[row * LDT + cv * 8]);
            const u32x4 hi = *reinterpret_cast<const u32x4 *>(&stg[row * LDT + cv * 8 + 4]);
            __builtin_amdgcn_raw_buffer_store_b128(lo, rp, mine + (row * BN + cv * 8) * 4, 0, DEVICE_SCOPE);
            __builtin_amdgcn_raw_buffer_store_b128(hi, rp, mine + (row * BN + cv * 8 + 4) * 4, 0, DEVICE_SCOPE);
        }
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // this lane's partial-tile stores have reached memory
        __syncthreads();
        __shared__ unsigned arrived;
        if (threadIdx.x == 0) {
            arrived = __hip_atomic_fetch_add(&p.cnt[tile], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (arrived == static_cast<unsigned>(p.split_k - 1))  // ready for the next launch
                __hip_atomic_store(&p.cnt[tile], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (arrived != static_cast<unsigned>(p.split_k - 1)) return;
        const int base = tile * p.split_k * (BM * BN * 4);
        constexpr int ITEMS = (BM * VPR + NTHR - 1) / NTHR;  // 8-channel groups per thread
        float sum[ITEMS][8];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) sum[i][e] = 0.f;
        for (int q = 0; q < p.split_k; ++q) {
            u32x4 a[ITEMS], b[ITEMS];
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {  // all loads of one partial tile in flight together
                const int it = threadIdx.x + i * NTHR;
                const int row = it / VPR, cv = it - row * VPR;
                const int off = it < BM * VPR ? base + q * (BM * BN * 4) + (row * BN + cv * 8) * 4 : static_cast<int>(OOB);
                a[i] = __builtin_amdgcn_raw_buffer_load_b128(rp, off, 0, DEVICE_SCOPE);
                b[i] = __builtin_amdgcn_raw_buffer_load_b128(rp, off + 16, 0, DEVICE_SCOPE);
            }
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sum[i][e] += __uint_as_float(a[i][e]);
                    sum[i][4 + e] += __uint_as_float(b[i][e]);
                }
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int it = threadIdx.x + i * NTHR;
            if (it < BM * VPR) {
                const int row = it / VPR, cv = it - row * VPR;
#pragma unroll
                for (int e = 0; e < 8; ++e) stg[row * LDT + cv * 8 + e] = sum[i][e];
            }
        }
        // each thread re-reads only what it wrote itself, in the same iteration order
    }
    finish_tile<BM, BN, NTHR, EXTRA>(p, stg, n0, bias_regs, pixel_of, EARLY_RES ? early : nullptr);
}

template <int BM, int BN, int CWM, int CWN, int NPROD, int NS, Depth DEPTH, bool EXTRA, bool SPLIT, int MF, int SPB>
__global__ __launch_bounds__((CWM * CWN + NPROD) * 64, waves_per_simd(BM, BN, NS, SPB, CWM * CWN + NPROD)) void conv_igemm_kernel(const ConvParams p) {
    conv_igemm_body<BM, BN, CWM, CWN, NPROD, NS, DEPTH, EXTRA, SPLIT, MF, SPB>(p, blockIdx.x);
}

// Several independent layers in one launch (branches of an inception block, a projection
// shortcut next to the first layer of its block): each workgroup finds the layer its block
// index falls into and runs that layer's tile as above.  The general instance serves 1x1
// members too (its bounds tests always pass for them); when every member is 1x1 the instance
// without bounds tests is used.  Either way a member's results are the bits of its own launch.
template <int BM, int BN, int CWM, int CWN, int NPROD, int NS, Depth DEPTH, int MF, int SPB>
__global__ __launch_bounds__((CWM * CWN + NPROD) * 64, waves_per_simd(BM, BN, NS, SPB, CWM * CWN + NPROD)) void conv_igemm_group_kernel(const ConvGroup g) {
    const int b = blockIdx.x;
    // The lines of every member's block are requested with the table of first workgroups: which member it is decides
    // only what is read from the scalar cache then.
#pragma unroll
    for (int i = 0; i < MAX_GROUP; ++i)
        asm volatile("" ::"s"(g.p[i].x), "s"(g.p[i].S), "s"(g.p[i].x_bytes), "s"(g.p[i].d_s.mul), "s"(g.first[i]));
    int j = 0;
#pragma unroll
    for (int i = 1; i < MAX_GROUP; ++i)
        if (b >= g.first[i]) j = i;
    conv_igemm_body<BM, BN, CWM, CWN, NPROD, NS, DEPTH, false, false, MF, SPB>(g.p[j], b - g.first[j]);
}

// ---------------------------------------------------------------------------
// Any channel count: every element of a chunk is decoded and loaded on its own.
// Used by the image stems (C = 3) and LeNet (C = 1, 6); one slice of prefetch.
// ---------------------------------------------------------------------------
template <int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(NTHREADS) void conv_igemm_any_kernel(const ConvParams p) {
    static_assert(WGM * WGN == 4, "four wavefronts per workgroup");
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int MT = WM / 32, NT = WN / 32;
    constexpr int AROWS = BM / 32, BROWS = BN / 32;

    __shared__ __attribute__((aligned(16))) __bf16 sA[2][BM * BK];
    __shared__ __attribute__((aligned(16))) __bf16 sB[2][BN * BK];

    const int tile = tile_of_block(p);
    if (tile >= p.n_tiles) return;
    const int tm = tile / p.tiles_n, tn = tile - tm * p.tiles_n;
    const int m0 = tm * BM, n0 = tn * BN;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wy = wave / WGN, wx = wave - wy * WGN;
    const int cc = tid & 7;
    const int lrow = tid >> 3;

    int a_base[AROWS], a_h0[AROWS], a_w0[AROWS];
#pragma unroll
    for (int i = 0; i < AROWS; ++i) {
        const int m = m0 + lrow + 32 * i;
        if (m < p.M) {
            const int n = m / (p.P * p.Q);
            const int pq = m - n * (p.P * p.Q);
            const int pp = pq / p.Q, qq = pq - pp * p.Q;
            a_h0[i] = pp * p.stride - p.pad;
            a_w0[i] = qq * p.stride - p.pad;
            a_base[i] = ((n * p.H + a_h0[i]) * p.W + a_w0[i]) * p.ldx;
        } else {
            a_h0[i] = -(1 << 28);
            a_w0[i] = -(1 << 28);
            a_base[i] = 0;
        }
    }
    int b_base[BROWS];
    bool b_ok[BROWS];
#pragma unroll
    for (int i = 0; i < BROWS; ++i) {
        const int k = n0 + lrow + 32 * i;
        b_ok[i] = k < p.K;
        b_base[i] = (b_ok[i] ? k : 0) * p.Kg;
    }

    uint4 ra[AROWS], rb[BROWS];
    const unsigned short *xs = reinterpret_cast<const unsigned short *>(p.x);
    const unsigned short *ws = reinterpret_cast<const unsigned short *>(p.w);

    auto load_slice = [&](int kt) {
        const int g0 = kt * BK + cc * CHUNK;
        int rs = g0 / p.C;
        int c = g0 - rs * p.C;
        int r = rs / p.S, s = rs - r * p.S;
        unsigned short ea[AROWS][CHUNK], eb[BROWS][CHUNK];
#pragma unroll
        for (int e = 0; e < CHUNK; ++e) {
            const bool g_ok = g0 + e < p.Kg;
            const int tap = (r * p.W + s) * p.ldx + c;
#pragma unroll
            for (int i = 0; i < AROWS; ++i) {
                const bool ok = g_ok && (unsigned)(a_h0[i] + r) < (unsigned)p.H &&
                                (unsigned)(a_w0[i] + s) < (unsigned)p.W;
                ea[i][e] = ok ? xs[a_base[i] + tap] : (unsigned short)0;
            }
#pragma unroll
            for (int i = 0; i < BROWS; ++i)
                eb[i][e] = (g_ok && b_ok[i]) ? ws[b_base[i] + g0 + e] : (unsigned short)0;
            if (++c == p.C) {
                c = 0;
                if (++s == p.S) {
                    s = 0;
                    ++r;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < AROWS; ++i)
            ra[i] = make_uint4(ea[i][0] | ((unsigned)ea[i][1] << 16), ea[i][2] | ((unsigned)ea[i][3] << 16),
                               ea[i][4] | ((unsigned)ea[i][5] << 16), ea[i][6] | ((unsigned)ea[i][7] << 16));
#pragma unroll
        for (int i = 0; i < BROWS; ++i)
            rb[i] = make_uint4(eb[i][0] | ((unsigned)eb[i][1] << 16), eb[i][2] | ((unsigned)eb[i][3] << 16),
                               eb[i][4] | ((unsigned)eb[i][5] << 16), eb[i][6] | ((unsigned)eb[i][7] << 16));
    };

    auto store_slice = [&](int buf) {
#pragma unroll
        for (int i = 0; i < AROWS; ++i) *reinterpret_cast<uint4 *>(&sA[buf][lds_pos(lrow + 32 * i, cc)]) = ra[i];
#pragma unroll
        for (int i = 0; i < BROWS; ++i) *reinterpret_cast<uint4 *>(&sB[buf][lds_pos(lrow + 32 * i, cc)]) = rb[i];
    };

    f32x16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const int nk = (p.Kg + BK - 1) / BK;
    const int frow = lane & 31, fhalf = lane >> 5;

    load_slice(0);
    store_slice(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) load_slice(kt + 1);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            bf16x8 fa[MT], fb[NT];
#pragma unroll
            for (int i = 0; i < MT; ++i)
                fa[i] = *reinterpret_cast<const bf16x8 *>(&sA[buf][lds_pos(wy * WM + i * 32 + frow, ks * 2 + fhalf)]);
#pragma unroll
            for (int j = 0; j < NT; ++j)
                fb[j] = *reinterpret_cast<const bf16x8 *>(&sB[buf][lds_pos(wx * WN + j * 32 + frow, ks * 2 + fhalf)]);
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < nk) store_slice(buf ^ 1);
        __syncthreads();
    }

    store_tile<MT, NT>(p, acc, m0 + wy * WM, n0 + wx * WN, lane);
}

// CWM x CWN consumers and NPROD producers for the main kernel; the scalar-gather
// kernel always runs four wavefronts as WGM x WGN.
template <int BM, int BN, int CWM, int CWN, int NPROD, int NS, int WGM, int WGN, int MF = 32, int SPB = 1>
hipError_t launch_tile(ConvParams p, bool vec, int split_k, hipStream_t stream) {
    const int tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.K + BN - 1) / BN;
    p.n_tiles = tiles_m * p.tiles_n;
    const int nk = (p.Kg + BK - 1) / BK;
    p.split_k = vec ? split_k : 1;
    p.d_tiles_n = make_fastdiv(p.tiles_n);
    p.d_split_k = make_fastdiv(p.split_k);
    p.sps = (nk + p.split_k - 1) / p.split_k;
    p.tiles_per_xcd = (p.n_tiles * p.split_k + 7) / 8;  // work items per die
    const bool pointwise = p.R == 1 && p.S == 1 && p.pad == 0;
    constexpr int THREADS = (CWM * CWN + NPROD) * 64;
    p.side_blocks = (vec && pointwise && p.side_pool.y) ? (p.side_pool.total + THREADS - 1) / THREADS : 0;
    if (p.side_pool.y && !p.side_blocks) return hipErrorInvalidValue;  // nobody would compute the pool
    const dim3 grid(static_cast<unsigned>(p.tiles_per_xcd * 8 + p.side_blocks));
    const dim3 block(THREADS);
    if constexpr (BM < 64 && BN < 64) {
        if (!vec) return hipErrorInvalidValue;   // the scalar-gather kernel has no such tile
    }
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, stream, p); };
    const bool split = p.split_k > 1;
    if (vec && pointwise && (p.side_blocks > 0 || p.k2 < p.K))
        split ? go(conv_igemm_kernel<BM, BN, CWM, CWN, NPROD, NS, Depth::POINT, true, true, MF, SPB>)
              : go(conv_igemm_kernel<BM, BN, CWM, CWN, NPROD, NS, Depth::POINT, true, false, MF, SPB>);
    else if (vec && pointwise)
        split ? go(conv_igemm_kernel<BM, BN, CWM, CWN, NPROD, NS, Depth::POINT, false, true, MF, SPB>)
              : go(conv_igemm_kernel<BM, BN, CWM, CWN, NPROD, NS, Depth::POINT, false, false, MF, SPB>);
    else if (vec && p.tap_inner)
        split ? go(conv_igemm_kernel<BM, BN, CWM, CWN, NPROD, NS, Depth::TAPS, false, true, MF, SPB>)
              : go(conv_igemm_kernel<BM, BN, CWM, CWN, NPROD, NS, Depth::TAPS, false, false, MF, SPB>);
    else if (vec)
        split ? go(conv_igemm_kernel<BM, BN, CWM, CWN, NPROD, NS, Depth::LINEAR, false, true, MF, SPB>)
              : go(conv_igemm_kernel<BM, BN, CWM, CWN, NPROD, NS, Depth::LINEAR, false, false, MF, SPB>);
    else if constexpr (BM >= 64 || BN >= 64)
        hipLaunchKernelGGL((conv_igemm_any_kernel<BM, BN, WGM, WGN>), grid, dim3(NTHREADS), 0, stream, p);
    return hipGetLastError();
}

template <int BM, int BN, int CWM, int CWN, int NPROD, int NS, int MF = 32, int SPB = 1>
hipError_t launch_group_tile(const ConvParams *ps, int n, hipStream_t stream) {
    ConvGroup g;
    int blocks = 0;
    bool pointwise = true;
    for (int j = 0; j < n; ++j) pointwise = pointwise && ps[j].R == 1 && ps[j].S == 1 && ps[j].pad == 0;
    for (int j = 0; j < MAX_GROUP; ++j) {
        g.first[j] = j < n ? blocks : INT_MAX;
        g.p[j] = ps[j < n ? j : 0];
        if (j >= n) continue;
        ConvParams &p = g.p[j];
        const int tiles_m = (p.M + BM - 1) / BM;
        p.tiles_n = (p.K + BN - 1) / BN;
        p.n_tiles = tiles_m * p.tiles_n;
        p.split_k = 1;
        p.d_tiles_n = make_fastdiv(p.tiles_n);
        p.d_split_k = make_fastdiv(1);
        p.sps = (p.Kg + BK - 1) / BK;
        p.tiles_per_xcd = (p.n_tiles + 7) / 8;
        p.side_blocks = 0;
        blocks += p.tiles_per_xcd * 8;
    }
    g.first[MAX_GROUP] = INT_MAX;
    const dim3 grid(static_cast<unsigned>(blocks)), block((CWM * CWN + NPROD) * 64);
    if (pointwise)
        hipLaunchKernelGGL((conv_igemm_group_kernel<BM, BN, CWM, CWN, NPROD, NS, Depth::POINT, MF, SPB>), grid, block, 0, stream, g);
    else
        hipLaunchKernelGGL((conv_igemm_group_kernel<BM, BN, CWM, CWN, NPROD, NS, Depth::MIXED, MF, SPB>), grid, block, 0, stream, g);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_igemm_group(const ConvParams *p, int n, int tile, bool two_stage, hipStream_t stream) {
    if (n < 2 || n > MAX_GROUP) return hipErrorInvalidValue;
    switch (tile) {
        case 0:
            if (two_stage) return launch_group_tile<128, 128, 4, 2, 4, 2>(p, n, stream);
            return launch_group_tile<128, 128, 4, 2, 4, 3>(p, n, stream);
        case 1: return launch_group_tile<128, 64, 4, 2, 4, 3>(p, n, stream);
        case 2: return launch_group_tile<64, 128, 2, 4, 4, 3>(p, n, stream);
        case 3: return launch_group_tile<64, 64, 2, 2, 4, 3>(p, n, stream);
        case 4: return launch_group_tile<128, 32, 4, 1, 2, 3>(p, n, stream);
        case 5: return launch_group_tile<32, 128, 1, 4, 2, 3>(p, n, stream);
        case 12: return launch_group_tile<192, 128, 2, 4, 4, 3>(p, n, stream);
        case 13: return launch_group_tile<96, 128, 1, 4, 4, 3>(p, n, stream);
        case 14: return launch_group_tile<32, 32, 2, 2, 4, 3, 16, 2>(p, n, stream);
        default: return launch_group_tile<256, 128, 4, 2, 4, 3>(p, n, stream);
    }
}

hipError_t launch_igemm(const ConvParams &p, bool vec, int tile, int split_k, bool two_stage, hipStream_t stream) {
    switch (tile) {
        case 0:
            // With more tiles than CUs, a two-stage ring (64 KB, two workgroups per CU, one's loads
            // overlapping the other's epilogue) beats the deeper prefetch of three stages.
            if (two_stage && split_k == 1) return launch_tile<128, 128, 4, 2, 4, 2, 2, 2>(p, vec, 1, stream);
            return launch_tile<128, 128, 4, 2, 4, 3, 2, 2>(p, vec, split_k, stream);
        case 1: return launch_tile<128, 64, 4, 2, 4, 3, 2, 2>(p, vec, split_k, stream);
        case 2: return launch_tile<64, 128, 2, 4, 4, 3, 2, 2>(p, vec, split_k, stream);
        case 3: return launch_tile<64, 64, 2, 2, 4, 3, 2, 2>(p, vec, split_k, stream);
        case 4: return launch_tile<128, 32, 4, 1, 2, 3, 4, 1>(p, vec, split_k, stream);
        case 5: return launch_tile<32, 128, 1, 4, 2, 3, 1, 4>(p, vec, split_k, stream);
        // three row tiles per consumer (96 pixels x 32 filters); the scalar-gather variant has no such
        // instance and takes the nearest shape
        case 12:
            if (!vec) return launch_tile<256, 128, 4, 2, 4, 3, 2, 2>(p, vec, split_k, stream);
            return launch_tile<192, 128, 2, 4, 4, 3, 2, 2>(p, vec, split_k, stream);
        case 13:
            if (!vec) return launch_tile<128, 128, 4, 2, 4, 3, 2, 2>(p, vec, split_k, stream);
            return launch_tile<96, 128, 1, 4, 4, 3, 2, 2>(p, vec, split_k, stream);
        // the scalar-gather variant has no 32x32 either: 64x64 stands in.  Chosen for it all the same, since it
        // beats what the cost formula would name next (100 -> 16, 5x5, 28x28, batch 29: 119.6 us, 128x64 168).
        case 14:
            if (!vec) return launch_tile<64, 64, 2, 2, 4, 3, 2, 2>(p, vec, split_k, stream);
            return launch_tile<32, 32, 2, 2, 4, 3, 2, 2, 16, 2>(p, vec, split_k, stream);
        case kTile16: return launch_tile<16, 16, 1, 1, 2, 3, 2, 2, 16, 4>(p, vec, split_k, stream);
        default: return launch_tile<256, 128, 4, 2, 4, 3, 2, 2>(p, vec, split_k, stream);
    }
}

}  // namespace conv
}  // namespace gpulet
