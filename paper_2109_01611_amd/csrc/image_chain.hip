// A run of consecutive small layers of a model as one launch, one workgroup per image.
//
// Models as small as LeNet-5 are nothing but launches: seven kernels of 2.5-7 us for layers whose
// arithmetic takes a fraction of a microsecond, each waiting for the one before.  Where every tensor
// of an image fits in LDS, a workgroup takes its image through the whole run: the input and the
// filters are staged once, every layer reads the tensor the one before left in LDS, and a workgroup
// barrier takes the place of a kernel boundary.  Tensors are still stored to their buffers (nobody
// waits for these stores), so the workspace holds what separate launches leave in it.
//
// Bound: the chain of barriers and latencies of one image; matrix cores and LDS are mostly idle.  16
// wavefronts, because only other wavefronts hide those latencies.  Weights of fully connected layers come
// to LDS by transfers while earlier layers run: fetched as matrix fragments, 64 bytes of a row at a time,
// they kept the load path busy for 2.7 us per layer.  LeNet-5 on 256 CUs, seven launches and one: 1 image 24.1
// and 12.4 us a pass, 32 images 29.2 and 12.8, 512 images 68 and 24, 2048 images 187 and 90; on 64 CUs 2048 images
// 642 and 349.  (Stamps at 15.3 us, when 101 spilled scalar registers still cost the convolutions 2.5: 1.2 until the
// arguments are there, 2 until the image and the filters are, 3.1 and 1.2 the convolutions, 1 and 0.6 the pools, 1.3
// each fully connected layer.)
//
// Every layer adds its products in the order of the kernel that runs it alone (convolution: depth
// as stored, or 64-channel blocks with the taps inside where that kernel walks so; fully connected:
// four quarters of the depth, added in order), so the results have the same bits.
#include <algorithm>
#include <cmath>

#include "conv_common.h"

namespace gpulet {

using namespace conv;

namespace {

constexpr int kWaves = 16, kThreads = kWaves * 64;
constexpr int kMaxSteps = 8;                  // depth steps of 32 a convolution holds in registers: Kg <= 256
constexpr int kFcSteps = 4;                   // depth steps of a fully connected layer read together
constexpr int kLdsBytes = 152 * 1024;         // tensors, weights, tables and partial sums of an image
constexpr long long kConvMacs = 4 << 20;      // per image and layer: the largest that image_chain_pays was fitted to

// Something in memory that transfers copy to LDS: `bytes` at `from` to LDS offset `to`.  A wavefront's last
// transfer may pass the end: it fills LDS with zeros up to a multiple of kPiece.
constexpr int kPiece = 1024, kBiasPiece = 256;
struct Staged {
    const void *from;
    int bytes, to;
};

struct ChainOp {
    void *y;            // destination of the batch, or null: the tensor is not wanted in memory
    int kind, C, H, W, K, P, Q, S, stride, pad, relu, out_fp32;
    int src, src_w;     // LDS byte offset of the source tensor, pixels per stored row (the border included)
    int dst_0, dst_w;   // the destination's first pixel inside its border, pixels per stored row
    int weights, table, bias;   // LDS byte offsets of the staged weights, the chunk table and the bias
    int zeros;          // LDS byte offset of a chunk of zeros
    int Kg, chunks, taps;       // depth in elements and in 16-byte chunks, taps of a filter
    FastDiv d_q, d_cv, d_kv, d_s, d_rs;   // by Q, C / 8, K / 8, S, R * S
};

struct ChainParams {
    const __bf16 *x;
    int n_ops, lds_tensors;    // bytes that hold tensors (cleared first: borders and tails read as zeros)
    int in_row, in_rows;       // 16-byte chunks per image row, rows of the input
    int in_border, in_edge;    // border in rows, in chunks of a row
    int in_wide, in_chunks;    // chunks per row with the border, of all rows with the border
    int partial;               // LDS byte offset of the partial sums of the fully connected layers
    FastDiv d_in_wide;
    // What is copied to LDS at once, while the first layer runs, and behind the second layer (over the first two
    // tensors).  The last two hold weights of fully connected layers.
    int n_bias, n_first, n_second, n_third;
    Staged bias[kMaxChain], first[kMaxChain], second[kMaxChain], third[kMaxChain];
    ChainOp op[kMaxChain];
};

// What a layer needs of its description, in one round trip to the scalar cache: read where they are needed, the fields
// would be half a dozen dependent loads of a few hundred cycles each in front of every layer.  No more than that: the
// whole description, or two of them, does not fit the scalar registers, and the spills cost the convolutions 1-2 us.
#define FETCH_CONV(o) \
    asm volatile("" ::"s"((o).C), "s"((o).K), "s"((o).P), "s"((o).Q), "s"((o).stride), "s"((o).relu), "s"((o).src), "s"((o).src_w), \
                 "s"((o).dst_0), "s"((o).dst_w), "s"((o).weights), "s"((o).table), "s"((o).bias), "s"((o).Kg), "s"((o).chunks), \
                 "s"((o).d_q.mul), "s"((o).d_q.shift))
#define FETCH_POOL(o) \
    asm volatile("" ::"s"((o).C), "s"((o).H), "s"((o).W), "s"((o).P), "s"((o).Q), "s"((o).stride), "s"((o).pad), "s"((o).src), \
                 "s"((o).src_w), "s"((o).dst_0), "s"((o).dst_w), "s"((o).d_q.mul), "s"((o).d_q.shift), "s"((o).d_cv.mul), "s"((o).d_cv.shift))
#define FETCH_FC(o) \
    asm volatile("" ::"s"((o).K), "s"((o).Kg), "s"((o).src), "s"((o).weights), "s"((o).zeros), "s"((o).bias), "s"((o).dst_0), \
                 "s"((o).relu), "s"((o).out_fp32))

// Barrier between layers: LDS is all they share, so nobody waits for memory.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Convolution: 16 filters x 16 pixels per wavefront and item, the product taken as filters x pixels so
// that a lane ends with four consecutive channels of the pixel whose fragments it supplied: one division
// and one 8-byte store per item.  The weights of 16 filters stay in the wavefront's registers for all of
// its pixel tiles.  Instruction issue bounds this loop (four wavefronts per SIMD, depths of a few hundred).
template <int STEPS>   // depth steps of 32
__device__ __forceinline__ void chain_conv(const ChainOp &g, char *lds, int wave, int lane) {
    const ChainOp o = g;
    FETCH_CONV(o);
    const int sub = lane & 15, kq = lane >> 4;
    const int M = o.P * o.Q, m_tiles = (M + 15) / 16;
    const int px_step = o.stride * o.C * 2, row_step = o.src_w * px_step;
    const int2 *table = reinterpret_cast<const int2 *>(lds + o.table);
    const unsigned limit = relu_limit(o.relu);
    for (int k0 = 0; k0 < o.K; k0 += 16) {
        bf16x8 fw[STEPS];
        int xo[STEPS], in[STEPS];
        const int wrow = o.weights + min(k0 + sub, o.K - 1) * o.Kg * 2;
        // no branch for chunks past the depth: they multiply zeros by zeros
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int c = s * 4 + kq;
            const int2 e = table[c];
            in[s] = c < o.chunks ? 1 : 0;
            xo[s] = e.x;
            fw[s] = *reinterpret_cast<const bf16x8 *>(lds + __mul24(in[s], wrow) + e.y);
        }
        const int k = k0 + kq * 4;
        const float4 bias = *reinterpret_cast<const float4 *>(lds + o.bias + min(k, o.K - 4) * 4);
        for (int mt = wave; mt < m_tiles; mt += kWaves) {
            const int m = min(mt * 16 + sub, M - 1);
            const int p = fdiv(m, o.d_q), q = m - p * o.Q;
            const int px = o.src + p * row_step + q * px_step;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            bf16x8 fx[STEPS];
#pragma unroll
            for (int s = 0; s < STEPS; ++s)
                fx[s] = *reinterpret_cast<const bf16x8 *>(lds + (__mul24(in[s], px) + xo[s]));
            __builtin_amdgcn_sched_barrier(0);   // all reads first: left alone, each waits for the product before
#pragma unroll
            for (int s = 0; s < STEPS; ++s) acc = Mma<16>::mul(fw[s], fx[s], acc);
            if (mt * 16 + sub < M && k < o.K) {
                const uint2 v = make_uint2(relu_or_pass(pack_bf16(acc[0] + bias.x, acc[1] + bias.y), limit),
                                           relu_or_pass(pack_bf16(acc[2] + bias.z, acc[3] + bias.w), limit));
                *reinterpret_cast<uint2 *>(lds + o.dst_0 + ((p * o.dst_w + q) * o.K + k) * 2) = v;
            }
        }
    }
}

// Max pool: 8 channels of one output pixel per thread, window coordinates clamped to the image,
// maximum on order-preserving integer keys (as pool_max_item).
template <int S>
__device__ __forceinline__ void chain_pool(const ChainOp &g, char *lds) {
    const ChainOp o = g;
    FETCH_POOL(o);
    const int cv = o.C / 8, items = o.P * o.Q * cv;
    for (int it = threadIdx.x; it < items; it += kThreads) {
        const int m = fdiv(it, o.d_cv), c8 = it - m * cv;
        const int p = fdiv(m, o.d_q), q = m - p * o.Q;
        const int h0 = p * o.stride - o.pad, w0 = q * o.stride - o.pad;
        const char *src = lds + o.src + c8 * 16;
        uint4 v[S * S];
#pragma unroll
        for (int r = 0; r < S; ++r) {
            const int row = min(max(h0 + r, 0), o.H - 1) * o.src_w;
#pragma unroll
            for (int s = 0; s < S; ++s)
                v[r * S + s] = *reinterpret_cast<const uint4 *>(src + (row + min(max(w0 + s, 0), o.W - 1)) * o.C * 2);
        }
        unsigned best[4];
#pragma unroll
        for (int t = 0; t < S * S; ++t) {
            const unsigned u[4] = {v[t].x, v[t].y, v[t].z, v[t].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned key = bf16_pair_order_key(u[i]);
                best[i] = t == 0 ? key : max_keys(best[i], key);
            }
        }
        *reinterpret_cast<uint4 *>(lds + o.dst_0 + ((p * o.dst_w + q) * o.C + c8 * 8) * 2) =
            make_uint4(bf16_pair_order_key(best[0]), bf16_pair_order_key(best[1]), bf16_pair_order_key(best[2]),
                       bf16_pair_order_key(best[3]));
    }
}

// Fully connected: an item is a quarter of the depth of 16 outputs, kFcSteps steps of it at a time.  Outputs,
// steps and elements that do not exist read zeros.
template <int VEC>   // elements per aligned read of a weight row
__device__ __forceinline__ void chain_fc(const ChainOp &o, char *lds, float *partial, int wave, int lane) {
    const int steps = (o.Kg + 31) / 32, quarter = (steps + 3) / 4;
    const int items = 4 * ((o.K + 15) / 16);
    for (int it = wave; it < items; it += kWaves) {
        const int out = (it >> 2) * 16 + (lane & 15);
        const int row = o.weights + out * o.Kg * 2;
        const int s0 = (it & 3) * quarter, s1 = min(steps, s0 + quarter);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int s = s0; s < s1; s += kFcSteps) {
            bf16x8 w[kFcSteps], x[kFcSteps];
#pragma unroll
            for (int u = 0; u < kFcSteps; ++u) {
                const int k = (s + u) * 32 + (lane >> 4) * 8;
                // all 16 rows of the instruction read the image, only the first matters; the source tensor ends
                // in zeros up to a multiple of 32 elements
                x[u] = *reinterpret_cast<const bf16x8 *>(lds + (s + u < s1 ? o.src + k * 2 : o.zeros));
                const bool live = s + u < s1 && out < o.K;
                if constexpr (VEC == 8) {
                    w[u] = *reinterpret_cast<const bf16x8 *>(lds + (live && k < o.Kg ? row + k * 2 : o.zeros));
                } else if constexpr (VEC == 4) {
                    const uint2 lo = *reinterpret_cast<const uint2 *>(lds + (live && k < o.Kg ? row + k * 2 : o.zeros));
                    const uint2 hi = *reinterpret_cast<const uint2 *>(lds + (live && k + 4 < o.Kg ? row + k * 2 + 8 : o.zeros));
                    const uint4 v = make_uint4(lo.x, lo.y, hi.x, hi.y);
                    w[u] = *reinterpret_cast<const bf16x8 *>(&v);
                } else {
                    unsigned e[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const char *lo = lds + (live && k + 2 * i < o.Kg ? row + (k + 2 * i) * 2 : o.zeros);
                        const char *hi = lds + (live && k + 2 * i + 1 < o.Kg ? row + (k + 2 * i + 1) * 2 : o.zeros);
                        e[i] = *reinterpret_cast<const unsigned short *>(lo) |
                               (static_cast<unsigned>(*reinterpret_cast<const unsigned short *>(hi)) << 16);
                    }
                    const uint4 v = make_uint4(e[0], e[1], e[2], e[3]);
                    w[u] = *reinterpret_cast<const bf16x8 *>(&v);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < kFcSteps; ++u) acc = Mma<16>::mul(x[u], w[u], acc);
        }
        if (lane < 16) partial[it * 16 + lane] = acc[0];
    }
}

__device__ __forceinline__ void stage(const Staged &e, char *lds, int wave, int lane) {
    const i32x4 r = make_rsrc(e.from, static_cast<unsigned>(e.bytes));
    for (int at = wave * kPiece; at < e.bytes; at += kWaves * kPiece)
        dma16(r, lds_addr(lds) + e.to + at, static_cast<unsigned>(at + lane * 16));
}

// The same for fp32 values whose address is a multiple of 4 only: 64 of them per wavefront.
__device__ __forceinline__ void stage_bias(const Staged &e, char *lds, int wave, int lane) {
    const i32x4 r = make_rsrc(e.from, static_cast<unsigned>(e.bytes));
    if (wave * kBiasPiece < e.bytes)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                     :
                     : "s"(lds_addr(lds) + e.to + wave * kBiasPiece), "v"(wave * kBiasPiece + lane * 4), "s"(r)
                     : "memory");
}

__global__ __launch_bounds__(kThreads) void image_chain_kernel(const ChainParams c) {
    __shared__ __attribute__((aligned(1024))) char lds[kLdsBytes];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int img = blockIdx.x;

    // The argument block in one round trip: a scalar load of a line that is not cached costs several hundred
    // nanoseconds, and the loops below would meet one after the other.
#pragma unroll
    for (int i = 0; i < kMaxChain; ++i) {
        asm volatile("" ::"s"(c.op[i].y), "s"(c.op[i].W), "s"(c.op[i].src), "s"(c.op[i].d_cv.mul), "s"(c.op[i].d_rs.shift));
        asm volatile("" ::"s"(c.bias[i].bytes), "s"(c.first[i].bytes), "s"(c.second[i].bytes), "s"(c.third[i].bytes));
    }

    // Everything from memory that the layers wait for, requested at once: this thread's chunk of the padded image,
    // then bias and weights, which land in LDS by themselves.
    const uint4 *x = reinterpret_cast<const uint4 *>(c.x) + static_cast<size_t>(img) * (c.in_rows * c.in_row);
    auto in_chunk = [&](int j) {   // chunk j of the image with its border of zeros
        const int r = fdiv(j, c.d_in_wide) - c.in_border, q = j - (r + c.in_border) * c.in_wide - c.in_edge;
        const bool inside = static_cast<unsigned>(r) < static_cast<unsigned>(c.in_rows) &&
                            static_cast<unsigned>(q) < static_cast<unsigned>(c.in_row);
        return inside ? x[r * c.in_row + q] : make_uint4(0u, 0u, 0u, 0u);
    };
    const uint4 x0 = in_chunk(tid);
#pragma unroll 1
    for (int i = 0; i < c.n_bias; ++i) stage_bias(c.bias[i], lds, wave, lane);
#pragma unroll 1
    for (int i = 0; i < c.n_first; ++i) stage(c.first[i], lds, wave, lane);

    // All other tensors start as zeros: their borders and tails stay so.
    for (int at = c.in_chunks * 16 + tid * 16; at < c.lds_tensors; at += kThreads * 16)
        *reinterpret_cast<uint4 *>(lds + at) = make_uint4(0u, 0u, 0u, 0u);
    // Where each 16-byte chunk of a layer's depth lies in the source tensor (from a pixel's first tap) and in a
    // filter; for chunks past the depth, where zeros lie.
    for (int i = 0; i < c.n_ops; ++i) {
        const ChainOp &o = c.op[i];
        if (o.kind != GPULET_OP_CONV || tid >= kMaxSteps * 4) continue;
        int2 e = make_int2(o.zeros, o.zeros);
        if (tid < o.chunks) {
            int tap, c8;
            if (o.C % BK == 0) {    // 64-channel blocks outermost, taps inside
                const int t = tid >> 3, block = fdiv(t, o.d_rs);
                tap = t - block * o.taps;
                c8 = block * 8 + (tid & 7);
            } else {
                tap = fdiv(tid, o.d_cv);
                c8 = tid - tap * (o.C / 8);
            }
            const int r = fdiv(tap, o.d_s), s = tap - r * o.S;
            e = make_int2(((r * o.src_w + s) * o.C + c8 * 8) * 2, (tap * o.C + c8 * 8) * 2);
        }
        reinterpret_cast<int2 *>(lds + o.table)[tid] = e;
    }
    if (tid < c.in_chunks) *reinterpret_cast<uint4 *>(lds + tid * 16) = x0;
    for (int j = tid + kThreads; j < c.in_chunks; j += kThreads) *reinterpret_cast<uint4 *>(lds + j * 16) = in_chunk(j);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    lds_barrier();

    float *partial = reinterpret_cast<float *>(lds + c.partial);
    // A layer's output is copied to memory while the next layer runs.
    auto to_memory = [&](const ChainOp &o) {
        if (!o.y) return;
        if (o.kind == GPULET_OP_FC) {
            const size_t at = static_cast<size_t>(img) * o.K + tid;
            if (tid >= o.K) return;
            if (o.out_fp32)
                static_cast<float *>(o.y)[at] = *reinterpret_cast<const float *>(lds + o.dst_0 + tid * 4);
            else
                static_cast<__bf16 *>(o.y)[at] = *reinterpret_cast<const __bf16 *>(lds + o.dst_0 + tid * 2);
            return;
        }
        const int cv = o.K / 8, n = o.P * o.Q * cv;
        uint4 *y = static_cast<uint4 *>(o.y) + static_cast<size_t>(img) * n;
        for (int j = tid; j < n; j += kThreads) {
            const int m = fdiv(j, o.d_kv), c8 = j - m * cv;
            const int p = fdiv(m, o.d_q), q = m - p * o.Q;
            y[j] = *reinterpret_cast<const uint4 *>(lds + o.dst_0 + ((p * o.dst_w + q) * o.K + c8 * 8) * 2);
        }
    };
#pragma unroll 1
    for (int i = 0; i < c.n_second; ++i) stage(c.second[i], lds, wave, lane);
    bool pending = true;   // weights of fully connected layers are on their way
    for (int i = 0;; ++i) {
        const ChainOp &o = c.op[i];
        if (o.kind == GPULET_OP_CONV) {
            switch ((o.chunks + 3) / 4) {
                case 1: chain_conv<1>(o, lds, wave, lane); break;
                case 2: chain_conv<2>(o, lds, wave, lane); break;
                case 3: chain_conv<3>(o, lds, wave, lane); break;
                case 4: chain_conv<4>(o, lds, wave, lane); break;
                case 5: chain_conv<5>(o, lds, wave, lane); break;
                case 6: chain_conv<6>(o, lds, wave, lane); break;
                case 7: chain_conv<7>(o, lds, wave, lane); break;
                default: chain_conv<8>(o, lds, wave, lane); break;
            }
        } else if (o.kind == GPULET_OP_POOL) {
            if (o.S == 3)
                chain_pool<3>(o, lds);
            else
                chain_pool<2>(o, lds);
        } else {
            FETCH_FC(o);
            if (pending) {
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
                lds_barrier();
                pending = false;
            }
            if ((o.Kg & 7) == 0)
                chain_fc<8>(o, lds, partial, wave, lane);
            else if ((o.Kg & 3) == 0)
                chain_fc<4>(o, lds, partial, wave, lane);
            else
                chain_fc<1>(o, lds, partial, wave, lane);
            lds_barrier();
            if (tid < o.K) {
                const float *q = partial + (tid >> 4) * 64 + (tid & 15);
                float v = q[0];
                v += q[16];
                v += q[32];
                v += q[48];
                v += *reinterpret_cast<const float *>(lds + o.bias + tid * 4);
                if (o.relu) v = v > 0.f ? v : 0.f;
                if (o.out_fp32)
                    *reinterpret_cast<float *>(lds + o.dst_0 + tid * 4) = v;
                else
                    *reinterpret_cast<__bf16 *>(lds + o.dst_0 + tid * 2) = static_cast<__bf16>(v);
            }
        }
        lds_barrier();
        if (i == 1) {
#pragma unroll 1
            for (int e = 0; e < c.n_third; ++e) stage(c.third[e], lds, wave, lane);
            pending = pending || c.n_third > 0;
        }
        to_memory(o);
        if (i + 1 == c.n_ops) break;
    }
}

int align_up(int v, int a) { return (v + a - 1) / a * a; }

// Fills the kernel's argument block for layers l[0 .. n) (pointers excepted); false when a layer, or
// the run as a whole, is not one the kernel takes.
bool chain_params(const ChainLayer *l, int n, ChainParams &c) {
    if (n < 2 || n > kMaxChain) return false;
    for (int i = n; i < kMaxChain; ++i) c.op[i] = ChainOp{};
    int at = 0, partial = 0, two_tensors = 0;
    for (int i = 0; i < n; ++i) {
        ChainOp &o = c.op[i];
        o = ChainOp{};
        const ChainLayer &s = l[i];
        o.kind = s.kind; o.C = s.C; o.H = s.H; o.W = s.W; o.K = s.K; o.P = s.P; o.Q = s.Q; o.S = s.S;
        o.stride = s.stride; o.pad = s.pad; o.relu = s.relu; o.out_fp32 = s.out_fp32;
        if (s.kind == GPULET_OP_FC) {
            // longer rows are not added in four quarters by the kernel that runs the layer alone
            if (1LL * s.C * s.H * s.W >= kFcLongRow) return false;
            o.Kg = s.C * s.H * s.W;
            // whole 16-byte transfers
            if (2LL * o.Kg * s.K > kLdsBytes || o.Kg * s.K % 8 != 0 || s.K > kThreads) return false;
            if (o.out_fp32 && i + 1 < n) return false;   // the next layer reads bf16
            o.d_q = o.d_cv = o.d_kv = o.d_s = o.d_rs = make_fastdiv(1);
            partial = std::max(partial, (s.K + 15) / 16 * 64 * 4);
            continue;
        }
        if (s.C % 8 != 0 || s.K % 8 != 0 || s.K > kThreads) return false;
        o.d_q = make_fastdiv(s.Q);
        o.d_cv = make_fastdiv(s.C / 8);
        o.d_kv = make_fastdiv(s.K / 8);
        o.d_s = make_fastdiv(s.S);
        o.d_rs = make_fastdiv(s.R * s.S);
        if (s.kind == GPULET_OP_POOL) {
            if (s.S != 2 && s.S != 3) return false;
        } else {
            if (1LL * s.R * s.S * s.C > kMaxSteps * 32) return false;
            o.Kg = s.R * s.S * s.C;
            o.chunks = o.Kg / 8;
            o.taps = s.R * s.S;
            if (1LL * s.P * s.Q * s.K * o.Kg > kConvMacs) return false;
        }
    }
    // Tensors one behind the other, each with the border of zeros its reader's padding asks for; a
    // fully connected layer's source ends in zeros up to a multiple of 32 elements.
    for (int i = 0; i <= n; ++i) {
        const int C = i == 0 ? l[0].C : l[i - 1].K, H = i == 0 ? l[0].H : l[i - 1].P, W = i == 0 ? l[0].W : l[i - 1].Q;
        const int border = i < n && l[i].kind == GPULET_OP_CONV ? l[i].pad : 0;
        const int wide = W + 2 * border;
        const int first = (border * wide + border) * C * 2;
        const long long elem = i == n && l[n - 1].out_fp32 ? 4 : 2;
        const long long bytes = elem * C * (H + 2 * border) * wide;
        if (at + bytes > kLdsBytes) return false;
        if (i < n) {
            c.op[i].src = at;
            c.op[i].src_w = wide;
        }
        if (i > 0) {
            c.op[i - 1].dst_w = wide;
            c.op[i - 1].dst_0 = at + first;
        } else {
            c.in_row = W * C / 8;
            c.in_rows = H;
            c.in_border = border;
            c.in_edge = border * C / 8;
            c.in_wide = wide * C / 8;
            c.in_chunks = (H + 2 * border) * c.in_wide;
            if ((W * C) % 8 != 0 || (border > 0 && C % 8 != 0)) return false;
        }
        at += align_up(static_cast<int>(bytes), 64);
        if (i == 1) two_tensors = at;
    }
    const int zeros = at;
    at += 64;
    for (int i = 0; i < n; ++i) {
        c.op[i].zeros = zeros;
        c.op[i].bias = at;
        if (c.op[i].kind != GPULET_OP_POOL && !l[i].b) at += align_up(c.op[i].K * 4, 16);   // no bias: zeros
    }
    c.lds_tensors = at;
    at = align_up(at, 256);
    c.n_bias = c.n_first = c.n_second = c.n_third = 0;
    for (int i = 0; i < n; ++i) {
        ChainOp &o = c.op[i];
        if (o.kind == GPULET_OP_CONV) {
            o.table = at;
            at += kMaxSteps * 4 * 8;
        }
        if (o.kind != GPULET_OP_POOL && l[i].b) {
            o.bias = at;
            c.bias[c.n_bias++] = Staged{l[i].b, o.K * 4, at};
            at += align_up(o.K * 4, kBiasPiece);
        }
    }
    c.partial = at;
    at += partial;
    // Weights of the convolutions are staged at once, those of the first fully connected layer while the
    // first layer runs.  Those of later ones lie over the first two tensors where these are done with and large enough.
    int over = 0, n_fc = 0;
    for (int i = 0; i < n; ++i) {
        ChainOp &o = c.op[i];
        if (o.kind == GPULET_OP_POOL) continue;
        const int bytes = o.K * o.Kg * 2, room = align_up(bytes, kPiece);
        if (o.kind == GPULET_OP_FC && n_fc++ > 0 && i >= 3 && over + room <= two_tensors) {
            o.weights = over;
            c.third[c.n_third++] = Staged{l[i].w, bytes, over};
            over += room;
            continue;
        }
        o.weights = at;
        if (o.kind == GPULET_OP_FC)
            c.second[c.n_second++] = Staged{l[i].w, bytes, at};
        else
            c.first[c.n_first++] = Staged{l[i].w, bytes, at};
        at += room;
    }
    if (at > kLdsBytes) return false;   // nothing above lies higher, tables and zeros of a run without weights included
    c.n_ops = n;
    c.d_in_wide = make_fastdiv(c.in_wide);
    return true;
}

// Estimated time (us) of the run in one launch, and of its layers one by one.  Fitted to 1600 runs of two to seven
// layers (8 to 256 channels on 4x4 to 40x40, 64 to 2048 features, batch 1 to 2048, 64 to 256 CUs); they miss the
// measured times by 7 and 12 % (standard deviation).
double together_us(const ChainLayer *l, int n, int N, int n_cu) {
    auto up = [](double a, double b) { return std::ceil(a / b); };
    const double in_kb = 2.0 * l[0].C * l[0].H * l[0].W / 1024;
    double image = 3.1 + 0.0082 * in_kb, kb = in_kb;   // arguments, staging, the first barrier
    for (int i = 0; i < n; ++i) {
        const ChainLayer &s = l[i];
        const double cols = up(s.K, 16), out_kb = 2.0 * s.K * s.P * s.Q / 1024;
        image += 0.79 + 0.053 * out_kb;
        if (s.kind == GPULET_OP_CONV) {
            const int depth = s.R * s.S * s.C;   // a multiple of 128: all filters start in the same banks
            image += cols * ((depth % 128 == 0 ? 0.056 : 0.034) * up(depth, 32) + 0.15 * up(up(1.0 * s.P * s.Q, 16), kWaves));
        } else if (s.kind == GPULET_OP_FC) {
            const double in = 1.0 * s.C * s.H * s.W;
            image += 0.33 * up(4 * cols, kWaves) * up(up(up(in, 32), 4), kFcSteps) + 0.015 * 2 * in * s.K / 1024;
        }
        kb += out_kb;
    }
    // one image per CU at a time; the next one's arguments and first loads overlap the last one's stores
    return image * (0.2 + 0.8 * up(N, n_cu)) + 0.066 * N * kb / 1024;
}

double separate_us(const ChainLayer *l, int n, int N, int n_cu) {
    auto up = [](double a, double b) { return std::ceil(a / b); };
    double us = 0.0;
    for (int i = 0; i < n; ++i) {
        const ChainLayer &s = l[i];
        const double out = 1.0 * s.K * s.P * s.Q, in = 1.0 * s.C * s.H * s.W;
        if (s.kind == GPULET_OP_CONV) {
            const bool plain = s.R * s.S == 1 || s.C % BK == 0;
            us += 2.9 + 0.19 * up(1.0 * s.R * s.S * s.C, BK) + (plain ? 0.98 : 1.87) * N * s.P * s.Q * up(s.K, 64) / 128 / n_cu +
                  0.0106 * N * 2 * (in + out) / 1024 / n_cu;
        } else if (s.kind == GPULET_OP_POOL) {
            us += 2.7 + 0.0106 * N * 2 * out * (s.R * s.S + 1) / 1024 / n_cu;
        } else {
            const double steps = up(in, 32) / 4;
            us += 2.9 + 0.1 * steps + 0.36 * up(N, 32) * up(s.K, 16) * steps / n_cu;
        }
    }
    return us;
}

}  // namespace

// A workgroup takes its image through the run alone, on one CU: few and small layers win by the launches they
// save, and by what separate kernels of many images waste on 8 channels; wide layers, short runs and several images per
// CU lose (LeNet-5 wins at every batch, batch 2048 187 and 90 us; 1x1 256 -> 64 -> 256 on 7x7 at batch 1 7.3 and 13.7,
// at batch 2048 30 and 102; 256 -> 256 -> 32 features at batch 2048 10.6 and 60).  Of the runs above 991 fit as a whole:
// with this line 565 share a launch, a third faster in the mean (17 of them 3 % slower and more), 0.7 % above always
// taking the faster way; sharing all of them is 10 % slower than sharing none.
bool image_chain_pays(const ChainLayer *l, int n, int N, int n_cu) {
    const int cus = n_cu < 1 ? 1 : n_cu;
    return together_us(l, n, N, cus) <= 0.95 * separate_us(l, n, N, cus);
}

bool image_chain_applicable(const ChainLayer *l, int n) {
    ChainParams c;
    if (!chain_params(l, n, c)) return false;
    for (int i = 0; i < n; ++i)
        if (l[i].kind != GPULET_OP_POOL && reinterpret_cast<uintptr_t>(l[i].w) % 16 != 0) return false;
    return true;
}

hipError_t launch_image_chain(const ChainLayer *l, int n, const void *x, int N, hipStream_t stream) {
    ChainParams c;
    if (!image_chain_applicable(l, n) || !chain_params(l, n, c) || N < 1) return hipErrorInvalidValue;
    c.x = static_cast<const __bf16 *>(x);
    if (reinterpret_cast<uintptr_t>(x) % 16 != 0) return hipErrorInvalidValue;
    for (int i = 0; i < n; ++i) {
        c.op[i].y = l[i].y;
        if (l[i].kind != GPULET_OP_FC && reinterpret_cast<uintptr_t>(l[i].y) % 16 != 0) return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(image_chain_kernel, dim3(static_cast<unsigned>(N)), dim3(kThreads), 0, stream, c);
    return hipGetLastError();
}

}  // namespace gpulet
