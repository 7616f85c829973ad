// Depthwise convolution of the forward pass served on a gpu-let (paper Sec. 5;
// the SSD-MobileNet of Table 4 is built from depthwise 3x3 + pointwise 1x1
// pairs), NHWC bf16, filter [R][S][C] bf16, fp32 accumulation, fused bias and
// ReLU, one rounding to bf16.
//
// One multiply-add per loaded input element: the layer is bound by memory
// traffic, not by arithmetic, so there is nothing for the matrix cores to do.
// Each thread owns 8 consecutive channels (one 16-byte load per tap, adjacent
// lanes adjacent in memory) of TQ horizontally adjacent output pixels, so the
// taps neighbouring pixels share are loaded once per thread and the filter
// once per TQ pixels; the remaining overlap between threads is served by the
// caches.  Algorithmic bytes: 2*(N*H*W*C + N*P*Q*C + R*S*C) + 4*C.
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "gpulet_internal.h"

namespace gpulet {
namespace {

struct DwParams {
    const __bf16 *x, *w;
    const float *b;
    __bf16 *y;
    int N, C, H, W, R, S, stride, pad, relu, P, Q;
    int qt;     // thread columns per output row = ceil(Q / TQ)
    int total;  // work items
    int p_tiles;         // 3x3 kernels: thread rows per image
    int blocks_per_die;  // 3x3 kernels: workgroups per die (die_block)
    FastDiv d_cv, d_qt, d_p;  // 3x3 kernels: divisions by the channel groups, qt and p_tiles
};

__device__ __forceinline__ void unpack8(const uint4 &v, float f[8]) {
    const unsigned u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(u[i] << 16);
        f[2 * i + 1] = __uint_as_float(u[i] & 0xFFFF0000u);
    }
}

__device__ __forceinline__ void unpack4(const uint2 &v, float f[4]) {
    f[0] = __uint_as_float(v.x << 16);
    f[1] = __uint_as_float(v.x & 0xFFFF0000u);
    f[2] = __uint_as_float(v.y << 16);
    f[3] = __uint_as_float(v.y & 0xFFFF0000u);
}

__device__ __forceinline__ unsigned short bf16_bits(float f) {
    const __bf16 h = static_cast<__bf16>(f);
    return *reinterpret_cast<const unsigned short *>(&h);
}

template <int TQ>
__global__ __launch_bounds__(256) void dwconv_vec8(const DwParams p) {
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= p.total) return;
    const int cv = p.C >> 3;
    const int c8 = idx % cv;
    int t = idx / cv;
    const int qg = t % p.qt;
    t /= p.qt;
    const int pp = t % p.P;
    const int n = t / p.P;
    const int q0 = qg * TQ;

    float acc[TQ][8];
    float bias[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (p.b) {
        const float4 b0 = *reinterpret_cast<const float4 *>(p.b + c8 * 8);
        const float4 b1 = *reinterpret_cast<const float4 *>(p.b + c8 * 8 + 4);
        bias[0] = b0.x; bias[1] = b0.y; bias[2] = b0.z; bias[3] = b0.w;
        bias[4] = b1.x; bias[5] = b1.y; bias[6] = b1.z; bias[7] = b1.w;
    }
#pragma unroll
    for (int j = 0; j < TQ; ++j)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[j][i] = bias[i];

    const int h0 = pp * p.stride - p.pad;
    const int w_first = q0 * p.stride - p.pad;               // input column of tap 0 of the first pixel
    const int span = (TQ - 1) * p.stride + p.S;              // input columns the TQ pixels touch
    for (int r = 0; r < p.R; ++r) {
        const int h = h0 + r;
        if ((unsigned)h >= (unsigned)p.H) continue;
        const __bf16 *xrow = p.x + ((n * p.H + h) * p.W) * p.C + c8 * 8;
        const __bf16 *wrow = p.w + (r * p.S) * p.C + c8 * 8;
        for (int u = 0; u < span; ++u) {
            const int w = w_first + u;
            if ((unsigned)w >= (unsigned)p.W) continue;
            float xv[8];
            unpack8(*reinterpret_cast<const uint4 *>(xrow + w * p.C), xv);
            // input column u is tap s = u - j*stride of pixel j
#pragma unroll
            for (int j = 0; j < TQ; ++j) {
                const int s = u - j * p.stride;
                if (s < 0 || s >= p.S) continue;
                float wv[8];
                unpack8(*reinterpret_cast<const uint4 *>(wrow + s * p.C), wv);
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[j][i] = fmaf(xv[i], wv[i], acc[j][i]);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < TQ; ++j) {
        const int q = q0 + j;
        if (q >= p.Q) break;
        unsigned o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float a = acc[j][2 * i], b = acc[j][2 * i + 1];
            if (p.relu) {
                a = a > 0.f ? a : 0.f;
                b = b > 0.f ? b : 0.f;
            }
            o[i] = static_cast<unsigned>(bf16_bits(a)) | (static_cast<unsigned>(bf16_bits(b)) << 16);
        }
        *reinterpret_cast<uint4 *>(p.y + (((n * p.P + pp) * p.Q + q) * p.C + c8 * 8)) =
            make_uint4(o[0], o[1], o[2], o[3]);
    }
}

// 3x3 filters (every depthwise layer of MobileNet): the generic kernel above walks rows and
// columns in loops with tests, so each of its 18 loads waits for the previous one's use, and a
// layer of 24 MB took 20 us.  In the two kernels below the taps are unrolled at compile time and
// every input load (buffer loads: an offset pushed out of range returns zero, so padding needs no
// branch) and every filter load is issued before the first multiply-add.  Same summation order
// (bias, then filter rows and columns ascending), so the bits are those of the kernel above.  Both
// give every die a contiguous run of work items (die_block): neighbouring output rows share input
// rows, and dealt round-robin over the dies each of these was fetched into two or three L2s
// (batch 32: 128 channels 75x75 stride 2 13.0 -> 10.2 us, 512 channels 19x19 9.3 -> 8.8).
//
// Stride 2: 8 channels x TQ adjacent pixels of one output row per thread.
typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2_t;

template <int TQ>
__global__ __launch_bounds__(256) void dwconv3x3_s2(const DwParams p, const unsigned x_bytes) {
    constexpr int STRIDE = 2;
    constexpr int SPAN = (TQ - 1) * STRIDE + 3;  // input columns the TQ pixels touch
    constexpr unsigned OOB = 0x80000000u;
    const int idx = die_block(p.blocks_per_die, blockIdx.x) * 256 + threadIdx.x;
    if (idx >= p.total) return;
    const int cv = p.C >> 3;
    int t = fdiv(idx, p.d_cv);
    const int c8 = idx - t * cv;
    const int t1 = fdiv(t, p.d_qt);
    const int qg = t - t1 * p.qt;
    const int n = fdiv(t1, p.d_p);
    const int pp = t1 - n * p.P;
    const int q0 = qg * TQ;
    const int h0 = pp * STRIDE - p.pad, w_first = q0 * STRIDE - p.pad;

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16 *>(p.x), 0, x_bytes, 0x00020000);
    u32x4_t xr[3][SPAN];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int h = h0 + r;
        const bool h_ok = static_cast<unsigned>(h) < static_cast<unsigned>(p.H);
        const int row = ((n * p.H + h) * p.W + w_first) * p.C + c8 * 8;
#pragma unroll
        for (int u = 0; u < SPAN; ++u) {
            const bool ok = h_ok && static_cast<unsigned>(w_first + u) < static_cast<unsigned>(p.W);
            xr[r][u] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok ? static_cast<unsigned>((row + u * p.C) * 2) : OOB, 0, 0);
        }
    }
    uint4 wr[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int sx = 0; sx < 3; ++sx) wr[r][sx] = *reinterpret_cast<const uint4 *>(p.w + (r * 3 + sx) * p.C + c8 * 8);

    float acc[TQ][8];
    {
        float bias[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (p.b) {
            const float4 b0 = *reinterpret_cast<const float4 *>(p.b + c8 * 8);
            const float4 b1 = *reinterpret_cast<const float4 *>(p.b + c8 * 8 + 4);
            bias[0] = b0.x; bias[1] = b0.y; bias[2] = b0.z; bias[3] = b0.w;
            bias[4] = b1.x; bias[5] = b1.y; bias[6] = b1.z; bias[7] = b1.w;
        }
#pragma unroll
        for (int j = 0; j < TQ; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[j][i] = bias[i];
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        float wv[3][8];
#pragma unroll
        for (int sx = 0; sx < 3; ++sx) unpack8(wr[r][sx], wv[sx]);
#pragma unroll
        for (int u = 0; u < SPAN; ++u) {
            float xv[8];
            unpack8(make_uint4(xr[r][u][0], xr[r][u][1], xr[r][u][2], xr[r][u][3]), xv);
#pragma unroll
            for (int j = 0; j < TQ; ++j) {
                const int sx = u - j * STRIDE;  // input column u is tap sx of pixel j
                if (sx < 0 || sx >= 3) continue;
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[j][i] = fmaf(xv[i], wv[sx][i], acc[j][i]);
            }
        }
    }
    const unsigned limit = relu_limit(p.relu);
#pragma unroll
    for (int j = 0; j < TQ; ++j) {
        const int q = q0 + j;
        if (q >= p.Q) break;
        unsigned o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = relu_or_pass(pack_bf16(acc[j][2 * i], acc[j][2 * i + 1]), limit);
        *reinterpret_cast<uint4 *>(p.y + (((n * p.P + pp) * p.Q + q) * p.C + c8 * 8)) =
            make_uint4(o[0], o[1], o[2], o[3]);
    }
}

// Stride 1: 4 channels of TQ x TP = 4 x 2 output pixels per thread.  With 8 channels of 4 x 1 pixels
// (the stride-2 kernel's split) a thread held 192 registers, two wavefronts per SIMD, and every input
// element was loaded 4.5 times and unpacked as often: the layer waited for issue and L1, not for memory.
// Half the channels leave room for a second output row (3 loads per element, 126 registers, four wavefronts):
// batch 32, 32 channels 150x150 (92 MB) 32.2 -> 28.1 us, 128 on 75x75 32.2 -> 27.5, 256 on 38x38 17.5 -> 13.2,
// 512 on 19x19 10.5 -> 9.3.  Smaller tiles load more (4 x 1 10.2 us on 19x19), 4 x 4 wants more registers
// (256 on 38x38 14.5 us); a rolling walk down the rows has too few wavefronts (44 us and more on 75x75), and
// at stride 2, where rows are shared less, two rows gain nothing (13.0 and 12.8 us).
template <int TQ, int TP>
__global__ __launch_bounds__(256) void dwconv3x3_tile(const DwParams p, const unsigned x_bytes) {
    constexpr int SPAN = TQ + 2, ROWS = TP + 2;   // input columns and rows of the tile
    constexpr unsigned OOB = 0x80000000u;
    const int idx = die_block(p.blocks_per_die, blockIdx.x) * 256 + threadIdx.x;
    if (idx >= p.total) return;
    const int cv = p.C >> 2;
    const int t = fdiv(idx, p.d_cv);
    const int c = (idx - t * cv) * 4;
    const int t1 = fdiv(t, p.d_qt);
    const int q0 = (t - t1 * p.qt) * TQ;
    const int n = fdiv(t1, p.d_p);
    const int p0 = (t1 - n * p.p_tiles) * TP;
    const int h0 = p0 - p.pad, w_first = q0 - p.pad;

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16 *>(p.x), 0, x_bytes, 0x00020000);
    u32x2_t xr[ROWS][SPAN];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        const bool h_ok = static_cast<unsigned>(h0 + i) < static_cast<unsigned>(p.H);
        const int row = (((n * p.H + h0 + i) * p.W + w_first) * p.C + c) * 2;
#pragma unroll
        for (int u = 0; u < SPAN; ++u) {
            const bool ok = h_ok && static_cast<unsigned>(w_first + u) < static_cast<unsigned>(p.W);
            xr[i][u] = __builtin_amdgcn_raw_buffer_load_b64(rx, ok ? static_cast<unsigned>(row + u * (p.C * 2)) : OOB, 0, 0);
        }
    }
    uint2 wr[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) wr[k] = *reinterpret_cast<const uint2 *>(p.w + k * p.C + c);
    float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
    if (p.b) bias = *reinterpret_cast<const float4 *>(p.b + c);
    float wt[9][4];
#pragma unroll
    for (int k = 0; k < 9; ++k) unpack4(wr[k], wt[k]);
    float acc[TP][TQ][4];
#pragma unroll
    for (int o = 0; o < TP; ++o)
#pragma unroll
        for (int j = 0; j < TQ; ++j) {
            acc[o][j][0] = bias.x;
            acc[o][j][1] = bias.y;
            acc[o][j][2] = bias.z;
            acc[o][j][3] = bias.w;
        }
    const unsigned limit = relu_limit(p.relu);
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
#pragma unroll
        for (int u = 0; u < SPAN; ++u) {
            float xv[4];
            unpack4(make_uint2(xr[i][u][0], xr[i][u][1]), xv);
#pragma unroll
            for (int o = 0; o < TP; ++o) {
                const int r = i - o;
                if (r < 0 || r >= 3) continue;
#pragma unroll
                for (int j = 0; j < TQ; ++j) {
                    const int sx = u - j;  // input column u is tap sx of pixel j
                    if (sx < 0 || sx >= 3) continue;
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[o][j][e] = fmaf(xv[e], wt[r * 3 + sx][e], acc[o][j][e]);
                }
            }
        }
        if (i >= 2) {
            const int o = i - 2;
            if (p0 + o < p.P) {
                __bf16 *y = p.y + (((n * p.P + p0 + o) * p.Q + q0) * p.C + c);
#pragma unroll
                for (int j = 0; j < TQ; ++j) {
                    if (q0 + j >= p.Q) break;
                    *reinterpret_cast<uint2 *>(y + j * p.C) =
                        make_uint2(relu_or_pass(pack_bf16(acc[o][j][0], acc[o][j][1]), limit),
                                   relu_or_pass(pack_bf16(acc[o][j][2], acc[o][j][3]), limit));
                }
            }
        }
    }
}

// Any channel count or alignment: one thread per output element.
__global__ __launch_bounds__(256) void dwconv_scalar(const DwParams p) {
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= p.total) return;
    const int c = idx % p.C;
    int t = idx / p.C;
    const int q = t % p.Q;
    t /= p.Q;
    const int pp = t % p.P;
    const int n = t / p.P;
    float acc = p.b ? p.b[c] : 0.f;
    for (int r = 0; r < p.R; ++r) {
        const int h = pp * p.stride - p.pad + r;
        if ((unsigned)h >= (unsigned)p.H) continue;
        for (int s = 0; s < p.S; ++s) {
            const int w = q * p.stride - p.pad + s;
            if ((unsigned)w >= (unsigned)p.W) continue;
            acc = fmaf(static_cast<float>(p.x[((n * p.H + h) * p.W + w) * p.C + c]),
                       static_cast<float>(p.w[(r * p.S + s) * p.C + c]), acc);
        }
    }
    if (p.relu) acc = acc > 0.f ? acc : 0.f;
    p.y[idx] = static_cast<__bf16>(acc);
}

}  // namespace

gpulet_status check_dwconv(int N, int C, int H, int W, int R, int S, int stride, int pad, int *P, int *Q) {
    if (N < 1 || C < 1 || H < 1 || W < 1 || R < 1 || S < 1 || stride < 1 || pad < 0) return GPULET_EINVAL;
    *P = out_extent(H, R, stride, pad);
    *Q = out_extent(W, S, stride, pad);
    if (*P < 1 || *Q < 1) return GPULET_EINVAL;
    const long long lim = 1LL << 30;
    if (1LL * N * H * W * C >= lim || 1LL * N * *P * *Q * C >= lim || 1LL * R * S * C >= lim) return GPULET_EINVAL;
    return GPULET_OK;
}

hipError_t launch_dwconv(const void *x, const void *w, const float *b, void *y, int N, int C, int H, int W,
                         int R, int S, int stride, int pad, int relu, int P, int Q, hipStream_t stream) {
    DwParams p;
    p.x = static_cast<const __bf16 *>(x);
    p.w = static_cast<const __bf16 *>(w);
    p.b = b;
    p.y = static_cast<__bf16 *>(y);
    p.N = N; p.C = C; p.H = H; p.W = W; p.R = R; p.S = S; p.stride = stride; p.pad = pad; p.relu = relu;
    p.P = P; p.Q = Q;
    const bool vec = (C % 8 == 0) && reinterpret_cast<uintptr_t>(x) % 16 == 0 &&
                     reinterpret_cast<uintptr_t>(w) % 16 == 0 && reinterpret_cast<uintptr_t>(y) % 16 == 0 &&
                     reinterpret_cast<uintptr_t>(b) % 16 == 0;
    if (vec && R == 3 && S == 3 && (stride == 1 || stride == 2)) {
        const unsigned x_bytes = static_cast<unsigned>(2LL * N * H * W * C);
        const int tq = stride == 1 ? 4 : 2, cv = C / (stride == 1 ? 4 : 8);
        p.qt = (Q + tq - 1) / tq;
        p.p_tiles = stride == 1 ? (P + 1) / 2 : P;
        p.total = N * p.p_tiles * p.qt * cv;
        p.d_cv = make_fastdiv(cv);
        p.d_qt = make_fastdiv(p.qt);
        p.d_p = make_fastdiv(p.p_tiles);
        p.blocks_per_die = (p.total + 8 * 256 - 1) / (8 * 256);
        const dim3 grid(static_cast<unsigned>(8 * p.blocks_per_die));
        if (stride == 1)
            hipLaunchKernelGGL((dwconv3x3_tile<4, 2>), grid, dim3(256), 0, stream, p, x_bytes);
        else
            hipLaunchKernelGGL(dwconv3x3_s2<2>, grid, dim3(256), 0, stream, p, x_bytes);
    } else if (vec) {
        constexpr int TQ = 4;
        p.qt = (Q + TQ - 1) / TQ;
        p.total = N * P * p.qt * (C / 8);
        hipLaunchKernelGGL(dwconv_vec8<TQ>, dim3((p.total + 255) / 256), dim3(256), 0, stream, p);
    } else {
        p.qt = Q;
        p.total = N * P * Q * C;
        hipLaunchKernelGGL(dwconv_scalar, dim3((p.total + 255) / 256), dim3(256), 0, stream, p);
    }
    return hipGetLastError();
}

}  // namespace gpulet
