// Prints which convolution kernel the library would launch: the launchers below take the place of the
// library's own (this program comes first in symbol resolution) and print their arguments instead.
// Reads lines "n_cu n" followed by n layers "N C H W K R S stride pad stored", where `stored` is the
// number of channels per input pixel in memory; n > 1 is a launch group.  For each line prints one
// line per launch.  No device is touched; the pointers are made up and never followed.
#include <cstdio>

#include "conv_common.h"

namespace gpulet {
namespace conv {

static hipError_t say(const char *kernel, const ConvParams *p, int n, int tile) {
    std::printf("%s %d", kernel, tile);
    for (int j = 0; j < n; ++j) std::printf(" %dx%dx%dx%dx%d", p[j].N, p[j].C, p[j].H, p[j].W, p[j].K);
    std::printf("\n");
    return hipSuccess;
}
hipError_t launch_igemm(const ConvParams &p, bool, int tile, int, bool, hipStream_t) { return say("gather", &p, 1, tile); }
hipError_t launch_igemm_group(const ConvParams *p, int n, int tile, bool, hipStream_t) { return say("group", p, n, tile); }
hipError_t launch_patch(ConvParams p, int, int variant, hipStream_t) { return say("patch", &p, 1, variant); }
hipError_t launch_c64(ConvParams p, int, int, bool, hipStream_t) { return say("c64", &p, 1, 0); }
hipError_t launch_tall(ConvParams p, int, int, bool, hipStream_t) { return say("tall", &p, 1, 0); }
hipError_t launch_stream(ConvParams p, int, hipStream_t) { return say("stream", &p, 1, 0); }
hipError_t launch_stem(ConvParams p, int, hipStream_t) { return say("stem", &p, 1, 0); }

}  // namespace conv
}  // namespace gpulet

int main() {
    using namespace gpulet;
    int n_cu, n;
    while (std::scanf("%d %d", &n_cu, &n) == 2) {
        ConvArgs a[kMaxGroup];
        if (n < 1 || n > kMaxGroup) return 1;
        for (int j = 0; j < n; ++j) {
            ConvArgs &l = a[j];
            l.x = reinterpret_cast<void *>(0x10000);
            l.w = reinterpret_cast<void *>(0x20000);
            l.b = nullptr;
            l.y = reinterpret_cast<void *>(0x40000 + j * 0x10000);
            l.residual = nullptr;
            if (std::scanf("%d %d %d %d %d %d %d %d %d %d", &l.N, &l.C, &l.H, &l.W, &l.K, &l.R, &l.S, &l.stride, &l.pad,
                           &l.x_ch_stride) != 10)
                return 1;
            l.relu = 1;
            l.P = out_extent(l.H, l.R, l.stride, l.pad);
            l.Q = out_extent(l.W, l.S, l.stride, l.pad);
            l.y_ch_stride = l.K;
            l.y_ch_offset = 0;
            if (check_conv(l) != GPULET_OK) return 1;
        }
        LaunchCtx ctx;
        ctx.n_cu = n_cu;
        const hipError_t st = n == 1 ? launch_conv(a[0], ctx, nullptr) : launch_conv_group(a, n, ctx, nullptr);
        if (st != hipSuccess) return 1;
        std::printf("end\n");
    }
    return 0;
}
