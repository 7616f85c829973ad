// Prints the launches gpulet_run_model would make: the launchers and the gpu-let functions below take the place of
// the library's own (this program comes first in symbol resolution).  No device is touched; the pointers are
// made up and never followed.  Reads requests
//   n_cu batch split_k in_at out_at n_layers n_bufs C H W in_buf out_buf
// followed by the layers, "op in_buf out_buf res_buf C K R S stride pad relu mode out_fp32 group_next
// bias" each.  The input lies at
// in_at, the output at out_at, and the workspace at kWorkspace; bias 0 stands for no bias.  Prints a line per launch: the
// kernel and how many layers it runs.
#include <cstdio>
#include <vector>

#include "gpulet_internal.h"

namespace gpulet {

static int g_n_cu;
static hipError_t say(const char *kernel, int layers) {
    std::printf("%s %d\n", kernel, layers);
    return hipSuccess;
}

bool live(const gpulet_partition *) { return true; }
LaunchCtx partition_ctx(const gpulet_partition *) {
    LaunchCtx c;
    c.n_cu = g_n_cu;
    c.scratch = reinterpret_cast<float *>(0x1000);
    c.scratch_bytes = 64u << 20;
    c.counters = reinterpret_cast<unsigned *>(0x1000);
    c.n_counters = 4096;
    return c;
}
hipError_t launch_conv(const ConvArgs &a, const LaunchCtx &, hipStream_t) { return a.post_pool2 ? say("conv+pool", 2) : say("conv", 1); }
hipError_t launch_conv_group(const ConvArgs *, int n, const LaunchCtx &, hipStream_t, int *launches) {
    *launches = 1;
    return say("group", n);
}
hipError_t launch_pool(const void *, void *, int, int, int, int, int, int, int, int, int, int, hipStream_t) { return say("pool", 1); }
hipError_t launch_dwconv(const void *, const void *, const float *, void *, int, int, int, int, int, int, int, int, int, int, int,
                         hipStream_t) {
    return say("dwconv", 1);
}
hipError_t launch_fc(const void *, const void *, const float *, void *, int N, int In, int Out, int, int, const LaunchCtx &c,
                     hipStream_t) {
    return say(fc_deep(N, In, Out, c.n_cu) ? "fc-deep" : "fc", 1);
}
hipError_t launch_image_chain(const ChainLayer *, int n, const void *, int, hipStream_t) { return say("chain", n); }
hipError_t launch_dwpw(const DwPwArgs &, int, hipStream_t) { return say("dwpw", 2); }

}  // namespace gpulet

int main() {
    constexpr unsigned long long kWorkspace = 0x100000000ULL, kWeights = 0x800000000ULL;
    int batch, split;
    unsigned long long in_at, out_at;
    gpulet_model_desc m{};
    while (std::scanf("%d %d %d %llx %llx %d %d %d %d %d %d %d", &gpulet::g_n_cu, &batch, &split, &in_at, &out_at, &m.n_layers,
                      &m.n_bufs, &m.in_C, &m.in_H, &m.in_W, &m.in_buf, &m.out_buf) == 12) {
        std::vector<gpulet_layer> l(static_cast<size_t>(m.n_layers));
        for (gpulet_layer &y : l) {
            y = gpulet_layer{};
            int bias = 0;
            if (std::scanf("%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d", &y.op, &y.in_buf, &y.out_buf, &y.res_buf, &y.C, &y.K, &y.R,
                           &y.S, &y.stride, &y.pad, &y.relu, &y.mode, &y.out_fp32, &y.group_next, &bias) != 15)
                return 1;
            y.w = reinterpret_cast<void *>(kWeights);
            y.b = bias ? reinterpret_cast<float *>(kWeights) : nullptr;
        }
        m.layers = l.data();
        gpulet_partition p{};
        if (gpulet_set_conv_split_k(split) != GPULET_OK) return 1;
        if (gpulet_run_model(&m, batch, &p, reinterpret_cast<void *>(in_at), reinterpret_cast<void *>(out_at),
                             reinterpret_cast<void *>(kWorkspace), ~0ULL >> 1, nullptr) != GPULET_OK)
            return 1;
        std::printf("end\n");
    }
    return 0;
}
