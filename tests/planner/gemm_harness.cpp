// Host-only harness around the projections' choice of GEMM tiles (the
// translation unit is included as is; launches are stubbed, and the device
// queries answer for a 256-CU device).  Input on stdin, one call per line:
//   M N K batch epilogue fp32_activations gathered bm bn depth
// (the last three: forced values, -1 for the library's choice).
// Output, one line per call:
//   bm bn depth kg
#include <hip/hip_runtime.h>

static hipError_t harness_get_device(int *d) {
    *d = 0;
    return hipSuccess;
}
static hipError_t harness_get_attribute(int *v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
#define hipGetDevice harness_get_device
#define hipDeviceGetAttribute harness_get_attribute
#include "../../paper_2607_02043_amd/csrc/proj_api.cpp"
#undef hipGetDevice
#undef hipDeviceGetAttribute

#include <cstdio>

namespace mla {
int set_error(int code, const char *, ...) { return code; }
int batch_rows(const mla_batch *, int *) { return MLA_ERR_UNSUPPORTED; }
int attn_workspace(const mla_batch *, size_t *, ChunkRoute) { return MLA_ERR_UNSUPPORTED; }
int attend_rows(const mla_batch *, const uint16_t *, const uint16_t *, uint16_t *, float, void *, int32_t, void *, size_t, void *,
                ChunkRoute) {
    return MLA_ERR_UNSUPPORTED;
}
}  // namespace mla
namespace proj {
hipError_t launch_gemm(const GemmArgs &, const GemmShape &, bool, int, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_mha_prefill(const MhaArgs &, hipStream_t) { return hipErrorNotSupported; }
}  // namespace proj
extern "C" int mixed_step(const mla_batch *, const uint16_t *, const uint16_t *, uint16_t *, float, void *, int32_t, float *, void *,
                          size_t, void *) {
    return MLA_ERR_UNSUPPORTED;
}

int main() {
    long long M;
    int N, K, batch, epi, f32, gathered, bm, bn, depth;
    while (std::scanf("%lld %d %d %d %d %d %d %d %d %d", &M, &N, &K, &batch, &epi, &f32, &gathered, &bm, &bn, &depth) == 10) {
        mla_layer_tune(MLA_TUNE_GEMM_BM, bm);
        mla_layer_tune(MLA_TUNE_GEMM_BN, bn);
        mla_layer_tune(MLA_TUNE_GEMM_DEPTH, depth);
        const proj::GemmShape t = pick_shape(M, N, K, batch, epi, f32 != 0, gathered != 0);
        std::printf("%d %d %d %d\n", t.bm, t.bn, t.depth, t.kg);
    }
}
