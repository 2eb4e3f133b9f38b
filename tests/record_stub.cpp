// Stand-in for the device side of the library that notes what each call would launch, for
// a host-only build of the C ABI (gemm_api.cpp) and the selector (selector.cpp): CPU tests
// call the GEMM entry points of that build and read back the launch.
#include <stdint.h>

#include "../include/gemm_mi355x.h"
#include "../paper_2512_13282_amd/csrc/launch.h"

static int64_t g_last[8];

namespace gemm {
int launch_gemm(const KernelArgs &a, int32_t config, int64_t grid, void *, bool static_scratch) {
    const int64_t v[8] = {config, a.split_k, a.k_chunk, a.reduce_in_kernel, grid, a.epilogue, static_scratch,
                          int64_t(a.tiles_m) * a.tiles_n};
    for (int i = 0; i < 8; ++i) g_last[i] = v[i];
    return LAUNCH_OK;
}
int release_workspaces() { return LAUNCH_OK; }
}  // namespace gemm

extern "C" void recorded_launch(int64_t *out) {
    for (int i = 0; i < 8; ++i) out[i] = g_last[i];
}
extern "C" int gemm_probe_mfma(int, int, int32_t, int64_t *, unsigned *, gemm_probe_info *, void *) {
    return GEMM_ERR_HIP;
}
extern "C" int gemm_probe_read(const void *, int64_t, unsigned *, int64_t, void *) { return GEMM_ERR_HIP; }
