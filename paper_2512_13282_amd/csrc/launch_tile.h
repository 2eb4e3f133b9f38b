// launch_tile.h -- the GENERIC, MACRO and register-staged SKINNY configurations.
// Instantiated for one dtype per translation unit (launch_tile_{i8,bf16}.hip).
#pragma once

#include "families.h"
#include "kern_tile.h"

namespace gemm {

// GENERIC: the 16-byte loader where the operands' rows allow it, else element by element.
template <int DT, int BM, int BN, int WM, int WN, int WPE, int AHEAD>
static hipError_t launch_any(const KernelArgs &a, int64_t grid, hipStream_t stream) {
    const dim3 g{unsigned(grid)}, b(64 * WM * WN);
    if (a.b_trans) hipLaunchKernelGGL((gemm_tile_kernel<DT, BM, BN, WM, WN, true, WPE, AHEAD>), g, b, 0, stream, a);
    else hipLaunchKernelGGL((gemm_tile_kernel<DT, BM, BN, WM, WN, false, WPE, AHEAD>), g, b, 0, stream, a);
    return hipGetLastError();
}

template <int DT, int BM, int BN, int WPE>
static hipError_t launch_element(const KernelArgs &a, int64_t grid, hipStream_t stream) {
    if (a.b_trans)
        hipLaunchKernelGGL((gemm_element_kernel<DT, BM, BN, 2, 2, WPE, true>), dim3(unsigned(grid)), dim3(256), 0,
                           stream, a);
    else
        hipLaunchKernelGGL((gemm_element_kernel<DT, BM, BN, 2, 2, WPE, false>), dim3(unsigned(grid)), dim3(256), 0,
                           stream, a);
    return hipGetLastError();
}

template <int DT, int BM, int BN, int WM, int WN, int WPE>
static hipError_t launch_vec(const KernelArgs &a, int64_t grid, hipStream_t stream) {
    if (a.b_trans) return hipErrorInvalidValue;
    hipLaunchKernelGGL((gemm_vec_kernel<DT, BM, BN, WM, WN, WPE>), dim3(unsigned(grid)), dim3(64 * WM * WN), 0,
                       stream, a);
    return hipGetLastError();
}

template <int DT>
hipError_t launch_tile_family(int32_t cfg, const KernelArgs &a, int64_t grid, hipStream_t s) {
    const bool wide = wide_rows_ok(a.dtype, a.b_trans, a.N, a.K, a.lda, a.ldb);
    if (kConfigs[cfg].family == FAM_GENERIC && !wide) {
        switch (cfg) {
            case 0: return launch_element<DT, 64, 64, 2>(a, grid, s);
            case 1: return launch_element<DT, 128, 128, 1>(a, grid, s);
            default: return hipErrorInvalidValue;
        }
    }
    switch (cfg) {
        case 0: return launch_any<DT, 64, 64, 2, 2, 4, 1>(a, grid, s);
        case 1: return launch_any<DT, 128, 128, 2, 2, 2, 2>(a, grid, s);
        case 2: return launch_vec<DT, 256, 256, 2, 2, 1>(a, grid, s);
        case 3: return launch_vec<DT, 128, 256, 2, 2, 1>(a, grid, s);
        case 4: return launch_vec<DT, 256, 128, 2, 2, 1>(a, grid, s);
        case 5: return launch_vec<DT, 128, 128, 2, 2, 2>(a, grid, s);
        case 6: return launch_vec<DT, 32, 256, 1, 4, 2>(a, grid, s);
        case 7: return launch_vec<DT, 64, 256, 1, 4, 2>(a, grid, s);
        case 41: return launch_any<DT, 32, 128, 1, 4, 4, 1>(a, grid, s);
        case 42: return launch_any<DT, 64, 128, 1, 4, 3, 1>(a, grid, s);
        case 43: return launch_any<DT, 256, 128, 4, 2, 2, 2>(a, grid, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace gemm
