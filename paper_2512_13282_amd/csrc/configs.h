// configs.h -- the tile configurations compiled into the library.
//
// One table, read by the host-side selector (selector.cpp) and by the launch
// code (gemm_launch.hip and the launch_*.hip family units), which instantiates
// exactly these kernels.  Pure C++:
// no HIP headers, so the selector builds and tests on a machine without a GPU.
//
// Tiling levels (paper, Sec. 4.1: instruction tile r x s x t -> per-core kernel
// m_ct x k_ct x n_ct -> whole-array tile -> full GEMM): here the MFMA
// instruction tile -> the wave tile -> the workgroup macro-tile BM x BK x BN
// staged through LDS -> the grid of output tiles.  Each workgroup owns one
// output tile and reduces K in time with the accumulators held in registers
// (output-stationary, Sec. 4.2.1); split-K (several workgroups per tile, each
// on a K slice) is only used where too few output tiles exist to fill the GPU.
#pragma once

#include <stdint.h>

namespace gemm {

enum Dtype : int32_t { DT_I8 = 0, DT_BF16 = 1 };

enum Family : int32_t { FAM_GENERIC = 0, FAM_MACRO = 1, FAM_SKINNY = 2, FAM_DIRECT = 3, FAM_RING = 4,
                        FAM_GEMV = 5 };

struct TileConfig {
    int32_t family;
    int32_t bm, bn;      // workgroup macro-tile (rows of C, cols of C)
    int32_t wm, wn;      // waves along M and N (wave tile = bm/wm x bn/wn)
    int32_t occupancy;   // workgroups resident per CU (LDS and register bound)
    int32_t stages;      // LDS stage buffers
    double  eff_i8;      // fraction of the 2.4 GHz dense MFMA peak that a CU full of these workgroups
    double  eff_bf16;    // sustains, int8 and bf16; fitted on timed calls with the model's constants
    int32_t col_major_b; // also compiled for B stored column-major (N x K)
    const char *name;
};

// K depth of one LDS stage is 128 bytes for both dtypes: 64 bf16 or 128 int8
// elements.  Every MFMA consumes 32 bytes of K per lane pair (bf16 32x32x16,
// int8 32x32x32), so a stage is 4 MFMA k-steps.
constexpr int32_t kStageKBytes = 128;

// The ring family walks K in 64-byte slots (two MFMA k-steps), `stages` of them
// resident in LDS at once.
constexpr int32_t kSlotKBytes = 64;

// Family GENERIC: operands at any address (any lda/ldb/K/N): 16-byte loads where
// wide_rows_ok, element by element (configurations 0 and 1 only) otherwise.
// Family MACRO: 16-byte vector loads staged through registers (B transposed
// in registers); large tiles.
// Family SKINNY: same loaders, narrow M tile for M <= 64.
// Family GEMV: M = 1 only, vector-ALU matrix-vector kernels, one per B layout
// (col_major_b = 1 marks the column-major-only one); the efficiencies are the
// vector-ALU multiply-add rate as a fraction of the MFMA peak.
// Family DIRECT: both operands stream global -> LDS directly (buffer loads with
// an LDS destination); B's fragments come from LDS transpose reads, or, for B
// stored column-major, from 16-byte reads like A's.  The three-stage 64 x 64 kernel's rates
// are a workgroup's alone and a full CU's on K = 4096 (0.17-0.18 and 0.17-0.23); fitted lower,
// it was passed by for slower tiles.  The ping-pong kernel has two rows:
// 44, both layouts, and kPingPongRowOnly, row-major B only, for plan files and forced plans
// that name it (by index); the selector's own choice passes it by.
constexpr TileConfig kConfigs[] = {
    // family       bm   bn  wm wn occ stages eff_i8 eff_bf16 colB name
    {FAM_GENERIC,   64,  64, 2, 2, 4, 2, 0.141, 0.156, 1, "generic_64x64_w4"},
    {FAM_GENERIC,  128, 128, 2, 2, 2, 2, 0.196, 0.225, 1, "generic_128x128_w4"},
    {FAM_MACRO,    256, 256, 2, 2, 1, 2, 0.331, 0.410, 0, "macro_256x256_w4"},
    {FAM_MACRO,    128, 256, 2, 2, 1, 2, 0.269, 0.339, 0, "macro_128x256_w4"},
    {FAM_MACRO,    256, 128, 2, 2, 1, 2, 0.306, 0.318, 0, "macro_256x128_w4"},
    {FAM_MACRO,    128, 128, 2, 2, 2, 2, 0.243, 0.269, 0, "macro_128x128_w4"},
    {FAM_SKINNY,    32, 256, 1, 4, 2, 2, 0.142, 0.180, 0, "skinny_32x256_w4"},
    {FAM_SKINNY,    64, 256, 1, 4, 2, 2, 0.232, 0.300, 0, "skinny_64x256_w4"},
    {FAM_DIRECT,   256, 256, 2, 2, 1, 2, 0.421, 0.507, 1, "direct_256x256_w4"},
    {FAM_DIRECT,   128, 256, 2, 2, 1, 2, 0.485, 0.364, 1, "direct_128x256_w4"},
    {FAM_DIRECT,   256, 256, 2, 4, 1, 2, 0.640, 0.674, 1, "direct_256x256_w8"},
    {FAM_DIRECT,   256, 256, 4, 2, 1, 2, 0.608, 0.694, 1, "direct_256x256_w8t"},
    {FAM_DIRECT,   128, 256, 2, 4, 1, 2, 0.457, 0.388, 1, "direct_128x256_w8"},
    {FAM_DIRECT,   256, 256, 2, 4, 1, 2, 0.779, 0.767, 0, "pingpong_256x256_w8"},
    {FAM_SKINNY,    32, 256, 1, 4, 1, 4, 0.128, 0.144, 0, "stream_32x256_s4"},
    {FAM_SKINNY,    64, 256, 1, 4, 1, 3, 0.215, 0.285, 0, "stream_64x256_s3"},
    {FAM_RING,     256, 256, 2, 4, 1, 4, 0.684, 0.662, 1, "ring_256x256_w8"},
    {FAM_RING,     256, 256, 4, 2, 1, 4, 0.699, 0.691, 1, "ring_256x256_w8t"},
    {FAM_RING,     128, 256, 2, 4, 1, 5, 0.529, 0.543, 1, "ring_128x256_w8"},
    {FAM_RING,     256, 256, 2, 2, 1, 4, 0.439, 0.620, 1, "ring_256x256_w4"},
    {FAM_RING,      32,  64, 1, 2, 2, 8, 0.058, 0.068, 1, "ring_32x64_w2"},
    {FAM_RING,      64,  64, 1, 2, 2, 8, 0.083, 0.133, 1, "ring_64x64_w2"},
    {FAM_RING,      32, 128, 1, 4, 1, 8, 0.068, 0.132, 1, "ring_32x128_w4"},
    {FAM_RING,      64, 128, 1, 4, 1, 8, 0.138, 0.149, 1, "ring_64x128_w4"},
    {FAM_RING,      32, 256, 1, 4, 1, 6, 0.151, 0.190, 1, "ring_32x256_w4"},
    {FAM_RING,      64, 256, 1, 4, 1, 6, 0.261, 0.339, 1, "ring_64x256_w4"},
    {FAM_GEMV,       1, 1024, 1, 4, 4, 1, 0.03, 0.06, 0, "gemv_1024"},
    {FAM_GEMV,       1,  16, 1, 4, 4, 1, 0.03, 0.06, 1, "gemv_bt_16"},
    {FAM_RING,      32, 256, 1, 4, 2, 4, 0.156, 0.214, 1, "ring_32x256_w4_r4"},
    {FAM_RING,      32, 128, 1, 4, 2, 6, 0.118, 0.149, 1, "ring_32x128_w4_r6"},
    {FAM_RING,      64, 128, 1, 4, 2, 5, 0.233, 0.224, 1, "ring_64x128_w4_r5"},
    {FAM_RING,     128, 128, 2, 2, 2, 4, 0.404, 0.361, 1, "ring_128x128_w4"},
    {FAM_RING,     128, 128, 2, 2, 1, 8, 0.333, 0.359, 1, "ring_128x128_w4_r8"},
    {FAM_RING,     128, 128, 2, 4, 1, 8, 0.269, 0.361, 1, "ring_128x128_w8"},
    {FAM_RING,     256, 256, 4, 2, 1, 5, 0.663, 0.691, 1, "ring_256x256_w8t_r5"},
    {FAM_RING,     256, 256, 2, 4, 1, 5, 0.659, 0.683, 1, "ring_256x256_w8_r5"},
    {FAM_RING,     256, 256, 2, 2, 1, 5, 0.426, 0.629, 1, "ring_256x256_w4_r5"},
    {FAM_RING,     128, 256, 2, 2, 2, 3, 0.451, 0.446, 1, "ring_128x256_w4_r3"},
    {FAM_RING,     256, 128, 2, 2, 2, 3, 0.555, 0.373, 1, "ring_256x128_w4_r3"},
    {FAM_RING,     128, 256, 1, 4, 2, 3, 0.413, 0.435, 1, "ring_128x256_w4c_r3"},
    {FAM_RING,     128, 256, 2, 4, 2, 3, 0.560, 0.549, 1, "ring_128x256_w8_r3"},
    {FAM_GENERIC,   32, 128, 1, 4, 4, 2, 0.104, 0.131, 1, "generic_32x128_w4"},
    {FAM_GENERIC,   64, 128, 1, 4, 3, 2, 0.164, 0.219, 1, "generic_64x128_w4"},
    {FAM_GENERIC,  256, 128, 4, 2, 1, 2, 0.232, 0.353, 1, "generic_256x128_w8"},
    {FAM_DIRECT,   256, 256, 2, 4, 1, 2, 0.779, 0.767, 1, "quad_256x256_w8"},
    {FAM_DIRECT,    64,  64, 2, 2, 3, 3, 0.180, 0.200, 1, "direct_64x64_w4_s3"},
};
constexpr int32_t kPingPongRowOnly = 13;
constexpr int32_t kNumConfigs = int32_t(sizeof(kConfigs) / sizeof(kConfigs[0]));

// The element-wise kernel (rows of under 16 bytes, strides past 4 MiB) that configurations 0
// and 1 run in place of the 16-byte loader: workgroups its registers allow on a CU, and what
// it sustains, as kConfigs says it of the loader.
struct ElementKernel {
    int32_t occupancy;
    double  eff_i8, eff_bf16;
};
constexpr ElementKernel kElementKernels[2] = {{2, 0.05, 0.07}, {1, 0.07, 0.10}};

// LDS bytes of one workgroup: `stages` copies of an A stage (bm x 128 B) and a
// B stage (bn x 128 B).  The analog of the paper's L1 budget (Eq. 5) without
// the C term: the output tile lives in registers, not in LDS.
constexpr int64_t lds_bytes(const TileConfig &c) {
    if (c.family == FAM_GEMV) return c.col_major_b ? 4 * int64_t(c.bn) : 4 * 4 * int64_t(c.bn);
    return int64_t(c.stages) * (int64_t(c.bm) + int64_t(c.bn)) * (c.family == FAM_RING ? kSlotKBytes : kStageKBytes);
}

// Whether gemm_tile_kernel's 16-byte loads, at any alignment, can read the operands:
// rows (K of A and of a column-major B, N of a row-major B) of at least 16 bytes, since
// a row's last piece is read ending at the row's end; and row strides of at most 4 MiB,
// which keeps a 256-row panel's byte offsets within 32 bits.
inline bool wide_rows_ok(int32_t dtype, int32_t trans_b, int64_t N, int64_t K, int64_t lda, int64_t ldb) {
    const int64_t e = dtype == DT_I8 ? 1 : 2, max_row_bytes = int64_t(1) << 22;
    return K * e >= 16 && (trans_b ? K : N) * e >= 16 && lda * e <= max_row_bytes && ldb * e <= max_row_bytes;
}

}  // namespace gemm
