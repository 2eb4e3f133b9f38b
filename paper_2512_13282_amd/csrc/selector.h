// selector.h -- shape-driven choice of kernel, tile and split-K (host only).
#pragma once

#include <stdint.h>

#include "configs.h"

namespace gemm {

struct Problem {
    int32_t dtype;
    int64_t M, N, K;
    int64_t lda, ldb, ldc;
    uintptr_t a_addr, b_addr, c_addr;
    int32_t trans_b = 0;   // 1: B stored column-major (N x K, row stride ldb)
    int32_t c_bytes = 4;   // of an output: 1 or 2 for int8 narrowed, whose slices cannot be added into C
};

struct Plan {
    int32_t config;      // index into kConfigs
    int32_t split_k;     // >= 1
    int32_t reduce_in_kernel;  // split-K reduction: REDUCE_SEPARATE, REDUCE_LAST_SLICE,
                               // REDUCE_ATOMIC or REDUCE_ATOMIC_FLAG (launch.h)
    int64_t k_chunk;     // K elements per slice (multiple of the stage depth)
    int64_t tiles_m, tiles_n;
    int64_t grid;
    int64_t workspace_bytes;
    double  traffic_bytes, t_comp_us, t_mem_us, t_total_us;
};

// Chip constants used by the model (AMD's published MI355X figures).
struct Chip {
    int32_t cus = 256;              // 8 XCDs x 32 CUs
    double  clock_hz = 2.4e9;
    double  i8_ops_per_clk_cu = 8192.0;   // dense int8 MFMA
    double  bf16_ops_per_clk_cu = 4096.0; // dense bf16 MFMA
    // Fitted with the configurations' efficiencies (configs.h) on measured plans: 283 calls of
    // all shapes, aligned and not, every configuration and split of each timed: the choice runs 1.03x the measured
    // best (with whole rounds of workgroups priced alike, as before, 1.10x).
    double  hbm_bytes_per_s = 5.1e12;     // compulsory traffic: streaming rate the kernels reach
    double  reread_bytes_per_s = 19.8e12;   // A/B tile re-reads mostly served by L2/MALL
    double  wg_cold_bytes_per_s = 31.2e9;  // one workgroup streaming its own strip of B (its loads
                                          // in flight over the latency)
    double  gemv_bytes_per_s = 18e9;      // ... one of the row-major GEMV, its launch and first loads included
    double  base_us = 0.367;              // of every plan
    double  separate_us = 3.61;           // split-K: the separate reduction's launch ...
    double  separate_slice_us = 0.25;     // ... each slice past 12 (its kernel: 4.5 us to 12, 7.7 at 24, 18 at 64),
    double  fill_us = 2.89;               // ... the fill kernel's ahead of atomic adds ...
    double  flag_us = 0.5, flag_row_us = 0.03;   // ... and waiting for the first slice's zeros, by the
                                          // tile's valid rows up to 24
    double  last_slice_below_us = 5.0;    // largest estimate that the last slice's own sum is taken at
    // The element-wise kernel: the rates of compulsory traffic and of re-reads, a round of
    // workgroups' first loads and C stores, and a launch, its own or beside it.
    double  element_hbm_bytes_per_s = 4.0e12, element_reread_bytes_per_s = 16.0e12;
    double  element_round_us = 2.0, element_launch_us = 5.0;
    // A GENERIC workgroup alone on a CU that holds four runs at this much under the full CU's rate.
    double  generic_solo = 1.05;
    // Prologue and C stores of a workgroup: per 1024 outputs of its tile, and each.
    double  us_per_kilo_output = 0.216, generic_us_per_kilo_output = 0.194;
    double  us_per_workgroup = 0.474, generic_us_per_workgroup = 0.166;
};

int32_t elem_bytes(int32_t dtype);
int32_t stage_k_elems(int32_t dtype);    // K elements per 128-byte LDS stage

// Whether the 16-byte vector loaders (MACRO / SKINNY) may run this problem.
bool vector_loads_ok(const Problem &p);

// What a call's addresses and strides allow, as bits: everything a plan depends on beside
// dtype, sizes, B's layout and an int8 call's output width (plans are cached by all of them).
enum : int32_t { ALIGN_VECTOR = 1, ALIGN_WIDE = 2 };
int32_t alignment_class(const Problem &p);

// Whether config `cfg` can run problem `p` at all.
bool config_applicable(const Problem &p, int32_t cfg);

// Evaluates the model for one (config, split) candidate.  reduce < 0 picks the
// cheaper split-K reduction by the model, 0 / 1 pins it.
Plan evaluate(const Problem &p, int32_t cfg, int32_t split, const Chip &chip = Chip(),
              int32_t reduce = -1);

// A plan measured fastest on the device for exactly this shape, if any applies
// (*reduce = -1 when the measurement left the reduction to the model).
bool tuned_plan(const Problem &p, int32_t *config, int32_t *split, int32_t *reduce);

// For M <= kNeighbourMaxM without a plan of its own: the plan measured for the nearest
// tuned M (same dtype, B layout, N and K, same number of tile rows), if any, with
// *reduce = -1 (the model picks the reduction).
constexpr int64_t kNeighbourMaxM = 2048;
bool neighbour_plan(const Problem &p, int32_t *config, int32_t *split, int32_t *reduce);

// Best plan: a tuned plan for this exact shape if one applies, else a neighbour's
// tuned plan (M <= kNeighbourMaxM), else the model's.  forced_family < 0 means any family; forced_config
// >= 0 pins the configuration; forced_split > 0 pins the split factor.
// Returns false if nothing applicable exists (only possible when forced).
// forced_reduce >= 0 pins the split-K reduction (0 separate kernel, 1 in-kernel).
// fixed_scratch: the best plan that fits_fixed_scratch (an unsplit one always does).
bool select_plan(const Problem &p, Plan *out, int32_t forced_family = -1,
                 int32_t forced_config = -1, int32_t forced_split = 0,
                 const Chip &chip = Chip(), int32_t forced_reduce = -1, bool fixed_scratch = false);

// Whether a plan's split-K partials and counters fit the fixed scratch (launch.h).
bool fits_fixed_scratch(const Plan &pl);

}  // namespace gemm
