// selector.cpp -- the paper's compute/memory balance model, transplanted.
//
// The paper picks its per-core tile by modelling compute time against data
// movement time and searching for the point where the two balance
// (Sec. 4.5.1, Eqs. 1-5; Sec. 4.5.2, Eqs. 6-10):
//   * off-chip reads of A scale as M*K*N*ty(A) / (width of the output tile in N)
//     and reads of B as M*K*N*ty(B) / (height in M) (Eqs. 6-7); C is written
//     once (Eq. 8);
//   * compute time is 2*M*K*N / (eff * peak) (Eq. 9), memory time is traffic /
//     bandwidth (Eq. 10), and the better tile is the one with the smaller
//     maximum of the two.
// On the GPU the same two terms decide between macro-tiles, with two terms
// the NPU does not have: wave quantization (output tiles are spread over 256
// CUs in whole rounds) and split-K partial traffic, which the paper avoids by
// never splitting K across cores (Sec. 4.2.1).  Split-K is therefore only
// chosen where the tile count alone cannot fill the chip.
#include "selector.h"
#include "launch.h"

#include <algorithm>
#include <cmath>

namespace gemm {

int32_t elem_bytes(int32_t dtype) { return dtype == DT_I8 ? 1 : 2; }

int32_t stage_k_elems(int32_t dtype) { return kStageKBytes / elem_bytes(dtype); }

static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

bool vector_loads_ok(const Problem &p) {
    // 16-byte pieces of A rows and B rows must start 16-byte aligned and never
    // straddle the end of a row; buffer offsets are 32-bit, so a 256-row panel
    // of either operand must span less than 2 GiB.  Rows of A and of a
    // column-major B hold K elements, rows of a row-major B hold N.
    const int64_t e = elem_bytes(p.dtype);
    const int64_t max_row_bytes = int64_t(1) << 22;
    const int64_t b_row_elems = p.trans_b ? p.K : p.N;
    return (p.a_addr % 16 == 0) && (p.b_addr % 16 == 0) &&
           ((p.lda * e) % 16 == 0) && ((p.ldb * e) % 16 == 0) &&
           ((p.K * e) % 16 == 0) && ((b_row_elems * e) % 16 == 0) &&
           p.lda * e <= max_row_bytes && p.ldb * e <= max_row_bytes;
}

int32_t alignment_class(const Problem &p) {
    return (vector_loads_ok(p) ? ALIGN_VECTOR : 0) |
           (wide_rows_ok(p.dtype, p.trans_b, p.N, p.K, p.lda, p.ldb) ? ALIGN_WIDE : 0);
}

bool config_applicable(const Problem &p, int32_t cfg) {
    if (cfg < 0 || cfg >= kNumConfigs) return false;
    const TileConfig &c = kConfigs[cfg];
    if (p.trans_b && !c.col_major_b) return false;
    if (c.family == FAM_GEMV) return p.M == 1 && (c.col_major_b != 0) == (p.trans_b != 0) && vector_loads_ok(p);
    // Configurations 0 and 1 also have an element-wise form for rows too short for 16-byte loads.
    if (c.family == FAM_GENERIC) return cfg < 2 || wide_rows_ok(p.dtype, p.trans_b, p.N, p.K, p.lda, p.ldb);
    return vector_loads_ok(p);
}

Plan evaluate(const Problem &p, int32_t cfg, int32_t split, const Chip &chip, int32_t reduce) {
    const TileConfig &c = kConfigs[cfg];
    const int64_t e = elem_bytes(p.dtype);
    const int64_t bk = stage_k_elems(p.dtype);
    Plan pl{};
    pl.config = cfg;
    pl.tiles_m = ceil_div(p.M, c.bm);
    pl.tiles_n = ceil_div(p.N, c.bn);
    const int64_t nkt = ceil_div(p.K, bk);  // K stages in total
    if (p.K == 0) {
        pl.split_k = 1;
        pl.k_chunk = 0;
    } else {
        int64_t s = std::max<int64_t>(1, std::min<int64_t>(split, nkt));
        pl.k_chunk = ceil_div(nkt, s) * bk;
        pl.split_k = int32_t(ceil_div(p.K, pl.k_chunk));
    }
    pl.grid = pl.tiles_m * pl.tiles_n * pl.split_k;

    // Configurations 0 and 1 run the element-wise kernel where the 16-byte loader cannot, and are
    // then priced as that kernel: its occupancy and rates, whole rounds of workgroups, 5 us for
    // every launch.  Over 157 such calls timed at every split the choice runs 1.01 times the best
    // (priced as the loader, 1.09: half as many slices, bf16 8192 x 7 x 8192 204 us against 127).
    const bool element =
        cfg < 2 && c.family == FAM_GENERIC && !wide_rows_ok(p.dtype, p.trans_b, p.N, p.K, p.lda, p.ldb);

    // Split-K reduction (REDUCE_* in launch.h).  Last slice: the last slice of each
    // tile reads the tile's partials, sixteen slices per round trip of 256 threads x 4
    // columns, at the end of the kernel.  Separate: one more launch streaming the
    // partial planes.  Atomic (int8 only): a fill launch ahead of the GEMM, the partial
    // tiles added into C, no workspace; the model's choice for int8, where it costs the
    // separate reduction's one extra launch without its partial planes (measured on the
    // skinny shapes: it matches or beats both others).  Atomic with C zeroed by each
    // tile's first slice (ring and GEMV kernels): no fill launch; the int8 choice for
    // those kernels, 2-12 % faster than the fill on the skinny shapes.
    double red_us = 0.0;
    pl.reduce_in_kernel = REDUCE_SEPARATE;
    if (pl.split_k > 1) {
        // Measured on the skinny bf16 shapes: the last-slice reduction beats the separate
        // kernel by 1-2 us at M = 1 and loses by 3-7 us at M = 16 (10-40 us at M = 64):
        // beside its three dependent round trips it issues the tile's device-coherent
        // partial stores, which grow with the tile's valid rows, and one workgroup reads
        // every other slice's partial tile.  The estimate decides between the two by a line of
        // its own, above the separate kernel's fitted price: over 295 pairs timed at M = 1 to 7
        // the last slice's sum is 0.3-0.5 us the faster below 3.9 us, the separate kernel by as
        // much from there to 5 and by 1.5 us past it; but with 12 or 16 slices at M = 2 and 3 the
        // last slice's is still 4-12 % the faster between 3.6 and 5.
        const int64_t rows = std::min<int64_t>(c.bm, p.M), cols = std::min<int64_t>(c.bn, p.N);
        const double in_kernel_us = 2.5 + 0.35 * double(rows) +
                                    double(pl.split_k - 1) * double(rows * cols) * 4.0 / chip.wg_cold_bytes_per_s * 1e6;
        int32_t mode = reduce >= 0 ? reduce
                     : p.dtype == DT_I8 ? ((c.family == FAM_RING || c.family == FAM_GEMV) ? REDUCE_ATOMIC_FLAG
                                                                                       : REDUCE_ATOMIC)
                     : (in_kernel_us <= chip.last_slice_below_us ? REDUCE_LAST_SLICE : REDUCE_SEPARATE);
        // Adds into C need an int32 C.  Narrowed int8 calls are priced without them, and by their own
        // width of C: with the int32 call's plans 57 of 340 ran more than 5 % slower (12 x 1024 x 320
        // 4.4 us whole, 7.8 in three slices summed apart).
        if ((mode == REDUCE_ATOMIC || mode == REDUCE_ATOMIC_FLAG) && (p.dtype != DT_I8 || p.c_bytes != 4))
            mode = REDUCE_SEPARATE;
        if (mode == REDUCE_ATOMIC_FLAG && c.family != FAM_RING && c.family != FAM_GEMV) mode = REDUCE_ATOMIC;
        pl.reduce_in_kernel = mode;
        // Atomic with slice 0's zeros: what the other slices wait for beyond their own work, by the
        // rows that are zeroed.  Priced at 0.4 us for all, the model split products of a few
        // microseconds that run faster whole (int8 80 x 256 x 256 5.6 us in two slices, 4.6 in one;
        // 385 x 1344 x 1184, B column-major, 8.0 and 6.0); at 1 us for all it ran a few rows whole
        // that gain by a split (1 x 2112 x 9856 10.0 us, 7.8 in two).  500 sampled int8 calls that
        // change plan between the first and this: 0.90 of the time, 18 of them more than 1.05.
        red_us = mode == REDUCE_LAST_SLICE ? in_kernel_us
               : mode == REDUCE_ATOMIC_FLAG ? chip.flag_us + chip.flag_row_us * double(std::min<int64_t>(rows, 24))
               : element ? chip.element_launch_us
               : mode == REDUCE_ATOMIC ? chip.fill_us
               : chip.separate_us + chip.separate_slice_us * double(std::max(0, pl.split_k - 12));
    }
    const bool partial_planes =
        pl.split_k > 1 && pl.reduce_in_kernel != REDUCE_ATOMIC && pl.reduce_in_kernel != REDUCE_ATOMIC_FLAG;
    pl.workspace_bytes = partial_planes ? int64_t(pl.split_k) * p.M * p.N * 4 : 0;

    // Compute: whole rounds of resident workgroups (wave quantization).
    const double ops_clk = p.dtype == DT_I8 ? chip.i8_ops_per_clk_cu : chip.bf16_ops_per_clk_cu;
    const double cu_rate = ops_clk * chip.clock_hz;                 // ops/s per CU
    const int32_t occupancy = element ? kElementKernels[cfg].occupancy : c.occupancy;
    const int64_t slots = int64_t(chip.cus) * occupancy;
    const int64_t rounds = ceil_div(pl.grid, slots);
    const double wg_ops = 2.0 * c.bm * c.bn * double(pl.k_chunk);
    const double eff = element ? (p.dtype == DT_I8 ? kElementKernels[cfg].eff_i8 : kElementKernels[cfg].eff_bf16)
                               : (p.dtype == DT_I8 ? c.eff_i8 : c.eff_bf16);
    const double wg_s = wg_ops / (cu_rate * eff / occupancy);
    // A CU's resident workgroups share its rate, so the last round costs what it leaves on the
    // fullest CU.  A workgroup alone then runs at a full CU's rate, which is how the timed calls
    // lie (charged a fifth or half more where two fit, the choice is 1.092 and 1.10 times the best
    // in place of 1.086), but for the small GENERIC tiles.
    const bool generic = c.family == FAM_GENERIC;
    const int64_t full = pl.grid / slots, last = pl.grid % slots;
    const double resident = last ? double(std::min<int64_t>(occupancy, ceil_div(last, chip.cus))) : 0.0;
    const double units = std::max(resident, generic && occupancy == 4 && last ? chip.generic_solo : 0.0);
    pl.t_comp_us = (element ? double(rounds) : double(full) + units / occupancy) * wg_s * 1e6;
    // Each workgroup's prologue and epilogue, which the K loop does not hide.
    const double overhead_us =
        element ? double(rounds) * chip.element_round_us / occupancy
                : (double(full * occupancy) + resident) *
                      ((generic ? chip.generic_us_per_kilo_output : chip.us_per_kilo_output) * double(c.bm * c.bn) / 1024.0 +
                       (generic ? chip.generic_us_per_workgroup : chip.us_per_workgroup));

    // Memory: compulsory traffic at HBM speed; tile re-reads (Eqs. 6-7 analog)
    // mostly from L2/MALL; split-K partials written and read back once, or added
    // into C once after C is zeroed.  Row-major B read in row pieces narrower than a
    // 128-byte line (64 int8 columns) costs whole lines: each tile's piece is half of a
    // line whose other half a neighbouring workgroup, often on another XCD, fetches again
    // (measured: the unsplit 64-column int8 plans at M = 32-64 run 1.3-1.7x the
    // 128-column ones).
    const double b_line = (!p.trans_b && c.bn * e < 128) ? 128.0 / double(c.bn * e) : 1.0;
    const double a_bytes = double(p.M) * p.K * e, b_bytes = double(p.K) * p.N * e * b_line;
    const double c_bytes = double(p.M) * p.N * p.c_bytes;
    const double a_reads = a_bytes * double(pl.tiles_n);
    const double b_reads = b_bytes * double(pl.tiles_m);
    const double ws = partial_planes ? 2.0 * double(pl.workspace_bytes)
                                     : (pl.split_k > 1 ? double(pl.split_k + 1) * p.M * p.N * 4 : 0.0);
    pl.traffic_bytes = a_reads + b_reads + c_bytes + ws;
    const double hbm = element ? chip.element_hbm_bytes_per_s : chip.hbm_bytes_per_s;
    const double reread = element ? chip.element_reread_bytes_per_s : chip.reread_bytes_per_s;
    pl.t_mem_us = ((a_bytes + b_bytes + c_bytes + ws) / hbm + (a_reads + b_reads - a_bytes - b_bytes) / reread) * 1e6;
    // With one tile row every workgroup streams a strip of B of its own from HBM, beside
    // its slice of A, at a rate one workgroup's loads in flight bound: too few workgroups
    // cannot reach the HBM rate (measured: 112 unsplit workgroups of 32 x 128 at M = 16
    // take 1.4x the time of 224 split ones).
    // The row-major GEMV walks its rows one after another whatever their width: columns past N
    // save it nothing (1 x 64 x 11264 int8 in eight slices 40 us, a 32-row ring tile 7.2).  It
    // streams at 18 GB/s, its launch included (at the tiles' rate in its price, 150 int8 calls
    // that it was chosen for ran 1.17 times the ring tiles' time).
    if (pl.tiles_m == 1 && p.K > 0) {
        const int64_t cols = c.family == FAM_GEMV ? c.bn : std::min<int64_t>(c.bn, p.N);
        const double wg_bytes = double(std::min<int64_t>(pl.k_chunk, p.K)) *
                                (double(std::min<int64_t>(c.bm, p.M)) + double(cols) * b_line) * e;
        const double rate = c.family == FAM_GEMV && !p.trans_b ? chip.gemv_bytes_per_s : chip.wg_cold_bytes_per_s;
        pl.t_mem_us = std::max(pl.t_mem_us, double(rounds) * wg_bytes / rate * 1e6);
    }

    // The longer of the two where they differ; where they are alike, more, since they hide each other
    // in part only: by the 6-norm, on 700 calls timed at their 14 likeliest plans, the choice runs
    // 1.04 times the best (1.06 by the larger one).  With one tile row the workgroups' rate above
    // bounds both.
    const double t_main = element || pl.tiles_m == 1 ? std::max(pl.t_comp_us, pl.t_mem_us)
                                                     : std::pow(std::pow(pl.t_comp_us, 6) + std::pow(pl.t_mem_us, 6), 1.0 / 6.0);
    pl.t_total_us = t_main + overhead_us + (element ? chip.element_launch_us : chip.base_us) + red_us;
    return pl;
}

// Plans measured fastest on the device for specific shapes (tune.py).
struct TunedPlan {
    int32_t dtype;
    int64_t M, N, K;
    int32_t config, split;
    int32_t reduce;      // -1: the model's choice
    int32_t trans_b;     // B layout the plan was measured with (1: column-major)
};
static const TunedPlan kTuned[] = {
#include "tuned_plans.inc"
    {-1, 0, 0, 0, 0, 0, -1, 0},   // sentinel
};

bool tuned_plan(const Problem &p, int32_t *config, int32_t *split, int32_t *reduce) {
    for (const TunedPlan &t : kTuned) {
        if (t.trans_b == p.trans_b && t.dtype == p.dtype && t.M == p.M && t.N == p.N && t.K == p.K &&
            t.config >= 0 && t.config < kNumConfigs && config_applicable(p, t.config)) {
            *config = t.config;
            *split = t.split;
            *reduce = t.reduce;
            return true;
        }
    }
    return false;
}

// A shape with M <= kNeighbourMaxM and no measured plan of its own borrows the plan
// measured for the nearest M at the same dtype, B layout, N and K.  Only plans whose
// tile covers the same number of rows of C at both sizes qualify, so the borrowed plan
// runs the same grid of tiles over the same reads of B as where it was measured (few
// rows: reading B is most of the work and does not depend on M; more: each tile's work
// barely changes); among them the nearest M on a log scale, the larger on a tie.  The split-K reduction is left to the model,
// whose price for it grows with the rows summed (at M = 1-4 the in-kernel sum wins over
// the separate kernel that a plan measured at M = 16 may have used).
bool neighbour_plan(const Problem &p, int32_t *config, int32_t *split, int32_t *reduce) {
    if (p.M < 1 || p.M > kNeighbourMaxM) return false;
    const TunedPlan *best = nullptr;
    double best_d = 0.0;
    for (const TunedPlan &t : kTuned) {
        if (t.dtype != p.dtype || t.trans_b != p.trans_b || t.N != p.N || t.K != p.K) continue;
        if (t.M < 1 || t.M > kNeighbourMaxM || t.config < 0 || t.config >= kNumConfigs) continue;
        const int64_t bm = kConfigs[t.config].bm;
        if ((t.M + bm - 1) / bm != (p.M + bm - 1) / bm || !config_applicable(p, t.config)) continue;
        const double d = std::fabs(std::log(double(t.M) / double(p.M)));
        if (!best || d < best_d - 1e-12 || (d <= best_d + 1e-12 && t.M > best->M)) {
            best = &t;
            best_d = d;
        }
    }
    if (!best) return false;
    *config = best->config;
    *split = best->split;
    *reduce = -1;
    return true;
}

// Longest rows of K (bytes) at which a GENERIC tile competes with the vectorised ones: a grid that
// leaves a compute unit too few of them to hide first loads is passed by for longer rows.
//   64 x 64, B column-major: 256 below three workgroups a compute unit (400 calls of up to 2 KiB
//     0.92 of its time on the narrow ring tiles and the three-stage one; at 256 alike; from three
//     on 0.96 of the others' time, 59367 x 64 x 960 14.1 us against 16.8).  Row-major calls take
//     0.9-0.96 of the time on it at any such length.
//   64 x 128: 128 below two workgroups a compute unit (500 calls 0.94 without it; with more, 150
//     calls 1.01 without it).
//   32 x 128: 128 (100 calls past it 0.93, mostly on the ring tile of its shape).
static int64_t generic_row_bytes(const Problem &p, int32_t cfg, const Chip &chip) {
    const TileConfig &c = kConfigs[cfg];
    if (c.bm > 64) return 0;
    if (c.bn == 128 && c.bm == 32) return 128;
    const int64_t per_cu = c.bn == 128 ? 2 : 3;
    if (ceil_div(p.M, c.bm) * ceil_div(p.N, c.bn) >= per_cu * chip.cus) return 2048;
    return c.bn == 128 ? 128 : p.trans_b ? 256 : 2048;
}

bool fits_fixed_scratch(const Plan &pl) {
    const int64_t counters = pl.split_k > 1 && pl.reduce_in_kernel == REDUCE_LAST_SLICE ? pl.tiles_m * pl.tiles_n : 0;
    return pl.workspace_bytes <= kStaticScratchBytes - kScratchCounterBytes && counters * 4 <= kScratchCounterBytes;
}

bool select_plan(const Problem &p, Plan *out, int32_t forced_family, int32_t forced_config,
                 int32_t forced_split, const Chip &chip, int32_t forced_reduce, bool fixed_scratch) {
    static const int32_t kSplits[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64};
    if (forced_family < 0 && forced_config < 0 && forced_split <= 0 && forced_reduce < 0) {
        int32_t cfg, split, reduce;
        if (tuned_plan(p, &cfg, &split, &reduce) || neighbour_plan(p, &cfg, &split, &reduce)) {
            *out = evaluate(p, cfg, split, chip, reduce);
            if (!fixed_scratch || fits_fixed_scratch(*out)) return true;
        }
    }
    bool found = false;
    Plan best{};
    for (int32_t cfg = 0; cfg < kNumConfigs; ++cfg) {
        if (forced_config >= 0 && cfg != forced_config) continue;
        if (forced_family >= 0 && kConfigs[cfg].family != forced_family) continue;
        if (!config_applicable(p, cfg)) continue;
        if (forced_family < 0 && forced_config < 0 && cfg == kPingPongRowOnly) continue;   // 44 is the same kernel
        // Where vectorised kernels can run, GENERIC ones compete only for short K, where a tile is
        // mostly prologue and C stores and their small tiles (64 rows at most, up to four to a CU)
        // win: bf16 25440 x 64 x 64 8.6 -> 4.6 us, int8 43840 x 64 x 128 9.2 -> 5.0 us.
        if (forced_family < 0 && forced_config < 0 && kConfigs[cfg].family == FAM_GENERIC && vector_loads_ok(p) &&
            p.K * elem_bytes(p.dtype) > generic_row_bytes(p, cfg, chip))
            continue;
        // The three-stage 64 x 64 kernel is for tiles more than half full: at M = 6 (bf16
        // 6 x 12288 x 6592, B row-major) it took 43 us against 33 of a 32-row tile, at M = 50
        // (50 x 1600 x 10944) 12.8 against 15.6.  A column-major B moves the line only where it
        // was measured: measured plans take the kernel from M = 8 on there, and the M = 2 to 31
        // that borrow them run 0.94 of the time of the 32-row ring tiles (130 calls); but where
        // the model has to price it, 150 calls of M = 2 to 32 with other N and K run 1.05 times.
        if (forced_family < 0 && forced_config < 0 && kConfigs[cfg].family == FAM_DIRECT && kConfigs[cfg].bm == 64 &&
            p.M <= 32)
            continue;
        for (int32_t s : kSplits) {
            if (forced_split > 0 && s != 1) break;
            const int32_t split = forced_split > 0 ? forced_split : s;
            Plan pl = evaluate(p, cfg, split, chip, forced_reduce);
            if (forced_split <= 0 && pl.split_k != split) continue;   // duplicate of a smaller split
            if (fixed_scratch && !fits_fixed_scratch(pl)) continue;
            // Ties (memory-bound shapes, where every tile of one size moves the same
            // bytes) go to the plan with the shorter compute time: the faster kernel.
            const bool tie = found && std::abs(pl.t_total_us - best.t_total_us) <= 1e-9 * best.t_total_us;
            if (!found || (!tie && pl.t_total_us < best.t_total_us) ||
                (tie && pl.t_comp_us < best.t_comp_us * (1.0 - 1e-9))) {
                best = pl;
                found = true;
            }
        }
    }
    if (found) *out = best;
    return found;
}

}  // namespace gemm
