// kern_direct.h -- direct-to-LDS kernels with two 128-byte K stages: all waves in
// step (gemm_lds_kernel) and two wave groups in turn (gemm_pingpong_kernel).
#pragma once

#include "gemm_common.h"

namespace gemm {

// ---------------------------------------------------------------------------
// Direct-to-LDS kernel (gfx950): both operands go from global memory straight
// into LDS with buffer_load ... lds, and B's K-contiguous MFMA fragments are
// produced by LDS transpose reads (ds_read_b64_tr_b16 / _b8) instead of an
// in-register transpose.  The K loop then holds only loads, LDS reads, MFMAs
// and one barrier per stage.
//
// LDS, per stage: A as BM rows of 128 K-bytes (16-byte chunks XOR-swizzled by
// swz(c, row)), B untransposed as BK rows (k) of BN*E bytes (chunks swizzled by
// a function of k mod 4 (bf16) or k mod 8 (int8), matched to the row sets the
// transpose reads touch together).
//
// Transpose read, per 16-lane group (lane g within the group): every lane
// supplies the address of one 8-byte piece; lane g receives column g of the
// block formed by the group's pieces -- b16: 4 rows x 16 columns, lane g
// addresses row g/4, columns 4(g%4)..+3; b8: 8 rows x 16 columns, lane g
// addresses row g/2, columns 8(g%2)..+7.
// ---------------------------------------------------------------------------
template <int DT, int BM, int BN, int WM, int WN, int WAVES_PER_EU, bool BT = false>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * WM * WN, 64 * WM * WN),
                          amdgpu_waves_per_eu(WAVES_PER_EU, WAVES_PER_EU)))
void gemm_lds_kernel(KernelArgs args) {
    using acc_vec = typename Types<DT>::acc_vec;
    using out_t = typename Types<DT>::out_t;
    constexpr int E = Types<DT>::E;
    constexpr int VECE = 16 / E;
    constexpr int BK = kStageKBytes / E;                  // K elements per stage
    constexpr int THREADS = 64 * WM * WN;
    constexpr int WAVES = WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int A_STAGE = BM * kStageKBytes;            // bytes
    // Row-major B sits in LDS as BK rows (k) of BN*E bytes; column-major B (BT)
    // as BN rows (n) of 128 K-bytes, exactly like A.
    constexpr int B_PITCH = BT ? kStageKBytes : BN * E;   // bytes per B row in LDS
    constexpr int B_STAGE = BN * kStageKBytes;
    constexpr int A_INSTR = A_STAGE / 1024 / WAVES;       // 1 KiB per wave-wide load
    constexpr int B_INSTR = B_STAGE / 1024 / WAVES;
    constexpr int B_ROWS_PER_KB = 1024 / B_PITCH;         // B rows covered by one wave-wide load
    static_assert(A_INSTR >= 1 && A_INSTR * 1024 * WAVES == A_STAGE, "A stage split");
    static_assert(B_INSTR >= 1 && B_INSTR * 1024 * WAVES == B_STAGE, "B stage split");
    static_assert(B_PITCH <= 1024 && 1024 % B_PITCH == 0, "B row pitch");

    // One LDS array per stage buffer and operand: with every access naming a
    // fixed array, the compiler can tell the direct-to-LDS writes of one stage
    // from the fragment reads of the other and does not serialise them.
    __shared__ __attribute__((aligned(1024))) uint8_t a_lds0[A_STAGE];
    __shared__ __attribute__((aligned(1024))) uint8_t a_lds1[A_STAGE];
    __shared__ __attribute__((aligned(1024))) uint8_t b_lds0[B_STAGE];
    __shared__ __attribute__((aligned(1024))) uint8_t b_lds1[B_STAGE];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wave_m = wave / WN, wave_n = wave % WN;

    int tm, tn, slice;
    map_tile(args, tm, tn, slice);
    const int64_t M = args.M, N = args.N;
    const int64_t m0 = int64_t(tm) * BM, n0 = int64_t(tn) * BN;
    const int64_t k_begin = int64_t(slice) * args.k_chunk;
    int64_t k_end = k_begin + args.k_chunk;
    if (k_end > args.K) k_end = args.K;
    const int nk = k_end > k_begin ? int((k_end - k_begin + BK - 1) / BK) : 0;
    const int64_t lda_b = args.lda * E, ldb_b = args.ldb * E;

    // ---- global source offsets of this lane's 16-byte pieces (constant over K) ----
    // A load i of this wave fills LDS bytes [(i*WAVES + wave) KiB, +1 KiB): lane L
    // writes physical chunk L%8 of row (i*WAVES + wave)*8 + L/8, which holds the
    // logical chunk c = (L%8) ^ f(row).  Rows at or past M are masked by the
    // resource size (rows_valid * lda bytes from the tile's first row).
    const int64_t a_rows_valid = (M - m0) < BM ? (M - m0) : BM;
    const uint32_t a_bytes = uint32_t(a_rows_valid * lda_b);
    uint32_t a_voff[A_INSTR];
    int a_chunk[A_INSTR];
#pragma unroll
    for (int i = 0; i < A_INSTR; ++i) {
        const int row = (i * WAVES + wave) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ((row ^ (row >> 3)) & 7);
        a_chunk[i] = c;
        a_voff[i] = uint32_t(row * lda_b + c * 16);
    }
    // B load i fills LDS bytes [(i*WAVES + wave) KiB, +1 KiB) of the B stage: lane L
    // writes physical chunk p = L % B_CPR of row (i*WAVES+wave)*B_ROWS_PER_KB + L / B_CPR,
    // holding logical chunk p ^ bswz(row).  Columns at or past N get an out-of-range
    // offset; K rows past the slice end are masked by the resource size.
    // Column-major B (BT): the same scheme as A over BN rows (n) of the N x K
    // matrix; rows at or past N are masked by the resource size.
    constexpr int B_CPR = B_PITCH / 16;                   // chunks per B row
    static_assert(BT || B_CPR >= 16, "transpose-read swizzle needs rows of at least 16 chunks");
    const int64_t b_rows_valid = (N - n0) < BN ? (N - n0) : BN;
    const uint32_t bt_bytes = uint32_t(b_rows_valid * ldb_b);
    uint32_t b_voff[B_INSTR];
    int b_chunk[B_INSTR];
#pragma unroll
    for (int i = 0; i < B_INSTR; ++i) {
        if constexpr (BT) {
            const int row = (i * WAVES + wave) * 8 + (lane >> 3);
            const int c = (lane & 7) ^ ((row ^ (row >> 3)) & 7);
            b_chunk[i] = c;
            b_voff[i] = uint32_t(row * ldb_b + c * 16);
        } else {
            const int row = (i * WAVES + wave) * B_ROWS_PER_KB + lane / B_CPR;
            const int c = (lane % B_CPR) ^ bswz<DT>(row);
            b_chunk[i] = 0;
            b_voff[i] = (n0 + int64_t(c) * VECE < N) ? uint32_t(row * ldb_b + c * 16) : kOOB;
        }
    }
    const uint8_t *const a_base = static_cast<const uint8_t *>(args.A) + (m0 * args.lda + k_begin) * E;
    const uint8_t *const b_base = static_cast<const uint8_t *>(args.B) +
                                  (BT ? n0 * args.ldb + k_begin : k_begin * args.ldb + n0) * E;
    // B resource of stage kt; `rows` valid K rows bound row-major B only.
    auto b_rsrc = [&](int kt, int64_t rows) {
        if constexpr (BT) return make_rsrc(b_base + int64_t(kt) * kStageKBytes, bt_bytes);
        else return make_rsrc(b_base + int64_t(kt) * BK * ldb_b, uint32_t(rows * ldb_b));
    };
    const int64_t k_len = k_end - k_begin;

    // Issues the loads of stage kt into LDS buffer BUF.  Full stages use the
    // precomputed offsets as they are; only a partial last stage (and stages past
    // the end, which load nothing) pays for the per-chunk K mask.
    auto load_stage = [&](int kt, auto buf_c) {
        constexpr int BUF = decltype(buf_c)::value;
        const int64_t rem = k_len - int64_t(kt) * BK;
        const __amdgpu_buffer_rsrc_t ra = make_rsrc(a_base + int64_t(kt) * kStageKBytes, a_bytes);
        const int64_t rows = rem <= 0 ? 0 : (rem < BK ? rem : BK);
        const __amdgpu_buffer_rsrc_t rb = b_rsrc(kt, rows);
        uint8_t *const as = BUF ? a_lds1 : a_lds0;
        uint8_t *const bs = BUF ? b_lds1 : b_lds0;
        if (rem >= BK) {
#pragma unroll
            for (int i = 0; i < A_INSTR; ++i) {
                load_lds16(ra, as + (i * WAVES + wave) * 1024, a_voff[i]);
                if (i < B_INSTR) load_lds16(rb, bs + (i * WAVES + wave) * 1024, b_voff[i]);
            }
#pragma unroll
            for (int i = A_INSTR; i < B_INSTR; ++i) load_lds16(rb, bs + (i * WAVES + wave) * 1024, b_voff[i]);
        } else {
#pragma unroll
            for (int i = 0; i < A_INSTR; ++i) {
                const uint32_t off = int64_t(a_chunk[i]) * VECE < rem ? a_voff[i] : kOOB;
                load_lds16(ra, as + (i * WAVES + wave) * 1024, off);
            }
#pragma unroll
            for (int i = 0; i < B_INSTR; ++i) {
                // Column-major B masks its K tail per chunk, as A does; row-major B by rows.
                const uint32_t off = (!BT || int64_t(b_chunk[i]) * VECE < rem) ? b_voff[i] : kOOB;
                load_lds16(rb, bs + (i * WAVES + wave) * 1024, off);
            }
        }
    };

    // A full stage's loads issued in two halves, at the start of k-steps 0 and 1:
    // issuing all of them in one burst backs up the vector memory path and
    // stalls the issuing waves (and their MFMAs) for longer than the spread
    // costs in latency.  A partial last stage is loaded whole with part 0.
    auto load_stage_part = [&](int kt, auto buf_c, int part) {
        constexpr int BUF = decltype(buf_c)::value;
        const int64_t rem = k_len - int64_t(kt) * BK;
        if (rem < BK) {
            if (part == 0) load_stage(kt, buf_c);
            return;
        }
        const __amdgpu_buffer_rsrc_t ra = make_rsrc(a_base + int64_t(kt) * kStageKBytes, a_bytes);
        const __amdgpu_buffer_rsrc_t rb = b_rsrc(kt, BK);
        uint8_t *const as = BUF ? a_lds1 : a_lds0;
        uint8_t *const bs = BUF ? b_lds1 : b_lds0;
#pragma unroll
        for (int i = 0; i < (A_INSTR > B_INSTR ? A_INSTR : B_INSTR); ++i) {
            if ((i & 1) != part) continue;
            if (i < A_INSTR) load_lds16(ra, as + (i * WAVES + wave) * 1024, a_voff[i]);
            if (i < B_INSTR) load_lds16(rb, bs + (i * WAVES + wave) * 1024, b_voff[i]);
        }
    };

    // ---- fragment offsets (lane constants; the k-step and tile index only add immediates) ----
    const int frag_row = lane & 31;
    const int frag_half = lane >> 5;
    const int wrow0 = wave_m * (BM / WM);
    const int wcol0 = wave_n * (BN / WN);
    // A tile i, k-step s: row r_i = wrow0 + 32 i + frag_row, chunk 2s + half, swizzled by
    // f(r_i) = f(r_0) ^ 4 (i & 1).  Offset = r_0*128 + 4096 i + 16 ((2s + half) ^ f(r_0) ^ 4(i&1)).
    const int r0 = wrow0 + frag_row;
    const int f0 = (r0 ^ (r0 >> 3)) & 7;
    int a_fo[2][4];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int st = 0; st < 4; ++st) a_fo[p][st] = r0 * kStageKBytes + 16 * ((2 * st + frag_half) ^ f0 ^ (4 * p));
    // B transpose reads: group = lane/16, g = lane%16.
    // bf16: rows 4*h + g/4 (+8 for the upper K half), byte columns 8*(g%4) (+32 for odd groups)
    // int8: rows 8*h + g/2 (+16 for the upper K half), byte columns 8*(g%2) (+16 for odd groups)
    // The row's swizzle depends only on g (k mod 4 or 8), so tile j, read h, k-step s
    // is b_fo[j] + (s*KSTEP + h*TR_ROWS) * B_PITCH.
    const int grp = lane >> 4, g16 = lane & 15;
    constexpr int TR_ROWS = DT == DT_BF16 ? 4 : 8;        // rows per transpose read
    constexpr int KSTEP = 32 / E;                         // K elements per MFMA
    const int tr_row = DT == DT_BF16 ? (g16 >> 2) : (g16 >> 1);
    const int tr_colb = (DT == DT_BF16 ? (g16 & 3) * 8 : (g16 & 1) * 8) + (grp & 1) * 16 * E;
    const int tr_khalf = (grp >> 1) * (KSTEP / 2);
    const int bz = bswz<DT>(tr_row);
    int b_fo[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int colb = (wcol0 + j * 32) * E + tr_colb;
        b_fo[j] = (tr_khalf + tr_row) * B_PITCH + (((colb >> 4) ^ bz) << 4) + (colb & 15);
    }
    // Column-major B: fragments are 16-byte reads of K-contiguous rows, as for A.
    const int rb0 = wcol0 + frag_row;
    const int fb0 = (rb0 ^ (rb0 >> 3)) & 7;
    int bt_fo[2][4];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int st = 0; st < 4; ++st) bt_fo[p][st] = rb0 * kStageKBytes + 16 * ((2 * st + frag_half) ^ fb0 ^ (4 * p));

    u32x4_t fa[2][TM], fb[2][TN];
    auto load_frags = [&](auto buf_c, auto s_c, auto slot_c) {
        constexpr int BUF = decltype(buf_c)::value;
        constexpr int S = decltype(s_c)::value;
        constexpr int SLOT = decltype(slot_c)::value;
        const uint8_t *const as = BUF ? a_lds1 : a_lds0;
        const uint8_t *const bs = BUF ? b_lds1 : b_lds0;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fa[SLOT][i] = *reinterpret_cast<const u32x4_t *>(as + a_fo[i & 1][S] + 4096 * i);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if constexpr (BT) {
                fb[SLOT][j] = *reinterpret_cast<const u32x4_t *>(bs + bt_fo[j & 1][S] + 4096 * j);
            } else {
                const u32x2_t lo = lds_read_tr<DT>(bs + b_fo[j] + (S * KSTEP) * B_PITCH);
                const u32x2_t hi = lds_read_tr<DT>(bs + b_fo[j] + (S * KSTEP + TR_ROWS) * B_PITCH);
                fb[SLOT][j] = u32x4_t{lo[0], lo[1], hi[0], hi[1]};
            }
        }
    };

    acc_vec acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = acc_vec{};
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[1][i] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[1][j] = u32x4_t{0u, 0u, 0u, 0u};

    auto mfma_slot = [&](auto slot_c) {
        constexpr int SLOT = decltype(slot_c)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = mfma32<DT>(fa[SLOT][i], fb[SLOT][j], acc[i][j]);
    };

    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;

    // One stage (buffer BUF holds stage kt, visible).  On entry slot 1 holds the
    // fragments of the previous stage's last k-step, whose MFMAs run here, under
    // the latency of this stage's first LDS reads; on exit slot 1 holds this
    // stage's last k-step and every wave has finished reading buffer BUF.
    auto stage = [&](int kt, auto buf_c) {
        constexpr int BUF = decltype(buf_c)::value;
        using OTHER = std::integral_constant<int, 1 - BUF>;
        load_stage_part(kt + 1, OTHER{}, 0);
        __builtin_amdgcn_sched_barrier(0);
        load_frags(buf_c, I0{}, I0{});
        mfma_slot(I1{});
        __builtin_amdgcn_sched_barrier(0);
        load_stage_part(kt + 1, OTHER{}, 1);
        __builtin_amdgcn_sched_barrier(0);
        load_frags(buf_c, I1{}, I1{});
        mfma_slot(I0{});
        __builtin_amdgcn_sched_barrier(0);
        load_frags(buf_c, I2{}, I0{});
        mfma_slot(I1{});
        __builtin_amdgcn_sched_barrier(0);
        load_frags(buf_c, I3{}, I1{});
        mfma_slot(I0{});
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };

    if (nk > 0) {
        load_stage(0, I0{});
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
        stage(kt, I0{});
        stage(kt + 1, I1{});
    }
    if (kt < nk) stage(kt, I0{});
    mfma_slot(I1{});

    __shared__ int s_last;
    store_tile<DT, BM, BN, TM, TN>(args, acc, tm, tn, slice, m0 + wrow0, n0 + wcol0, lane, s_last);
}

// ---------------------------------------------------------------------------
// The same kernel for few rows (memory-bound shapes): narrow tiles, NS stages of 128
// K-bytes in flight, two or more workgroups to a CU.  The narrow ring kernels read a
// column-major B in 64-byte pieces, half lines that cost HBM and the L2 a whole request
// each; this one reads whole 128-byte lines and keeps (NS - 1) stages of each workgroup
// on the way.  Each iteration waits only for its own stage (vmcnt counts the younger
// stages' loads), then one barrier publishes it and retires the buffer that the next
// loads overwrite; stages past the end of K load zeros through an empty resource, so
// every iteration counts the same loads.  LDS layouts and fragment reads are
// gemm_lds_kernel's (row-major B by the ring's row-width swizzles).
//
// Compiled as 64 x 64 with three stages, three workgroups to a CU.  Measured with B from
// HBM, against the best of the ring kernels: bf16 48 x 11008 x 4096 column-major 25.5
// against 29.5 us, 64 x 14336 x 4096 column-major bf16 31.8 against 33.3 and int8 17.8
// against 18.8, bf16 32 x 4096 x 4096 row-major 11.5 against 12.2; 32 x 128 and 64 x 128
// tiles were behind it.
// ---------------------------------------------------------------------------
template <int DT, int BM, int BN, int WM, int WN, int WAVES_PER_EU, bool BT, int NS>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * WM * WN, 64 * WM * WN),
                          amdgpu_waves_per_eu(WAVES_PER_EU, WAVES_PER_EU)))
void gemm_lds_kernel(KernelArgs args) {
    using acc_vec = typename Types<DT>::acc_vec;
    constexpr int E = Types<DT>::E;
    constexpr int VECE = 16 / E;
    constexpr int BK = kStageKBytes / E;
    constexpr int WAVES = WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int A_STAGE = BM * kStageKBytes, B_STAGE = BN * kStageKBytes;
    constexpr int B_PITCH = BT ? kStageKBytes : BN * E;
    constexpr int B_CPR = B_PITCH / 16;
    constexpr int A_INSTR = A_STAGE / 1024 / WAVES, B_INSTR = B_STAGE / 1024 / WAVES;
    constexpr int LPS = A_INSTR + B_INSTR;                 // loads per wave per stage
    static_assert(A_INSTR >= 1 && A_INSTR * 1024 * WAVES == A_STAGE, "A stage split");
    static_assert(B_INSTR >= 1 && B_INSTR * 1024 * WAVES == B_STAGE, "B stage split");
    static_assert(NS >= 3 && (NS - 1) * LPS < 64, "loads in flight must fit vmcnt");

    __shared__ __attribute__((aligned(1024))) uint8_t lds[NS][A_STAGE + B_STAGE];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = wave / WN, wave_n = wave % WN;

    int tm, tn, slice;
    map_tile(args, tm, tn, slice);
    const int64_t M = args.M, N = args.N;
    const int64_t m0 = int64_t(tm) * BM, n0 = int64_t(tn) * BN;
    const int64_t k_begin = int64_t(slice) * args.k_chunk;
    int64_t k_end = k_begin + args.k_chunk;
    if (k_end > args.K) k_end = args.K;
    const int k_len = k_end > k_begin ? int(k_end - k_begin) : 0;
    const int nk = (k_len + BK - 1) / BK;
    const int64_t lda_b = args.lda * E, ldb_b = args.ldb * E;

    const int64_t a_rows_valid = (M - m0) < BM ? (M - m0) : BM;
    const uint32_t a_bytes = uint32_t(a_rows_valid * lda_b);
    uint32_t a_voff[A_INSTR];
    int a_chunk[A_INSTR];
#pragma unroll
    for (int i = 0; i < A_INSTR; ++i) {
        const int row = (i * WAVES + wave) * 8 + (lane >> 3);
        a_chunk[i] = swz(lane & 7, row);
        a_voff[i] = uint32_t(row * lda_b + a_chunk[i] * 16);
    }
    const int64_t b_rows_valid = (N - n0) < BN ? (N - n0) : BN;
    const uint32_t bt_bytes = uint32_t(b_rows_valid * ldb_b);
    uint32_t b_voff[B_INSTR];
    int b_chunk[B_INSTR];
#pragma unroll
    for (int i = 0; i < B_INSTR; ++i) {
        if constexpr (BT) {
            const int row = (i * WAVES + wave) * 8 + (lane >> 3);
            b_chunk[i] = swz(lane & 7, row);
            b_voff[i] = uint32_t(row * ldb_b + b_chunk[i] * 16);
        } else {
            const int row = (i * WAVES + wave) * (1024 / B_PITCH) + lane / B_CPR;
            const int c = (lane % B_CPR) ^ ring_bswz<DT, B_CPR>(row);
            b_chunk[i] = 0;
            b_voff[i] = (n0 + int64_t(c) * VECE < N) ? uint32_t(row * ldb_b + c * 16) : kOOB;
        }
    }
    const uint8_t *const a_base = static_cast<const uint8_t *>(args.A) + (m0 * args.lda + k_begin) * E;
    const uint8_t *const b_base = static_cast<const uint8_t *>(args.B) +
                                  (BT ? n0 * args.ldb + k_begin : k_begin * args.ldb + n0) * E;

    auto load_stage = [&](int kt, auto buf_c) {
        constexpr int BUF = decltype(buf_c)::value;
        const int rem = k_len - kt * BK;
        const uint32_t dst = lds_addr(lds[BUF]) + uint32_t(wave) * 1024u;
        const i32x4_t ra = ring_rsrc(a_base + int64_t(kt) * kStageKBytes, rem > 0 ? a_bytes : 0u);
#pragma unroll
        for (int i = 0; i < A_INSTR; ++i)
            ring_load16(ra, dst + i * (WAVES * 1024), a_chunk[i] * VECE < rem ? a_voff[i] : kOOB);
        i32x4_t rb;
        if constexpr (BT) {
            rb = ring_rsrc(b_base + int64_t(kt) * kStageKBytes, rem > 0 ? bt_bytes : 0u);
        } else {
            const int rows = rem <= 0 ? 0 : (rem < BK ? rem : BK);
            // readfirstlane: the compiler otherwise clamps the (uniform) size on the vector unit
            rb = ring_rsrc(b_base + int64_t(kt) * BK * ldb_b,
                           uint32_t(__builtin_amdgcn_readfirstlane(int(rows * ldb_b))));
        }
#pragma unroll
        for (int i = 0; i < B_INSTR; ++i)
            ring_load16(rb, dst + A_STAGE + i * (WAVES * 1024), (!BT || b_chunk[i] * VECE < rem) ? b_voff[i] : kOOB);
    };

    const int frag_row = lane & 31, frag_half = lane >> 5;
    const int wrow0 = wave_m * (BM / WM), wcol0 = wave_n * (BN / WN);
    const int r0 = wrow0 + frag_row, rb0 = wcol0 + frag_row;
    int a_fo[4], bt_fo[4];                                 // k-step st of the wave's first 32 rows
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        a_fo[st] = r0 * kStageKBytes + 16 * swz(2 * st + frag_half, r0);
        bt_fo[st] = rb0 * kStageKBytes + 16 * swz(2 * st + frag_half, rb0);
    }
    const int grp = lane >> 4, g16 = lane & 15;            // transpose reads, as above
    constexpr int TR_ROWS = DT == DT_BF16 ? 4 : 8;
    constexpr int KSTEP = 32 / E;
    const int tr_row = DT == DT_BF16 ? (g16 >> 2) : (g16 >> 1);
    const int tr_colb = (DT == DT_BF16 ? (g16 & 3) * 8 : (g16 & 1) * 8) + (grp & 1) * 16 * E;
    const int tr_khalf = (grp >> 1) * (KSTEP / 2);
    const int bz = BT ? 0 : ring_bswz<DT, B_CPR>(tr_row);
    int b_fo[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int colb = (wcol0 + j * 32) * E + tr_colb;
        b_fo[j] = (tr_khalf + tr_row) * B_PITCH + (((colb >> 4) ^ bz) << 4) + (colb & 15);
    }

    acc_vec acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = acc_vec{};

    auto iteration = [&](int kt, auto buf_c) {
        constexpr int BUF = decltype(buf_c)::value;
        ring_barrier<(NS - 2) * LPS>();
        load_stage(kt + NS - 1, std::integral_constant<int, (BUF + NS - 1) % NS>{});
        const uint8_t *const as = lds[BUF];
        const uint8_t *const bs = as + A_STAGE;
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            u32x4_t fa[TM], fb[TN];
#pragma unroll
            // rows 32 further down: the chunk of k-step st ^ 2
            for (int i = 0; i < TM; ++i)
                fa[i] = *reinterpret_cast<const u32x4_t *>(as + a_fo[st ^ (2 * (i & 1))] + 4096 * i);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if constexpr (BT) {
                    fb[j] = *reinterpret_cast<const u32x4_t *>(bs + bt_fo[st ^ (2 * (j & 1))] + 4096 * j);
                } else {
                    const u32x2_t lo = lds_read_tr<DT>(bs + b_fo[j] + (st * KSTEP) * B_PITCH);
                    const u32x2_t hi = lds_read_tr<DT>(bs + b_fo[j] + (st * KSTEP + TR_ROWS) * B_PITCH);
                    fb[j] = u32x4_t{lo[0], lo[1], hi[0], hi[1]};
                }
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = mfma32<DT>(fa[i], fb[j], acc[i][j]);
        }
    };

    if (nk > 0) {
        static_for<0, NS - 1>([&](auto u) { load_stage(decltype(u)::value, u); });
        for (int kt = 0; kt < nk; kt += NS) {
            static_for<0, NS>([&](auto u) {
                if (kt + decltype(u)::value < nk) iteration(kt + decltype(u)::value, u);
            });
        }
    }
    // Drain the loads past the end, by every wave, before the last-slice flag borrows a word
    // of the buffers that they write (store_tile synchronises only among later accesses).
    stage_barrier();
    store_tile<DT, BM, BN, TM, TN>(args, acc, tm, tn, slice, m0 + wrow0, n0 + wcol0, lane,
                                   *reinterpret_cast<int *>(lds[0]));
}

// ---------------------------------------------------------------------------
// Ping-pong kernel: 256 x 256 macro-tile, 8 waves, two wave groups that alternate
// between reading fragments and running MFMAs.
//
// Waves w and w + 4 share a SIMD; group 0 is waves 0-3, group 1 waves 4-7.  Every
// wave owns a 128 x 64 block of C as four quadrants, 64 rows x 32 columns each.  A
// stage (128 K-bytes) sits in LDS as four units of 16 KiB: A0, A1 (128 rows each: the
// first and second 64 rows of both wave rows) and B0, B1 (columns 0-127 and 128-255).
// A phase is one quadrant over the whole stage: read one unit's fragments, issue two
// loads, barrier, eight MFMAs, barrier:
//   phase 1: read A0, MFMA A0 x B0, load B0 two stages ahead
//   phase 2: read B1, MFMA A0 x B1, load A0 two stages ahead
//   phase 3: read A1, MFMA A1 x B0, load B1 two stages ahead
//   phase 4: read B0 of the next stage, MFMA A1 x B1, load A1 two stages ahead
// Group 1 runs one barrier behind, so between any two barriers one wave of each SIMD
// runs MFMAs from registers while the other reads and loads; neither waits for the
// other's LDS latency.
//
// Why units and quadrants: a unit is free as soon as both groups have read it, a phase
// after its own, so its successor's loads leave six phases (about 3000 clocks) before
// the wait for them with only two stages of LDS, and every load still takes whole
// 128-byte row pieces.  gemm_lds_kernel waits at the end of each stage for loads issued
// at its beginning, too late for the fifth of them that miss L2; gemm_ring_kernel leads
// as far, but in 64-byte pieces, which cost the L2 twice the lines.
//
// Order of every access to a unit: loads into it are waited for (vmcnt) by the wave
// that issued them before the barrier that ends its fragment reads of the phase before
// the unit is read, by both groups; reads of it complete (lgkmcnt) before the barrier
// that ends them; and the next loads into it are issued after both groups' barriers.
// Stages past the end of K load zeros through an empty resource, so that every phase
// issues the same two loads and the wait is a fixed count (12: six phases' loads).
//
// Measured against gemm_lds_kernel at the same tile: 8192^3 bf16 847 -> 787 us (1397
// TFLOP/s), column-major B 838 -> 787; int8 466 -> 439 us (2505 TOPS), column-major 459
// -> 438 (medians of the tracked traces; a cooler card runs them in 771 and 421).  What bounds
// it now: MFMAs, busy 85 and 77 % at the clock the power limit leaves (1.5-1.65 GHz).
// ---------------------------------------------------------------------------
template <int DT, bool BT>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void gemm_pingpong_kernel(KernelArgs args) {
    using acc_vec = typename Types<DT>::acc_vec;
    constexpr int BM = 256, BN = 256, HALF = 128, WAVES = 8;
    constexpr int E = Types<DT>::E;
    constexpr int VECE = 16 / E;
    constexpr int BK = kStageKBytes / E;
    constexpr int TM = 4, TN = 2;
    constexpr int UNIT = HALF * kStageKBytes;              // 16 KiB
    constexpr int B_PITCH = BT ? kStageKBytes : HALF * E;  // bytes per B row in LDS
    constexpr int B_CPR = B_PITCH / 16;                    // 16-byte chunks per B row
    enum { U_B0, U_A0, U_B1, U_A1 };                       // units of a stage, in load order

    __shared__ __attribute__((aligned(1024))) uint8_t lds[2][4][UNIT];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2;                             // also the wave's row of the tile
    const int wave_n = wave & 3;

    int tm, tn, slice;
    map_tile(args, tm, tn, slice);
    const int64_t M = args.M, N = args.N;
    const int64_t m0 = int64_t(tm) * BM, n0 = int64_t(tn) * BN;
    const int64_t k_begin = int64_t(slice) * args.k_chunk;
    int64_t k_end = k_begin + args.k_chunk;
    if (k_end > args.K) k_end = args.K;
    const int k_len = k_end > k_begin ? int(k_end - k_begin) : 0;
    const int ns = (k_len + BK - 1) / BK;
    const int64_t lda_b = args.lda * E, ldb_b = args.ldb * E;

    // ---- global source offsets of this lane's pieces: load i of unit h fills unit bytes
    // [(8 i + wave) KiB, + 1 KiB) ----
    const int64_t a_rows_valid = (M - m0) < BM ? (M - m0) : BM;
    const uint32_t a_bytes = uint32_t(a_rows_valid * lda_b);
    const int64_t b_rows_valid = (N - n0) < BN ? (N - n0) : BN;
    const uint32_t bt_bytes = uint32_t(b_rows_valid * ldb_b);
    uint32_t a_voff[2][2], b_voff[2][2];
    int a_chunk[2], b_chunk[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (i * WAVES + wave) * 8 + (lane >> 3);
        const int c = swz(lane & 7, row);
        a_chunk[i] = c;
        // unit row r of A_h: tile row (r / 64) * 128 + h * 64 + r % 64
#pragma unroll
        for (int h = 0; h < 2; ++h)
            a_voff[h][i] = uint32_t(((row >> 6) * 128 + h * 64 + (row & 63)) * lda_b + c * 16);
        if constexpr (BT) {
            b_chunk[i] = c;
#pragma unroll
            for (int h = 0; h < 2; ++h) b_voff[h][i] = uint32_t((h * HALF + row) * ldb_b + c * 16);
        } else {
            const int k = (i * WAVES + wave) * (1024 / B_PITCH) + lane / B_CPR;
            const int cb = (lane % B_CPR) ^ ring_bswz<DT, B_CPR>(k);
            b_chunk[i] = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h)
                b_voff[h][i] = n0 + h * HALF + cb * VECE < N ? uint32_t(k * ldb_b + h * HALF * E + cb * 16) : kOOB;
        }
    }
    const uint8_t *const a_base = static_cast<const uint8_t *>(args.A) + (m0 * args.lda + k_begin) * E;
    const uint8_t *const b_base = static_cast<const uint8_t *>(args.B) +
                                  (BT ? n0 * args.ldb + k_begin : k_begin * args.ldb + n0) * E;

    // Issues this wave's two loads of unit U of stage kt (buffer BUF).
    auto load_unit = [&](int kt, auto buf_c, auto u_c) {
        constexpr int BUF = decltype(buf_c)::value, U = decltype(u_c)::value;
        const int rem = k_len - kt * BK;
        const uint32_t dst = lds_addr(lds[BUF][U]) + uint32_t(wave) * 1024u;
        if constexpr (U == U_A0 || U == U_A1) {
            const i32x4_t r = ring_rsrc(a_base + int64_t(kt) * kStageKBytes, rem > 0 ? a_bytes : 0u);
#pragma unroll
            for (int i = 0; i < 2; ++i)
                ring_load16(r, dst + i * (WAVES * 1024), a_chunk[i] * VECE < rem ? a_voff[U == U_A1][i] : kOOB);
        } else if constexpr (BT) {
            const i32x4_t r = ring_rsrc(b_base + int64_t(kt) * kStageKBytes, rem > 0 ? bt_bytes : 0u);
#pragma unroll
            for (int i = 0; i < 2; ++i)
                ring_load16(r, dst + i * (WAVES * 1024), b_chunk[i] * VECE < rem ? b_voff[U == U_B1][i] : kOOB);
        } else {
            const int rows = rem <= 0 ? 0 : (rem < BK ? rem : BK);
            // readfirstlane: the compiler otherwise clamps the (uniform) size on the vector unit
            const i32x4_t r = ring_rsrc(b_base + int64_t(kt) * BK * ldb_b,
                                        uint32_t(__builtin_amdgcn_readfirstlane(int(rows * ldb_b))));
#pragma unroll
            for (int i = 0; i < 2; ++i) ring_load16(r, dst + i * (WAVES * 1024), b_voff[U == U_B1][i]);
        }
    };

    // ---- fragment offsets within a unit ----
    const int frag_row = lane & 31, frag_half = lane >> 5;
    const int ra0 = grp * 64 + frag_row, rb0 = wave_n * 32 + frag_row;
    int a_fo[4], bt_fo[4];                                 // k-step st of the first 32 rows
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        a_fo[st] = ra0 * kStageKBytes + 16 * swz(2 * st + frag_half, ra0);
        bt_fo[st] = rb0 * kStageKBytes + 16 * swz(2 * st + frag_half, rb0);
    }
    const int lgrp = lane >> 4, g16 = lane & 15;           // transpose reads, as in gemm_lds_kernel
    constexpr int TR_ROWS = DT == DT_BF16 ? 4 : 8;
    constexpr int KSTEP = 32 / E;
    const int tr_row = DT == DT_BF16 ? (g16 >> 2) : (g16 >> 1);
    const int tr_colb = (DT == DT_BF16 ? (g16 & 3) * 8 : (g16 & 1) * 8) + (lgrp & 1) * 16 * E;
    const int tr_khalf = (lgrp >> 1) * (KSTEP / 2);
    const int b_colb = wave_n * 32 * E + tr_colb;
    const int b_fo = (tr_khalf + tr_row) * B_PITCH +
                     (((b_colb >> 4) ^ (BT ? 0 : ring_bswz<DT, B_CPR>(tr_row))) << 4) + (b_colb & 15);

    u32x4_t fa[2][4], fb[2][4];                            // A: two 32-row tiles; B: halves 0 and 1; four k-steps
    auto read_a = [&](auto buf_c, auto u_c) {
        const uint8_t *const p = lds[decltype(buf_c)::value][decltype(u_c)::value];
#pragma unroll
        for (int st = 0; st < 4; ++st)
#pragma unroll
            // the swizzle of rows 32 further down differs by chunk ^ 4: k-step st ^ 2's chunk
            for (int i = 0; i < 2; ++i) fa[i][st] = *reinterpret_cast<const u32x4_t *>(p + a_fo[st ^ (2 * i)] + 4096 * i);
    };
    auto read_b = [&](auto buf_c, auto u_c) {
        constexpr int U = decltype(u_c)::value;
        const uint8_t *const p = lds[decltype(buf_c)::value][U];
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            if constexpr (BT) {
                fb[U == U_B1][st] = *reinterpret_cast<const u32x4_t *>(p + bt_fo[st]);
            } else {
                const u32x2_t lo = lds_read_tr<DT>(p + b_fo + (st * KSTEP) * B_PITCH);
                const u32x2_t hi = lds_read_tr<DT>(p + b_fo + (st * KSTEP + TR_ROWS) * B_PITCH);
                fb[U == U_B1][st] = u32x4_t{lo[0], lo[1], hi[0], hi[1]};
            }
        }
    };

    acc_vec acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = acc_vec{};

    // Ends a phase's reads and loads, then runs its quadrant (row half H, column half J).
    auto quadrant = [&](auto h_c, auto j_c) {
        constexpr int H = decltype(h_c)::value, J = decltype(j_c)::value;
        __builtin_amdgcn_sched_barrier(0);
        ring_barrier<12>();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int st = 0; st < 4; ++st)
#pragma unroll
            for (int i = 0; i < 2; ++i) acc[2 * H + i][J] = mfma32<DT>(fa[i][st], fb[J][st], acc[2 * H + i][J]);
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using B0 = std::integral_constant<int, U_B0>;
    using A0 = std::integral_constant<int, U_A0>;
    using B1 = std::integral_constant<int, U_B1>;
    using A1 = std::integral_constant<int, U_A1>;
    auto stage = [&](int kt, auto buf_c) {
        using NEXT = std::integral_constant<int, 1 - decltype(buf_c)::value>;
        read_a(buf_c, A0{});
        load_unit(kt + 2, buf_c, B0{});
        quadrant(I0{}, I0{});
        read_b(buf_c, B1{});
        load_unit(kt + 2, buf_c, A0{});
        quadrant(I0{}, I1{});
        read_a(buf_c, A1{});
        load_unit(kt + 2, buf_c, B1{});
        quadrant(I1{}, I0{});
        read_b(NEXT{}, B0{});
        load_unit(kt + 2, buf_c, A1{});
        quadrant(I1{}, I1{});
    };

    if (ns > 0) {
        static_for<0, 2>([&](auto s) {
            load_unit(decltype(s)::value, s, B0{});
            load_unit(decltype(s)::value, s, A0{});
            load_unit(decltype(s)::value, s, B1{});
            load_unit(decltype(s)::value, s, A1{});
        });
        ring_barrier<12>();                                // B0 and A0 of stage 0 have landed
        read_b(I0{}, B0{});
        phase_barrier();                                   // ... and B0 is read, before phase 1 refills it
        if (grp == 1) asm volatile("s_barrier" ::: "memory");
        int kt = 0;
        for (; kt + 1 < ns; kt += 2) {
            stage(kt, I0{});
            stage(kt + 1, I1{});
        }
        if (kt < ns) stage(kt, I0{});
        if (grp == 0) asm volatile("s_barrier" ::: "memory");
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // drain the loads past the end before exit

    __shared__ int s_last;
    store_tile<DT, BM, BN, TM, TN, HALF>(args, acc, tm, tn, slice, m0 + grp * 128, n0 + wave_n * 32, lane, s_last);
}

}  // namespace gemm
