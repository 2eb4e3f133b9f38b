// kern_tile.h -- register-staged tile kernels: GENERIC (any alignment: 16-byte
// loads at any address, or element by element for the shortest rows) and MACRO /
// SKINNY (16-byte buffer loads, B transposed in registers).
#pragma once

#include "gemm_common.h"
#include "pieces.h"

namespace gemm {

// Element-wise kernel: every element is loaded and masked by itself.  Only for rows
// shorter than one 16-byte piece (K or N of a few elements) and strides past 4 MiB,
// which gemm_tile_kernel does not take.
template <int DT, int BM, int BN, int WM, int WN, int WAVES_PER_EU, bool BT>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * WM * WN, 64 * WM * WN),
                          amdgpu_waves_per_eu(WAVES_PER_EU, WAVES_PER_EU)))
void gemm_element_kernel(KernelArgs args) {
    using T = TileKernel<DT, BM, BN, WM, WN, false>;
    using acc_vec = typename Types<DT>::acc_vec;
    constexpr int E = T::E, BK = T::BK, VECE = T::VECE;
    constexpr int TM = T::TM, TN = T::TN;

    __shared__ __attribute__((aligned(16))) uint8_t smem[2 * (BM + BN) * kStageKBytes];
    uint8_t *const a_lds = smem;                               // [2][BM][128]
    uint8_t *const b_lds = smem + 2 * BM * kStageKBytes;       // [2][BN][128]

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
    const int64_t nk = k_end > k_begin ? (k_end - k_begin + BK - 1) / BK : 0;

    const uint8_t *const A = static_cast<const uint8_t *>(args.A);
    const uint8_t *const B = static_cast<const uint8_t *>(args.B);
    const int64_t lda = args.lda, ldb = args.ldb;

    u32x4_t ra[T::A_CHUNKS], rb[T::B_CHUNKS];

    auto load_stage = [&](int64_t kt) {
        const int64_t k0 = k_begin + kt * BK;
#pragma unroll
        for (int i = 0; i < T::A_CHUNKS; ++i) {
            const int q = i * T::THREADS + tid;
            const int row = q >> 3, c = q & 7;
            const int64_t gm = m0 + row, gk = k0 + int64_t(c) * VECE;
            unsigned w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < VECE; ++e) {
                unsigned x = 0;
                if (gm < M && gk + e < k_end) {
                    if (E == 1) x = A[gm * lda + gk + e];
                    else x = reinterpret_cast<const uint16_t *>(A)[gm * lda + gk + e];
                }
                w[(e * E) >> 2] |= x << (8 * ((e * E) & 3));
            }
            ra[i] = u32x4_t{w[0], w[1], w[2], w[3]};
        }
#pragma unroll
        for (int i = 0; i < T::B_CHUNKS; ++i) {
            // Row-major B: neighbouring threads take neighbouring columns.  Column-major
            // B (stored N x K): neighbouring threads take neighbouring K chunks of a column.
            const int q = i * T::THREADS + tid;
            const int n = BT ? q >> 3 : q % BN, c = BT ? q & 7 : q / BN;
            const int64_t gn = n0 + n, gk = k0 + int64_t(c) * VECE;
            unsigned w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < VECE; ++e) {
                unsigned x = 0;
                if (gn < N && gk + e < k_end) {
                    const int64_t idx = BT ? gn * ldb + gk + e : (gk + e) * ldb + gn;
                    if (E == 1) x = B[idx];
                    else x = reinterpret_cast<const uint16_t *>(B)[idx];
                }
                w[(e * E) >> 2] |= x << (8 * ((e * E) & 3));
            }
            rb[i] = u32x4_t{w[0], w[1], w[2], w[3]};
        }
    };

    auto store_stage = [&](int buf) {
        uint8_t *const as = a_lds + buf * BM * kStageKBytes;
        uint8_t *const bs = b_lds + buf * BN * kStageKBytes;
#pragma unroll
        for (int i = 0; i < T::A_CHUNKS; ++i) {
            const int q = i * T::THREADS + tid;
            const int row = q >> 3, c = q & 7;
            *reinterpret_cast<u32x4_t *>(as + row * kStageKBytes + swz(c, row) * 16) = ra[i];
        }
#pragma unroll
        for (int i = 0; i < T::B_CHUNKS; ++i) {
            const int q = i * T::THREADS + tid;
            const int n = BT ? q >> 3 : q % BN, c = BT ? q & 7 : q / BN;
            *reinterpret_cast<u32x4_t *>(bs + n * kStageKBytes + swz(c, n) * 16) = rb[i];
        }
    };

    acc_vec acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = acc_vec{};

    const int frag_row = lane & 31;
    const int frag_half = lane >> 5;
    const int wrow0 = wave_m * (BM / WM);
    const int wcol0 = wave_n * (BN / WN);

    if (nk > 0) {
        load_stage(0);
        store_stage(0);
        __syncthreads();
    }
    for (int64_t kt = 0; kt < nk; ++kt) {
        const int buf = int(kt & 1);
        if (kt + 1 < nk) load_stage(kt + 1);
        const uint8_t *const as = a_lds + buf * BM * kStageKBytes;
        const uint8_t *const bs = b_lds + buf * BN * kStageKBytes;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int chunk = 2 * s + frag_half;
            u32x4_t af[TM], bfr[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = wrow0 + i * 32 + frag_row;
                af[i] = *reinterpret_cast<const u32x4_t *>(as + row * kStageKBytes + swz(chunk, row) * 16);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = wcol0 + j * 32 + frag_row;
                bfr[j] = *reinterpret_cast<const u32x4_t *>(bs + col * kStageKBytes + swz(chunk, col) * 16);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = mfma32<DT>(af[i], bfr[j], acc[i][j]);
        }
        if (kt + 1 < nk) store_stage(buf ^ 1);
        __syncthreads();
    }

    // ---------------- epilogue ----------------
    __shared__ int s_last;
    store_tile<DT, BM, BN, TM, TN>(args, acc, tm, tn, slice, m0 + wrow0, n0 + wcol0, lane, s_last);
}

// ---------------------------------------------------------------------------
// Tile kernel for operands at any address (GENERIC): the data path of
// gemm_lds_kernel, its direct-to-LDS loads (which need 16-byte aligned rows)
// replaced by 16-byte loads at whatever address a row starts at, staged through
// registers and written to LDS in gemm_lds_kernel's layouts (swizzled 16-byte
// chunks; row-major B untransposed, read back with the transpose reads).  The
// memory system takes a misaligned 16-byte load at the cost of the extra line it
// touches, so a stage needs one load instruction per KiB instead of the one per 64
// elements of an element-wise loader, which bound this family before.
//
// What keeps every access inside the operands: rows of A (and of a column-major B)
// past M (N) repeat the last row, and their results are not stored.  A row-major B
// piece that starts left of column N may run past the row's end into the row below,
// which exists for every row but the last; only columns past N see those bytes.  The
// stage that reaches the end of K (the only one whose pieces may run past K, or past
// the last row) takes its pieces through load_tail: read ending at the row's end and
// shifted down, zero from K on.  It needs rows of at least 16 bytes (wide_rows_ok).
//
// A stage's loads are issued AHEAD stages and a half before it is read: one set of
// staging registers for the small tiles, of which several share a CU, two for the
// large ones.
//
// Measured against element-wise loads: bf16 256 x 32003 x 4096, row-major B, 1397 -> 86 us
// (94 with one stage in flight; int8 6314 x 932 x 2271 41 -> 35 us by the second);
// bf16 2047 x 2051 x 2049, column-major B, 350 -> 47 us; int8 50176 x 64 x 147 28.1 -> 6.7 us
// (kernel time; 8.5 with the host's launch).  The load path bounds it: each misaligned
// 128-byte row piece touches two lines, and a 256 x 128 tile's stage takes about 2900 clocks
// beside 1024 of MFMAs (counters of the first call: address units busy 63 % of the time,
// matrix cores 35 %).  A 256 x 256 tile over eight waves goes to scratch.
// ---------------------------------------------------------------------------
typedef unsigned u32x4_any_t __attribute__((ext_vector_type(4), aligned(1)));

__device__ __forceinline__ u32x4_t load_any16(const uint8_t *base, uint32_t off) {
    return *reinterpret_cast<const u32x4_any_t *>(base + off);
}

// v shifted down by s bytes, zeros from the top (s >= 16: all zeros).
__device__ __forceinline__ u32x4_t shift_down(u32x4_t v, int s) {
    uint64_t lo = uint64_t(v[0]) | (uint64_t(v[1]) << 32), hi = uint64_t(v[2]) | (uint64_t(v[3]) << 32);
    if (s >= 8) { lo = hi; hi = 0; s -= 8; }
    if (s >= 8) { lo = 0; s = 0; }
    if (s > 0) {
        lo = (lo >> (8 * s)) | (hi << (64 - 8 * s));
        hi >>= 8 * s;
    }
    return u32x4_t{uint32_t(lo), uint32_t(lo >> 32), uint32_t(hi), uint32_t(hi >> 32)};
}

template <int DT, int BM, int BN, int WM, int WN, bool BT, int WAVES_PER_EU, int AHEAD>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * WM * WN, 64 * WM * WN),
                          amdgpu_waves_per_eu(WAVES_PER_EU, WAVES_PER_EU)))
void gemm_tile_kernel(KernelArgs args) {
    static_assert(AHEAD == 1 || AHEAD == 2, "register stages in flight");
    using acc_vec = typename Types<DT>::acc_vec;
    constexpr int E = Types<DT>::E;
    constexpr int VECE = 16 / E;
    constexpr int BK = kStageKBytes / E;                  // K elements per stage
    constexpr int THREADS = 64 * WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int A_STAGE = BM * kStageKBytes, B_STAGE = BN * kStageKBytes;   // bytes
    constexpr int A_CH = A_STAGE / 16 / THREADS, B_CH = B_STAGE / 16 / THREADS;   // 16-byte pieces per thread
    constexpr int A_STEP = THREADS / 8;                   // rows between a thread's A pieces
    constexpr int B_PITCH = BT ? kStageKBytes : BN * E;   // bytes per B row in LDS
    constexpr int B_CPR = B_PITCH / 16;                   // pieces per B row
    constexpr int B_STEP = THREADS / B_CPR;               // rows between a thread's B pieces
    static_assert(A_CH >= 1 && A_CH * THREADS * 16 == A_STAGE, "A stage split");
    static_assert(B_CH >= 1 && B_CH * THREADS * 16 == B_STAGE, "B stage split");
    static_assert(B_STEP >= 1 && B_STEP * B_CPR == THREADS, "B rows per pass");

    __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * (A_STAGE + B_STAGE)];

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

    // ---- this thread's pieces: piece i of A is row a_row + i * A_STEP, chunk a_c ----
    const int a_c = tid & 7, a_row = tid >> 3;
    const int a_last = int(M - m0 < BM ? M - m0 : BM) - 1;         // last valid row of the tile
    uint32_t a_voff[A_CH];
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
        a_voff[i] = uint32_t(row_piece(a_row + i * A_STEP, a_last, lda_b, a_c));
    }
    // B: column-major as A over the tile's rows (n); row-major: row b_row + i * B_STEP (k),
    // columns from b_col (pieces wholly past N take the row's last column on).
    const int b_c = BT ? (tid & 7) : tid % B_CPR, b_row = BT ? (tid >> 3) : tid / B_CPR;
    const int b_last = int(N - n0 < BN ? N - n0 : BN) - 1;
    const int64_t b_col = n0 + int64_t(b_c) * VECE;
    uint32_t b_voff[B_CH];
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
        const int row = b_row + i * B_STEP;
        b_voff[i] = BT ? uint32_t(row_piece(row, b_last, ldb_b, b_c))
                       : uint32_t(row * ldb_b) + uint32_t(col_piece(b_col, N) * E);
    }
    const uint8_t *const a_base = static_cast<const uint8_t *>(args.A) + (m0 * args.lda + k_begin) * E;
    const uint8_t *const b_base =
        static_cast<const uint8_t *>(args.B) + (BT ? n0 * args.ldb + k_begin : k_begin * args.ldb) * E;

    u32x4_t ra_[AHEAD][A_CH], rb_[AHEAD][B_CH];
    // Stage kt into register set SET: any stage but the one with the end of K ...
    auto load_full = [&](int kt, auto set_c) {
        u32x4_t(&ra)[A_CH] = ra_[decltype(set_c)::value];
        u32x4_t(&rb)[B_CH] = rb_[decltype(set_c)::value];
        const uint8_t *const ap = a_base + int64_t(kt) * kStageKBytes;
        const uint8_t *const bp = b_base + (BT ? int64_t(kt) * kStageKBytes : int64_t(kt) * BK * ldb_b);
#pragma unroll
        for (int i = 0; i < A_CH; ++i) ra[i] = load_any16(ap, a_voff[i]);
#pragma unroll
        for (int i = 0; i < B_CH; ++i) rb[i] = load_any16(bp, b_voff[i]);
    };
    // ... and any stage at all.
    auto load_stage = [&](int kt, auto set_c) {
        u32x4_t(&ra)[A_CH] = ra_[decltype(set_c)::value];
        u32x4_t(&rb)[B_CH] = rb_[decltype(set_c)::value];
        const uint8_t *const ap = a_base + int64_t(kt) * kStageKBytes;
        const uint8_t *const bp = b_base + (BT ? int64_t(kt) * kStageKBytes : int64_t(kt) * BK * ldb_b);
        if (kt + 1 < nk || k_end < args.K) {
            load_full(kt, set_c);
        } else {
            const int rem = int(k_end - k_begin - int64_t(kt) * BK);          // 1 .. BK
            // K-contiguous rows: bytes past the row's end (offset from this stage's start)
            auto back = [&](int c) { return row_piece_back(c, rem * E); };
#pragma unroll
            for (int i = 0; i < A_CH; ++i)
                ra[i] = shift_down(*reinterpret_cast<const u32x4_any_t *>(ap + int64_t(a_voff[i]) - back(a_c)), back(a_c));
#pragma unroll
            for (int i = 0; i < B_CH; ++i) {
                if constexpr (BT) {
                    rb[i] = shift_down(*reinterpret_cast<const u32x4_any_t *>(bp + int64_t(b_voff[i]) - back(b_c)),
                                       back(b_c));
                } else {
                    const int row = b_row + i * B_STEP;
                    const int64_t col = col_piece_tail(b_col, N, VECE);
                    const u32x4_t v = shift_down(
                        load_any16(bp + row_tail(row, rem) * ldb_b, uint32_t(col * E)), int(b_col - col) * E);
                    rb[i] = row < rem ? v : u32x4_t{0u, 0u, 0u, 0u};
                }
            }
        }
    };
    const int a_wr = a_row * kStageKBytes;
    auto store_stage = [&](auto buf_c, auto set_c) {
        constexpr int BUF = decltype(buf_c)::value;
        const u32x4_t(&ra)[A_CH] = ra_[decltype(set_c)::value];
        const u32x4_t(&rb)[B_CH] = rb_[decltype(set_c)::value];
        uint8_t *const as = smem + BUF * (A_STAGE + B_STAGE);
        uint8_t *const bs = as + A_STAGE;
#pragma unroll
        for (int i = 0; i < A_CH; ++i)
            *reinterpret_cast<u32x4_t *>(as + a_wr + i * A_STEP * kStageKBytes + swz(a_c, a_row + i * A_STEP) * 16) = ra[i];
#pragma unroll
        for (int i = 0; i < B_CH; ++i) {
            const int row = b_row + i * B_STEP;
            const int chunk = BT ? swz(b_c, row) : (b_c ^ ring_bswz<DT, B_CPR>(row));
            *reinterpret_cast<u32x4_t *>(bs + row * B_PITCH + chunk * 16) = rb[i];
        }
    };

    // ---- fragment offsets, as in gemm_lds_kernel ----
    const int frag_row = lane & 31, frag_half = lane >> 5;
    const int wrow0 = wave_m * (BM / WM), wcol0 = wave_n * (BN / WN);
    const int r0 = wrow0 + frag_row, f0 = (r0 ^ (r0 >> 3)) & 7;
    const int rb0 = wcol0 + frag_row, fb0 = (rb0 ^ (rb0 >> 3)) & 7;
    int a_fo[2][4], bt_fo[2][4];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            a_fo[p][st] = r0 * kStageKBytes + 16 * ((2 * st + frag_half) ^ f0 ^ (4 * p));
            bt_fo[p][st] = rb0 * kStageKBytes + 16 * ((2 * st + frag_half) ^ fb0 ^ (4 * p));
        }
    const int grp = lane >> 4, g16 = lane & 15;
    constexpr int TR_ROWS = DT == DT_BF16 ? 4 : 8;        // rows per transpose read
    constexpr int KSTEP = 32 / E;                         // K elements per MFMA
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

    u32x4_t fa[2][TM], fb[2][TN];
    auto load_frags = [&](auto buf_c, auto s_c, auto slot_c) {
        constexpr int BUF = decltype(buf_c)::value, S = decltype(s_c)::value, SLOT = decltype(slot_c)::value;
        const uint8_t *const as = smem + BUF * (A_STAGE + B_STAGE);
        const uint8_t *const bs = as + A_STAGE;
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
    for (int i = 0; i < TM; ++i) {
        fa[1][i] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = acc_vec{};
    }
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

    // One stage (LDS buffer BUF holds stage kt, visible; the registers hold stage kt + 1, and
    // kt + 2 if two sets are in flight: stage s in set s % AHEAD).
    // Slot 1 carries the last k-step's fragments over the barrier, as in gemm_lds_kernel.
    // The other buffer is free from the barrier that ended stage kt - 1 on.
    // STEADY: stage kt + 1 + AHEAD is a full one, loaded without a branch, so that the waits
    // before the LDS writes can leave the younger set in flight.
    auto stage = [&](int kt, auto buf_c, auto steady_c) {
        constexpr bool STEADY = decltype(steady_c)::value;
        using OTHER = std::integral_constant<int, 1 - decltype(buf_c)::value>;
        using SET = std::integral_constant<int, OTHER::value % AHEAD>;
        load_frags(buf_c, I0{}, I0{});
        mfma_slot(I1{});
        __builtin_amdgcn_sched_barrier(0);
        load_frags(buf_c, I1{}, I1{});
        mfma_slot(I0{});
        __builtin_amdgcn_sched_barrier(0);
        if (STEADY || kt + 1 < nk) store_stage(OTHER{}, SET{});
        if constexpr (STEADY) load_full(kt + 1 + AHEAD, SET{});
        else if (kt + 1 + AHEAD < nk) load_stage(kt + 1 + AHEAD, SET{});
        __builtin_amdgcn_sched_barrier(0);
        load_frags(buf_c, I2{}, I0{});
        mfma_slot(I1{});
        __builtin_amdgcn_sched_barrier(0);
        load_frags(buf_c, I3{}, I1{});
        mfma_slot(I0{});
        phase_barrier();
    };

    if (nk > 0) {
        load_stage(0, I0{});
        if constexpr (AHEAD == 2)
            if (nk > 1) load_stage(1, I1{});
        store_stage(I0{}, I0{});
        if (nk > AHEAD) load_stage(AHEAD, I0{});
        phase_barrier();
        int kt = 0;
        for (; kt + 2 + AHEAD < nk - 1; kt += 2) {
            stage(kt, I0{}, std::true_type{});
            stage(kt + 1, I1{}, std::true_type{});
        }
        for (; kt + 1 < nk; kt += 2) {
            stage(kt, I0{}, std::false_type{});
            stage(kt + 1, I1{}, std::false_type{});
        }
        if (kt < nk) stage(kt, I0{}, std::false_type{});
        mfma_slot(I1{});
    }

    // Every wave is past its last fragment read (the last stage's barrier), so the
    // last-slice flag borrows a word of the operand buffers.
    store_tile<DT, BM, BN, TM, TN>(args, acc, tm, tn, slice, m0 + wrow0, n0 + wcol0, lane,
                                   *reinterpret_cast<int *>(smem));
}

// ---------------------------------------------------------------------------
// Vectorised kernel: 16-byte (A, bf16 B) and 8-byte (int8 B) buffer loads.
//
// Every global load goes through a buffer resource.  A load whose offset is
// at or past the resource's size returns zero without touching memory, which
// replaces all bounds branches: rows past M and columns past N get an offset
// that is out of range by construction, the K tail of A is masked per chunk,
// and the K tail of B (and every stage past the end of the slice) is masked
// by shrinking the resource's size to the valid rows of the stage.  The loop
// body is therefore branch-free, so loads, LDS traffic and MFMAs of one stage
// live in one scheduling region.
// ---------------------------------------------------------------------------

template <int DT, int BM, int BN, int WM, int WN, int WAVES_PER_EU>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * WM * WN, 64 * WM * WN),
                          amdgpu_waves_per_eu(WAVES_PER_EU, WAVES_PER_EU)))
void gemm_vec_kernel(KernelArgs args) {
    using T = TileKernel<DT, BM, BN, WM, WN, true>;
    using acc_vec = typename Types<DT>::acc_vec;
    using out_t = typename Types<DT>::out_t;
    constexpr int E = T::E, BK = T::BK, VECE = T::VECE;
    constexpr int TM = T::TM, TN = T::TN;
    constexpr int THREADS = T::THREADS;
    constexpr int KPB = T::KPB, OUTB = T::OUTB, B_BLOCKS = T::B_BLOCKS;
    constexpr int A_CHUNKS = T::A_CHUNKS;

    __shared__ __attribute__((aligned(16))) uint8_t smem[2 * (BM + BN) * kStageKBytes];
    uint8_t *const a_lds = smem;
    uint8_t *const b_lds = smem + 2 * BM * kStageKBytes;

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
    const int64_t lda_b = args.lda * E, ldb_b = args.ldb * E;   // row strides in bytes

    // ---- per-thread global offsets (constant over the K loop) ----
    // A: chunk i of this thread is row (i * THREADS + tid) / 8, logical chunk tid % 8.
    // The per-chunk row step is uniform; rows at or past M are masked by the
    // resource size (rows are contiguous with stride lda from the tile's first row).
    const int a_c = tid & 7;
    const uint32_t a_voff0 = uint32_t((tid >> 3) * lda_b + a_c * 16);
    constexpr int A_ROW_STEP = THREADS / 8;
    const int64_t a_rows_valid = (M - m0) < BM ? (M - m0) : BM;
    const uint32_t a_bytes = uint32_t(a_rows_valid * lda_b);
    // B: block bI of this thread covers k-rows kb*KPB .. +KPB and 8 columns from nb*8.
    // Row r of the block is the uniform offset r * ldb_b.  Columns at or past N get an
    // out-of-range base; K rows past the slice end are masked by the resource size
    // (whole blocks, since the slice length is a multiple of KPB).
    uint32_t b_voff[B_BLOCKS];
#pragma unroll
    for (int bI = 0; bI < B_BLOCKS; ++bI) {
        const int b = bI * THREADS + tid;
        const int nb = b % (BN / 8), kb = b / (BN / 8);
        b_voff[bI] = (n0 + nb * 8 < N) ? uint32_t(kb * KPB * ldb_b + nb * 8 * E) : kOOB;
    }
    const uint8_t *const a_base = static_cast<const uint8_t *>(args.A) + (m0 * args.lda + k_begin) * E;
    const uint8_t *const b_base = static_cast<const uint8_t *>(args.B) + (k_begin * args.ldb + n0) * E;

    // One stage of staged global data.
    struct Stage {
        u32x4_t a[A_CHUNKS];
        u32x4_t b4[DT == DT_BF16 ? B_BLOCKS * KPB : 1];
        u32x2_t b2[DT == DT_I8 ? B_BLOCKS * KPB : 1];
    };

    // Loads stage kt into st (kt may be past the last stage: every load then returns 0).
    auto load_stage = [&](Stage &st, int kt) {
        const int64_t rem = (k_end - k_begin) - int64_t(kt) * BK;   // valid K elements left
        const __amdgpu_buffer_rsrc_t ra_rsrc = make_rsrc(a_base + int64_t(kt) * kStageKBytes, a_bytes);
        const uint32_t a0 = int64_t(a_c) * VECE < rem ? a_voff0 : kOOB;
#pragma unroll
        for (int i = 0; i < A_CHUNKS; ++i)
            st.a[i] = __builtin_amdgcn_raw_buffer_load_b128(ra_rsrc, a0 + uint32_t(i * A_ROW_STEP * lda_b), 0, 0);
        const int64_t rows = rem <= 0 ? 0 : (rem < BK ? rem : BK);
        const __amdgpu_buffer_rsrc_t rb_rsrc =
            make_rsrc(b_base + int64_t(kt) * BK * ldb_b, uint32_t(rows * ldb_b));
#pragma unroll
        for (int bI = 0; bI < B_BLOCKS; ++bI)
#pragma unroll
            for (int r = 0; r < KPB; ++r) {
                const int soff = int(r * ldb_b);
                if (DT == DT_BF16)
                    st.b4[bI * KPB + r] = __builtin_amdgcn_raw_buffer_load_b128(rb_rsrc, b_voff[bI], soff, 0);
                else
                    st.b2[bI * KPB + r] = __builtin_amdgcn_raw_buffer_load_b64(rb_rsrc, b_voff[bI], soff, 0);
            }
    };

    auto store_stage = [&](const Stage &st, int buf) {
        uint8_t *const as = a_lds + buf * BM * kStageKBytes;
        uint8_t *const bs = b_lds + buf * BN * kStageKBytes;
#pragma unroll
        for (int i = 0; i < A_CHUNKS; ++i) {
            const int row = (i * THREADS + tid) >> 3;
            *reinterpret_cast<u32x4_t *>(as + row * kStageKBytes + swz(a_c, row) * 16) = st.a[i];
        }
#pragma unroll
        for (int bI = 0; bI < B_BLOCKS; ++bI) {
            const int b = bI * THREADS + tid;
            const int nb = b % (BN / 8), kb = b / (BN / 8);
            const int byte = kb * OUTB;
            const int chunk = byte >> 4, half = (byte >> 3) & 1;
            const int base = bI * KPB;
            constexpr int DW = OUTB / 4;                 // dwords per column piece
            unsigned col[8][DW];
            if (DT == DT_BF16) bf16_transpose<KPB>(st.b4, base, *reinterpret_cast<unsigned(*)[8][KPB / 2]>(&col));
            else i8_transpose<KPB>(st.b2, base, *reinterpret_cast<unsigned(*)[8][KPB / 4]>(&col));
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int n = nb * 8 + c;
                uint8_t *dst = bs + n * kStageKBytes + swz(chunk, n) * 16 + half * 8;
                if (DW == 4)
                    *reinterpret_cast<u32x4_t *>(dst) = u32x4_t{col[c][0], col[c][DW > 1 ? 1 : 0],
                                                                col[c][DW > 2 ? 2 : 0], col[c][DW > 3 ? 3 : 0]};
                else
                    *reinterpret_cast<u32x2_t *>(dst) = u32x2_t{col[c][0], col[c][DW > 1 ? 1 : 0]};
            }
        }
    };

    const int frag_row = lane & 31;
    const int frag_half = lane >> 5;
    const int wrow0 = wave_m * (BM / WM);
    const int wcol0 = wave_n * (BN / WN);
    u32x4_t fa[2][TM], fb[2][TN];
    auto load_frags = [&](int buf, int s, int slot) {
        const uint8_t *const as = a_lds + buf * BM * kStageKBytes;
        const uint8_t *const bs = b_lds + buf * BN * kStageKBytes;
        const int chunk = 2 * s + frag_half;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int row = wrow0 + i * 32 + frag_row;
            fa[slot][i] = *reinterpret_cast<const u32x4_t *>(as + row * kStageKBytes + swz(chunk, row) * 16);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = wcol0 + j * 32 + frag_row;
            fb[slot][j] = *reinterpret_cast<const u32x4_t *>(bs + col * kStageKBytes + swz(chunk, col) * 16);
        }
    };

    acc_vec acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = acc_vec{};

    // MFMAs over the stage in LDS buffer `buf`; fragments of k-step s+1 are read
    // while the MFMAs of k-step s run.  Expects k-step 0's fragments in slot 0.
    auto compute = [&](int buf) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s < 3) load_frags(buf, s + 1, (s + 1) & 1);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = mfma32<DT>(fa[s & 1][i], fb[s & 1][j], acc[i][j]);
        }
    };

    // Software pipeline, two stages of global loads in flight:
    //   loop top (kt even): LDS[0] = stage kt, s1 = stage kt+1, s0 = stage kt+2 (in flight).
    Stage s0, s1;
    if (nk > 0) {
        load_stage(s0, 0);
        load_stage(s1, 1);
        store_stage(s0, 0);
        __syncthreads();
        load_stage(s0, 2);
        load_frags(0, 0, 0);
    }
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
        compute(0);
        store_stage(s1, 1);
        __syncthreads();
        load_stage(s1, kt + 3);
        load_frags(1, 0, 0);
        compute(1);
        store_stage(s0, 0);
        __syncthreads();
        load_stage(s0, kt + 4);
        load_frags(0, 0, 0);
    }
    if (kt < nk) compute(0);

    // Every wave is past its last fragment read when store_tile first synchronises, so
    // the last-slice flag borrows a word of the operand buffers (a separate __shared__
    // word would take the 64 x 256 tile past half of the CU's LDS).
    store_tile<DT, BM, BN, TM, TN>(args, acc, tm, tn, slice, m0 + wrow0, n0 + wcol0, lane,
                                   *reinterpret_cast<int *>(smem));
}

}  // namespace gemm
