// Every 16-byte read of gemm_tile_kernel, by the offsets that it computes (pieces.h), over small
// products of every any-alignment configuration: prints the first read that leaves its operand
// and exits 1, or prints how many reads it looked at.
#include <stdio.h>

#include "../paper_2512_13282_amd/csrc/configs.h"
#include "../paper_2512_13282_amd/csrc/pieces.h"

using namespace gemm;

static int64_t g_reads = 0;
static bool g_in_place = false;   // with an argument: the last stage read in place, to see the walk fail
static bool inside(const char *what, int cfg, int dt, int bt, int64_t M, int64_t N, int64_t K, int64_t ld, int64_t off,
                   int64_t span) {
    ++g_reads;
    if (off >= 0 && off + 16 <= span) return true;
    printf("%s: config %d dtype %d b_trans %d M %lld N %lld K %lld ld %lld reads [%lld, +16) of %lld bytes\n", what, cfg,
           dt, bt, (long long)M, (long long)N, (long long)K, (long long)ld, (long long)off, (long long)span);
    return false;
}

// The reads of one K-contiguous operand (rows x K, a tile of `tile` rows from row r0).
static bool rows_ok(const char *what, int cfg, int dt, int bt, int64_t M, int64_t N, int64_t K, int64_t rows, int64_t ld,
                    int64_t r0, int tile, int64_t k_begin, int64_t k_end) {
    const int e = dt == DT_I8 ? 1 : 2, bk = kStageKBytes / e;
    const int64_t span = ((rows - 1) * ld + K) * e;
    const int last = int(rows - r0 < tile ? rows - r0 : tile) - 1;
    const int nk = int((k_end - k_begin + bk - 1) / bk);
    for (int kt = 0; kt < nk; ++kt) {
        const bool full = kt + 1 < nk || k_end < K;
        const int rem = int(k_end - k_begin - int64_t(kt) * bk);
        const int64_t base = (r0 * ld + k_begin) * e + int64_t(kt) * kStageKBytes;
        for (int row = 0; row < tile; ++row)
            for (int c = 0; c < 8; ++c) {
                const int64_t off = base + row_piece(row, last, ld * e, c) - (full || g_in_place ? 0 : row_piece_back(c, rem * e));
                if (!inside(what, cfg, dt, bt, M, N, K, ld, off, span)) return false;
            }
    }
    return true;
}

static bool cols_ok(int cfg, int dt, int64_t M, int64_t N, int64_t K, int64_t ld, int64_t n0, int tile, int64_t k_begin,
                    int64_t k_end) {
    const int e = dt == DT_I8 ? 1 : 2, bk = kStageKBytes / e, vece = 16 / e;
    const int64_t span = ((K - 1) * ld + N) * e;
    const int nk = int((k_end - k_begin + bk - 1) / bk);
    for (int kt = 0; kt < nk; ++kt) {
        const bool full = kt + 1 < nk || k_end < K;
        const int rem = int(k_end - k_begin - int64_t(kt) * bk);
        const int64_t base = (k_begin + int64_t(kt) * bk) * ld * e;
        for (int row = 0; row < bk; ++row)
            for (int c = 0; c < tile * e / 16; ++c) {
                const int64_t col = n0 + int64_t(c) * vece;
                const int64_t off = full ? base + row * ld * e + col_piece(col, N) * e
                                         : base + row_tail(row, rem) * ld * e + col_piece_tail(col, N, vece) * e;
                if (!inside("row-major B", cfg, dt, 0, M, N, K, ld, off, span)) return false;
            }
    }
    return true;
}

int main(int argc, char **) {
    g_in_place = argc > 1;
    for (int cfg = 0; cfg < kNumConfigs; ++cfg) {
        const TileConfig &c = kConfigs[cfg];
        if (c.family != FAM_GENERIC) continue;
        for (int dt = 0; dt < 2; ++dt) {
            const int e = dt == DT_I8 ? 1 : 2, bk = kStageKBytes / e;
            const int64_t edge = 16 / e;                     // the shortest row
            const int64_t Ks[] = {edge, edge + 1, bk - 1, bk, bk + 1, bk + edge - 1, 2 * bk, 2 * bk + 3, 3 * bk - 1};
            const int64_t Ms[] = {1, 2, c.bm - 1, c.bm, c.bm + 1};
            const int64_t Ns[] = {1, edge, edge + 1, c.bn - 1, c.bn, c.bn + 1, c.bn + edge - 1};
            for (int64_t K : Ks)
                for (int64_t N : Ns)
                    for (int64_t M : Ms)
                        for (int bt = 0; bt < 2; ++bt)
                            for (int64_t pad = 0; pad < 6; pad = 2 * pad + 1) {
                                const int64_t lda = K + pad, ldb = (bt ? K : N) + pad;
                                if (!wide_rows_ok(dt, bt, N, K, lda, ldb)) continue;
                                for (int64_t chunk = bk; chunk < K + bk; chunk += bk)     // every split
                                    for (int64_t k0 = 0; k0 < K; k0 += chunk) {
                                        const int64_t k1 = k0 + chunk < K ? k0 + chunk : K;
                                        for (int64_t m0 = 0; m0 < M; m0 += c.bm)
                                            if (!rows_ok("A", cfg, dt, bt, M, N, K, M, lda, m0, c.bm, k0, k1)) return 1;
                                        for (int64_t n0 = 0; n0 < N; n0 += c.bn)
                                            if (!(bt ? rows_ok("column-major B", cfg, dt, bt, M, N, K, N, ldb, n0, c.bn, k0, k1)
                                                     : cols_ok(cfg, dt, M, N, K, ldb, n0, c.bn, k0, k1)))
                                                return 1;
                                    }
                            }
        }
    }
    printf("%lld reads\n", (long long)g_reads);
    return 0;
}
