// Calls of the rows kernels (w4_tile.hip, w4_slices.hip): how far K may be split, and the one plan that the workspace queries, the
// forwards and dmr_qlinear_kernel_path share.  Pure host arithmetic for 256 CUs.
#pragma once
#include "mid_plan.hpp"
#include "rows_plan.hpp"

namespace dmr {

// Splits of K for 17..64 rows of a layer whose K divides into chunks of four groups; 0: those of plan_mid.  K is split until every CU
// has 128 columns while a split keeps two chunks; two splits of more than seven chunks give way to plan_mid's two or four times
// as many while those fit the fixed scratch of dmr_qlinear_forward_static.
inline int panel_splits(int64_t M, int64_t K, int64_t N) {
    constexpr int kChunk = 4;      // groups
    const int64_t groups = K / kGroup;
    if (groups % kChunk != 0) return 0;
    const int nch = (int)(groups / kChunk);
    int sk = (int)(kCus / ((N + kTileCols - 1) / kTileCols));
    sk = sk < 1 ? 1 : sk > nch ? nch : sk;
    const int cps = (nch + sk - 1) / sk;
    sk = (nch + cps - 1) / cps;
    if (sk == 1 || cps < 2) return 0;
    const MidPlan m = plan_mid(M, K, N);
    if (m.R == 1 && m.wgs <= kCus && m.gps % 4 == 0) return 0;
    return sk == 2 && cps > 7 && (size_t)m.SK * (size_t)(M * N) * sizeof(float) <= DMR_STATIC_SCRATCH_BYTES ? 0 : sk;
}

// What a call may split K into at most, and so what it may ask for: partials of 64 rows fit the fixed scratch but for layers that also
// run without.  Layers of 16384 .. 32768 outputs stay whole at 17..64 rows: 64 columns to a workgroup fill the CUs (14336 -> 16384,
// 17 / 32 rows 30.6 / 32.1 us whole, 35.6 / 34.1 in two; 11008 -> 16384, 17 rows 24.9 / 27.6); above, K is split where it is no
// multiple of 512 (7936 -> 33216, 49 rows 79.3 whole, 71.8 in two).
inline int row_splits(int64_t M, int64_t K, int64_t N) {
    const int64_t tiles = N / kTileRows;
    if (M <= 64 && tiles >= 1024) return tiles <= 2048 || K / kGroup % 4 == 0 ? 1 : plan_mid(M, K, N).SK;
    const int panels = M <= 64 ? panel_splits(M, K, N) : 0;
    if (panels > 0) return panels;
    return M <= 128 || blocks128(M, N) < kTiledMinBlocks ? plan_mid(M, K, N).SK : 1;
}

// `partials`: whether the call has memory for them.
inline RowsPlan rows_call(int64_t M, int64_t K, int64_t N, bool partials = true) {
    return plan_rows(M, K, N, partials ? row_splits(M, K, N) : 1);
}
inline size_t rows_workspace_bytes(int64_t M, int64_t K, int64_t N) {
    const RowsPlan p = rows_call(M, K, N);
    return p.SK > 1 ? (size_t)p.SK * (size_t)M * (size_t)N * sizeof(float) : 0;
}

// Layers that give half of the CUs a workgroup without a split: 17..64 rows also run without the partials that the query asks for.
inline bool runs_unsplit(int64_t M, int64_t K, int64_t N) {
    return M <= 64 && rows_kernels_fit(M, K) && N / kTileRows >= 1024;
}

}  // namespace dmr
