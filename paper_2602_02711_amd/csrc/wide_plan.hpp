// Splits of K that a workspace is sized for, 17..64 rows: pure host arithmetic for 256 CUs.
#pragma once
#include "common.hpp"
#include "mid_plan.hpp"
#include "rows_plan.hpp"

namespace dmr {

struct WidePlan {
    bool ok;
    int MT;    // row tiles of 16
    int SK;    // splits of K over blockIdx.y
    int cps;   // chunks per split (the last one may have fewer)
};

constexpr int kWideChunk = 4;       // groups
constexpr int kWideTilesPerWg = 8;  // row tiles of 128 columns

// 17 <= M <= 64: how many fp32 partials the workspace of a call holds, which bounds the splits that plan_rows (rows_plan.hpp)
// chooses from, on layers whose K divides into chunks of four groups.  Layers of 1024 row tiles or more split K in two if that
// fills the CUs and leaves each half three chunks, narrower ones until every CU has 128 columns while a split keeps two chunks;
// elsewhere, and where `ok` is false, the splits are those of plan_mid.  Sizes that callers hold stay valid, and a call of 64 rows
// needs at most 8 MiB (splits x column blocks <= 256), the fixed scratch of dmr_qlinear_forward_static: two splits of more than
// seven chunks give way to plan_mid's two or four times as many only while those fit it.  `with_workspace` false: unsplit or not
// at all.
inline WidePlan plan_wide(int64_t M, int64_t K, int64_t N, bool with_workspace = true) {
    WidePlan p{};
    p.ok = false;
    if (M > 64 || !rows_kernels_fit(M, K)) return p;
    const int64_t groups = K / kGroup, tiles = N / kTileRows;
    if (groups % kWideChunk != 0) return p;
    p.MT = (int)((M + 15) / 16);
    const int nch = (int)(groups / kWideChunk);
    const int64_t wgs = (tiles + kWideTilesPerWg - 1) / kWideTilesPerWg;
    const bool wide = tiles >= 128 * kWideTilesPerWg;
    int sk = (int)(kCus / wgs);
    sk = sk < 1 || !with_workspace || (wide && nch < 6) ? 1 : sk > nch ? nch : sk;
    p.cps = (nch + sk - 1) / sk;
    p.SK = (nch + p.cps - 1) / p.cps;
    if (wide) {
        p.ok = true;
    } else if (p.SK > 1 && p.cps >= 2) {
        const MidPlan m = plan_mid(M, K, N);
        const bool one_round = m.R == 1 && m.wgs <= kCus && m.gps % 4 == 0;
        const bool long_halves = p.SK == 2 && p.cps > 7;
        p.ok = !one_round && (!long_halves || (size_t)m.SK * (size_t)(M * N) * sizeof(float) > DMR_STATIC_SCRATCH_BYTES);
    }
    return p;
}

inline bool w4_wide_applies(int64_t M, int64_t K, int64_t N) { return plan_wide(M, K, N).ok; }
inline size_t w4_wide_workspace_bytes(int64_t M, int64_t K, int64_t N) {
    const WidePlan p = plan_wide(M, K, N);
    return p.ok && p.SK > 1 ? (size_t)p.SK * (size_t)M * (size_t)N * sizeof(float) : 0;
}

}  // namespace dmr
