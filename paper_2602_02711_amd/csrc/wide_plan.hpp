// Launch planning of the chunked-panel kernel (w4_wide.hip): pure host arithmetic for 256 CUs.
#pragma once
#include "common.hpp"
#include "mid_plan.hpp"

namespace dmr {

struct WidePlan {
    bool ok;
    int MT;    // row tiles of 16
    int SK;    // splits of K over blockIdx.y
    int cps;   // chunks per split (the last one may have fewer)
};

constexpr int kWideChunk = 4;       // groups per LDS panel
constexpr int kWideTilesPerWg = 8;  // 4 tile lanes x 2 tiles per wave

inline size_t wide_lds_bytes(int MT, int R, int S, int CG) {
    const size_t panels = 2 * (size_t)(MT * 16) * (CG * 16 + 1) * 16 + 2 * (size_t)CG * MT * 4 * 16;
    const size_t red = S > 1 ? (size_t)8 * R * MT * 1024 : 0;
    return panels > red ? panels : red;
}

// 17 <= M <= 64.  Layers of 1024 row tiles or more (half of the CUs without a split) are this kernel's; K is split in two
// there if that fills the CUs and leaves each half three chunks (us unsplit / split at 17 and 64 rows: 3072 -> 16384 16.4 / 13.9
// and 23.4 / 21.1, 4096 -> 16384 20.1 / 16.6 and 29.0 / 24.5; but 2048 -> 16384 17.1 / 17.9, 1536 -> 16384 14.2 / 17.2 at 64).
// Narrower layers split K until every CU has a workgroup, while a split keeps two chunks, and go here where that beats the
// rollout-batch kernel.  16 K x 12 N x 17, 32, 48, 64 rows, both formats; us at 17 / 64 rows, that kernel then this one:
//   its two weight tiles per wave, or more workgroups than CUs:  4096 -> 6144 11.4 / 18.3, 11.1 / 16.5;  14336 -> 4096 18.6 / 27.1,
//     17.0 / 24.3;  8192 -> 8192 18.8 / 28.9, 17.5 / 25.3;  4608 -> 8192 14.9 / 22.8, 13.2 / 19.4
//   all its workgroups at once with one tile each and whole steps of its four groups:  1536 -> 12288 8.2 / 11.9, 10.3 / 15.8;
//     6144 -> 4096 11.4 / 16.5, 11.7 / 16.8;  12288 -> 2048 12.3 / 17.3, 13.0 / 18.2: left to it (9 groups, 4608 -> 4096: 11.3 /
//     16.4, 11.0 / 15.8;  14 groups, 3584 -> 5120: 11.6 / 17.4, 10.6 / 15.7)
//   two splits of more than seven chunks:  14336 -> 12288 31.5 / 48.6, 35.9 / 52.8: left to it while its partials, twice or four
//     times as many, stay within the fixed scratch of dmr_qlinear_forward_static, which such a call otherwise would not fit
// (Splits x column blocks <= 256: the partials of 64 rows take at most 8 MiB.)  `with_workspace` false: unsplit or not at all.
inline WidePlan plan_wide(int64_t M, int64_t K, int64_t N, bool with_workspace = true) {
    WidePlan p{};
    p.ok = false;
    if (M < 17 || M > 64 || M * K >= (int64_t(1) << 31)) return p;
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

size_t w4_wide_workspace_bytes(int64_t M, int64_t K, int64_t N);     // fp32 partials when K is split
bool w4_wide_applies(int64_t M, int64_t K, int64_t N);
hipError_t launch_w4_wide(const LayerView &L, const uint16_t *x, int64_t M, void *y, bool out_f32,
                          const uint16_t *res, void *ws, hipStream_t stream);
// The same kernel on a 3-bit layer.
hipError_t launch_w3_wide(const LayerView3 &L, const uint16_t *x, int64_t M, void *y, bool out_f32,
                          const uint16_t *res, void *ws, hipStream_t stream);

}  // namespace dmr
