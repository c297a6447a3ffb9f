// Launch planning of the chunked-panel kernel (w4_wide.hip): pure host arithmetic for 256 CUs.
#pragma once
#include "common.hpp"

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

// 17 <= M <= 64.  K is split until every CU has a workgroup, while a split keeps two chunks or more: measured against the
// rollout-batch kernel (us at 64 rows, that kernel / this one) 4096 -> 6144 17.5 / 16.5, 14336 -> 4096 26.2 / 24.4,
// 2560 -> 13824 22.5 / 20.2, 8192 -> 8192 29.0 / 25.7; with one chunk per split 4096 -> 4096 13.4 / 15.1, 2048 -> 3072
// 10.8 / 11.3.  (Splits x column blocks <= 256: the partials of 64 rows take at most 8 MiB.)
inline WidePlan plan_wide(int64_t M, int64_t K, int64_t N) {
    WidePlan p{};
    p.ok = false;
    if (M < 17 || M > 64 || M * K >= (int64_t(1) << 31)) return p;
    const int64_t groups = K / kGroup, tiles = N / kTileRows;
    if (groups % kWideChunk != 0) return p;
    p.MT = (int)((M + 15) / 16);
    const int nch = (int)(groups / kWideChunk);
    const int64_t wgs = (tiles + kWideTilesPerWg - 1) / kWideTilesPerWg;
    int sk = (int)(kCus / wgs);
    sk = sk < 1 ? 1 : sk > nch ? nch : sk;
    p.cps = (nch + sk - 1) / sk;
    p.SK = (nch + p.cps - 1) / p.cps;
    p.ok = p.SK > 1 && p.cps >= 2;
    if (!p.ok && tiles >= 128 * kWideTilesPerWg) {      // half of the CUs or more without a split
        p.cps = nch;
        p.SK = 1;
        p.ok = true;
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
