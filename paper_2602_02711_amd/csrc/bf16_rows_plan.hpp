// Launch planning of the bf16 kernel that keeps its activations in registers (bf16_rows.hip): pure host arithmetic for 256 CUs.
#pragma once
#include "common.hpp"

namespace dmr {

struct Bf16RowsPlan {
    bool ok;
    int MT, GPW;    // row tiles of 16, groups of 128 k that a wave holds
    int SK, gps;    // splits of K over blockIdx.y, groups per split
    int tpw;        // weight tiles of 16 rows per workgroup
};

// MT GPW 16 <= 128 registers of activations, eight waves along K; K is split as little as that allows (a split costs its partials
// and a launch: 32 rows 4096 -> 4096 whole 11.6 us, in two 14.7; 4096 -> 28672 42.1 / 47.8), at most into max_splits, what the
// caller's workspace holds.  At 2..8 rows the direct-from-L2 kernel, whose workgroups are smaller, keeps layers of up to 2.6 million
// weights, rows of up to 512, and layers of up to 4096 outputs (one round of its workgroups) while K <= 1536, or 2048 up to four rows
// (us, that kernel / this one, 2 rows: 1024 -> 4096 4.0 / 4.4, 2048 -> 4096 6.2 / 6.4; over K = 512 .. 8192 x N = 1024 .. 16384 at 2, 4
// and 8 rows it is ahead by 1..18 % there, behind by up to 60 % elsewhere, but for 8192 outputs at K = 2048 and 4096, 0.91 .. 0.98).
inline Bf16RowsPlan plan_bf16_rows(int64_t M, int64_t K, int64_t N, int max_splits) {
    Bf16RowsPlan p{};
    p.ok = false;
    if (M < 2 || M > 64 || K >= (int64_t(1) << 22) || N >= (int64_t(1) << 24)) return p;      // 32-bit byte offsets
    if (M <= 8 && (K * N <= (int64_t(5) << 19) || K <= 512 || (N <= 4096 && K <= (M <= 4 ? 2048 : 1536)))) return p;
    const int groups = (int)(K / kGroup), tiles = (int)(N / kTileRows);
    p.MT = (int)((M + 15) / 16);
    const int held = p.MT == 1 ? 8 : p.MT == 2 ? 4 : 2;
    const int sk = (groups + 8 * held - 1) / (8 * held);
    if (sk > max_splits) return p;
    p.gps = (groups + sk - 1) / sk;
    p.SK = (groups + p.gps - 1) / p.gps;
    const int need = (p.gps + 7) / 8;
    p.GPW = need <= 4 ? need : need <= 6 ? 6 : 8;
    const int wgs = kCus / p.SK > 0 ? kCus / p.SK : 1;
    p.tpw = (tiles + wgs - 1) / wgs;
    p.ok = (int64_t)p.tpw * kTileRows * K * 2 < (int64_t(1) << 32);
    return p;
}

hipError_t launch_bf16_rows(const uint16_t *w, const uint16_t *x, int64_t M, int64_t K, int64_t N, void *y, bool out_f32,
                            const uint16_t *res, void *ws, const Bf16RowsPlan &p, hipStream_t stream);

}  // namespace dmr
