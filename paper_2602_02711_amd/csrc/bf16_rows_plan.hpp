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

// Short rows, where the fixed part of a launch decides (the first items of eight rings and the activations, then a barrier per tile).
// From K and N = 256 .. 5120 x 1024 .. 28672 at 2..16 rows, up to 1024 at 17..64 rows, weights from memory; us, the other kernel / this one:
//   2..8 rows, the direct-from-L2 kernel's smaller workgroups are ahead, least with most rows
//     on any width up to K = 896 .. 640          4 rows 640 -> 8192 4.5 / 5.3, 768 -> 16384 7.3 / 7.9;  8 rows 640 -> 12288 5.9 / 6.5
//     up to 4096 outputs to K = 2560 .. 1536     2 rows 1024 -> 4096 4.0 / 4.4, 2560 -> 4096 6.4 / 7.0
//     up to 8192, one round of them, to K = 1536 .. 768    2 rows 1280 -> 8192 6.3 / 6.9
//     8192 itself also at K = 2048 and 4096 (2 rows 9.3 / 10.2 and 15.1 / 17.2; 2560 and 3072 0.99 and 0.91 of its time)
//   9..64 rows up to K = 512, the rollout-batch kernel on 4097 .. 16384 outputs (32 rows 512 -> 9216 5.4 / 6.5; 512 -> 4096 and 18432 1.09
//     and 1.18 of this one's time), at K <= 256 also beyond and, at 17..32 rows, below
// What is left behind the other kernel: 2 and 3 rows 4224 .. 4608 -> 4096 (4 %), 2048 -> 20480 (5 %), 2..5 rows 2048 -> 12288 (4 %), 8 rows 768 ->
// 12288 (4 %); and 9..16 rows 512 -> 16384 behind a kernel that is gone (6.3 / 5.8).
inline bool bf16_rows_too_short(int64_t M, int64_t K, int64_t N) {
    if (M <= 8) {
        const int c = M <= 5 ? 0 : M <= 7 ? 1 : 2;
        constexpr int64_t any[3] = {896, 768, 640}, to4096[3] = {2560, 1792, 1536}, to8192[3] = {1536, 1280, 768};
        if (K <= any[c] || (M <= 3 && K <= 1024 && N >= 16384)) return true;
        if (N <= 4096) return K <= to4096[c];
        return N <= 8192 && (K <= to8192[c] || (N > 8128 && (K == 2048 || K == 4096)));
    }
    if (K > 512) return false;
    if (N <= 4096) return K <= 256 && M > 16 && M <= 32;
    return K <= 256 || N <= 16384;
}

// MT GPW 16 <= 128 registers of activations, eight waves along K (GPW 5 and 7 for one row tile: with 6 and 8 in their place 4608 and 6656
// deep layers took 2 .. 4 % more); K is split as little as that allows (a split costs its partials
// and a launch: 32 rows 4096 -> 4096 whole 11.6 us, in two 14.7; 4096 -> 28672 42.1 / 47.8), at most into max_splits, what the
// caller's workspace holds.
inline Bf16RowsPlan plan_bf16_rows(int64_t M, int64_t K, int64_t N, int max_splits) {
    Bf16RowsPlan p{};
    p.ok = false;
    if (M < 2 || M > 64 || K >= (int64_t(1) << 22) || N >= (int64_t(1) << 24)) return p;      // 32-bit byte offsets
    if (bf16_rows_too_short(M, K, N)) return p;
    const int groups = (int)(K / kGroup), tiles = (int)(N / kTileRows);
    p.MT = (int)((M + 15) / 16);
    const int held = p.MT == 1 ? 8 : p.MT == 2 ? 4 : 2;
    const int sk = (groups + 8 * held - 1) / (8 * held);
    if (sk > max_splits) return p;
    p.gps = (groups + sk - 1) / sk;
    p.SK = (groups + p.gps - 1) / p.gps;
    p.GPW = (p.gps + 7) / 8;
    const int wgs = kCus / p.SK > 0 ? kCus / p.SK : 1;
    p.tpw = (tiles + wgs - 1) / wgs;
    p.ok = (int64_t)p.tpw * kTileRows * K * 2 < (int64_t(1) << 32);
    return p;
}

hipError_t launch_bf16_rows(const uint16_t *w, const uint16_t *x, int64_t M, int64_t K, int64_t N, void *y, bool out_f32,
                            const uint16_t *res, void *ws, const Bf16RowsPlan &p, hipStream_t stream);

}  // namespace dmr
