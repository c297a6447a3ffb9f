// Launch planning of the two kernels for 17 rows up to several hundred (w4_tile.hip, w4_slices.hip): pure host arithmetic for
// 256 CUs.
#pragma once
#include "common.hpp"

namespace dmr {

struct RowsPlan {
    bool slices;    // w4_slices.hip, else w4_tile.hip
    int MT, WM;     // row tiles of 16 per wave, waves along the rows (tile kernel)
    int R;          // weight tiles per workgroup (slices kernel)
    int SK, gps;    // splits of K over blockIdx.y, groups per split (the last one may have fewer)
    bool half;      // tile kernel: codes in units that keep the sums small
};

constexpr int kTileCols = 128;      // columns of a workgroup of the tile kernel

// Above 64 rows, both formats: the tiled MFMA GEMMs win from about 140 output blocks of 128 x 128 on (measured: ahead at 144 and from
// there on, on 128-row tiles up to 256 blocks and on 256-row tiles beyond; behind at 128), but not where one round of the tile
// kernel covers up to 512 rows (rows_fit_one_round).
constexpr int kTiledMinBlocks = 140;
inline int64_t blocks128(int64_t M, int64_t N) { return ((M + 127) / 128) * ((N + 127) / 128); }

// Rows of activations and of a layer's tiles are addressed with 32-bit byte offsets inside a block of at most 128 rows.
inline bool rows_kernels_fit(int64_t M, int64_t K) { return M >= 17 && K < (int64_t(1) << 24); }

// The candidate with the least estimated time.  us per launch = rounds of 256 workgroups x (fixed + chunks x time of a chunk), plus
// the reduction's launch and its partials where K is split:
//   tile kernel, 128 columns:  6.2 + chunks x (1.3 / 1.9 / 2.3 for 2 / 3 / 4 row tiles, 4 groups each, blocks of up to 64 rows;
//     1.7 / 2.1 for row blocks of 96 / 128, 2 groups each).  Above 64 rows the smaller blocks are offered while one round holds
//     them: 96 rows 1024 -> 16384 in two blocks of 48 8.9 us, in one of 96 on half of the chip 12.6
//   slices kernel, 16 R columns, blocks of 64 rows at most:  4.5 + ceil(groups / 8) x (0.24 + MT (0.18 + 0.06 R) + 0.18 R); two of
//     its workgroups share a CU at two row tiles and R <= 2, and 257 of them take what 512 do, 1.5 times the time of 256 (32 rows 8192 ->
//     9216 in 288 workgroups 23.9 us, in 144 of R = 4 17.8)
//   reduction: 2.0 + 2.3 per million partials
// Fitted to 16 to 20 candidates at each of 750 points (17 .. 512 rows, K = 512 .. 14336, N = 1024 .. 28672, weights from memory) and
// checked on 3388: what it picks takes 0.3 % more than the best of its candidates on average, 19 % at worst.  Against the kernels
// these replaced (one panel or one group of x at a time through registers) 1.36 x up to 64 rows and 1.49 x above over 5020 points of
// INT4, none of them slower.
// us, old / picked:  17 rows 4096 -> 6144 11.3 / 8.9;  32 rows 14336 -> 4096 17.4 / 15.0;  64 rows 4096 -> 28672 33.3 / 25.5, 4096 ->
// 4096 13.0 / 10;  96 rows 4096 -> 28672 48.7 / 39;  200 rows 4096 -> 6144 38.5 / 30, 14336 -> 4096 59.8 / 45.
// `max_splits`: what the caller's workspace holds.
inline RowsPlan plan_rows(int64_t M, int64_t K, int64_t N, int max_splits) {
    RowsPlan best{};
    double least = 1e30;
    const int groups = (int)(K / kGroup);
    const int64_t tiles = N / kTileRows;
    auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    auto offer = [&](const RowsPlan &p, double us) {
        if (us < least) {
            least = us;
            best = p;
        }
    };
    // calls of a size that the tiled GEMM would have, while it is the more exact one on 128 + q (see w4_tile.hip)
    const bool half = M > 128 && blocks128(M, N) >= kTiledMinBlocks && K < 8192;
    for (int sk = 1; sk <= max_splits; ++sk) {
        const int gps = (int)cdiv(groups, sk);
        if (sk > 1 && cdiv(groups, gps) != sk) continue;
        const double red = sk > 1 ? 2.0 + 2.3e-6 * (double)sk * (double)M * (double)N : 0.0;
        auto tile = [&](int MT, int WM) {
            const int64_t wgs = cdiv(N, kTileCols) * sk * cdiv(M, 16 * MT * WM);
            if (M > 64 && WM == 1 && wgs > kCus) return;
            const double chunk = WM == 1 ? (MT == 2 ? 1.28 : MT == 3 ? 1.9 : 2.31) : (MT == 3 ? 1.73 : 2.11);
            offer({false, MT, WM, 0, sk, gps, half}, (double)cdiv(wgs, kCus) * (6.25 + (double)cdiv(gps, WM == 1 ? 4 : 2) * chunk) + red);
        };
        const int64_t blocks = cdiv(M, 64);
        const int MT = (int)cdiv(cdiv(M, blocks), 16);
        if (M > 64) {
            tile(3, 2);
            tile(4, 2);
            tile((int)cdiv(cdiv(M, cdiv(M, 48)), 16), 1);
        }
        tile(MT, 1);
        for (int R = 1; R <= 4; R *= 2) {
            const int64_t wgs = cdiv(tiles, R) * sk * blocks;
            if (wgs > (MT == 2 && R <= 2 ? 2 : 1) * kCus) continue;
            const double step = 0.24 + MT * (0.18 + 0.06 * R) + 0.18 * R;
            offer({true, MT, 1, R, sk, gps, false}, (4.51 + (double)cdiv(gps, 8) * step) * (wgs > kCus ? 1.5 : 1.0) + red);
        }
    }
    return best;
}

// 65 .. 512 rows on layers that the crossover in blocks of 128 x 128 would give to the tiled MFMA kernels: the tile kernel while
// its workgroups fit one round (us, tiled / this one: 200 rows 4096 -> 12288 54.9 / 39.5, 400 rows 4096 -> 6144 51.2 / 34.2, 512
// rows 4096 -> 8192 54.3 / 43.6 and 14336 -> 8192 160 / 134; in two rounds 200 rows 4096 -> 28672 80 / 81, 512 rows 4096 -> 12288
// 74.5 / 79.5).
inline bool rows_fit_one_round(int64_t M, int64_t K, int64_t N) {
    if (!rows_kernels_fit(M, K) || M > 512) return false;
    const int64_t cols = (N + kTileCols - 1) / kTileCols;
    return cols * ((M + 127) / 128) <= kCus;
}

inline bool rows_beat_tiled(int64_t M, int64_t K, int64_t N) {
    return M <= 128 || blocks128(M, N) < kTiledMinBlocks || rows_fit_one_round(M, K, N);
}

hipError_t launch_w4_tile(const LayerView &L, const uint16_t *x, int64_t M, void *y, bool out_f32, const uint16_t *res, void *ws,
                          const RowsPlan &p, hipStream_t stream);
hipError_t launch_w3_tile(const LayerView3 &L, const uint16_t *x, int64_t M, void *y, bool out_f32, const uint16_t *res, void *ws,
                          const RowsPlan &p, hipStream_t stream);
hipError_t launch_w4_slices(const LayerView &L, const uint16_t *x, int64_t M, void *y, bool out_f32, const uint16_t *res, void *ws,
                            const RowsPlan &p, hipStream_t stream);
hipError_t launch_w3_slices(const LayerView3 &L, const uint16_t *x, int64_t M, void *y, bool out_f32, const uint16_t *res, void *ws,
                            const RowsPlan &p, hipStream_t stream);

// `ws`: fp32 partials for the plan's splits.
inline hipError_t launch_w4_rows(const LayerView &L, const uint16_t *x, int64_t M, void *y, bool out_f32, const uint16_t *res, void *ws,
                                 const RowsPlan &p, hipStream_t stream) {
    return (p.slices ? launch_w4_slices : launch_w4_tile)(L, x, M, y, out_f32, res, ws, p, stream);
}
inline hipError_t launch_w3_rows(const LayerView3 &L, const uint16_t *x, int64_t M, void *y, bool out_f32, const uint16_t *res, void *ws,
                                 const RowsPlan &p, hipStream_t stream) {
    return (p.slices ? launch_w3_slices : launch_w3_tile)(L, x, M, y, out_f32, res, ws, p, stream);
}

}  // namespace dmr
