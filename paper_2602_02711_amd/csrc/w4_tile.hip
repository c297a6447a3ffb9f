// W4A16 / W3A16 for 17 rows up to several hundred: tiles of 16 MT WM rows by 128 columns, the activations of a chunk of S groups
// staged once per workgroup, the weights straight into registers.
//
// Eight wavefronts: WM along the rows, 2 lanes of four weight tiles (64 columns), S along k, each on its own group of the
// chunk.  The chunk's panel of x (16 MT WM rows x 256 S bytes, 64 KiB at most) sits in one of two LDS buffers; it goes there by
// buffer loads into LDS, one barrier per chunk, 16-byte pieces XOR-swizzled with the row.  (That spreads 16 consecutive lanes over
// all banks, but a 16-byte read is not served so: four conflict cycles each were counted, 9.2e5 of 2.2e6 LDS cycles at 64 rows 4096
// -> 28672; w4_slices.hip the same, bf16_rows.hip none.)  A wave takes its group's 16 A fragments once and feeds each to four weight tiles; every unpacked word feeds
// MT MFMAs.  Weights and scales are requested one chunk ahead into the registers they are used from; loads return in order, so
// they are requested behind the next panel's pieces, and the wait for the panel leaves them in flight.  The group sums of x come
// from MFMAs against all-ones, and a group contributes  acc += s (D - (128 + z) X)  (exact codes, fp32 scale).  The S partial
// tiles meet in LDS (rows padded by 16 bytes), are added in ascending order and stored a row's 8 or 16 bytes per lane.
// K may be split over blockIdx.y (fp32 partials for the shared reduction kernel); blockIdx.z takes blocks of rows.
// Rows beyond M are staged as copies of row M - 1 and never stored; a group past the end is the last one again with scale 0.
//
// What bounds it: a chunk takes 2.2 us at MT = 4 whatever its shape (4 groups x 64 rows, 2 x 128, 1 x 256), 1.9 of them with
// all loads taken out, 1.2 without the fold: its two FMAs per result and group do not overlap with the MFMAs (matrix pipe busy
// 39 %), the unpacking does.  Weights and x alone would take 1.4 and 0.6 us.  The order of the instructions within a wave (k
// steps outside, tiles outside, every load pinned between MFMAs) changed nothing.  Against the kernels it replaced (weights the
// same way, x through registers, two barriers per chunk, LDS reads shared by two tiles), us: 4096 -> 28672 64 rows 33.3 / 25.5,
// 128 rows 58.8 / 45;  128 rows 4096 -> 6144 29.0 / 24.5, 14336 -> 4096 42.3 / 32.8 (200 rows 59.8 / 44.9).
// BITS = 3 runs the same kernel on the 3-bit streaming layout (768-byte blocks, three words per lane).
// HALF multiplies (16 + q) / 2 instead of 128 + q and doubles the sums at the end: the error against fp64 falls from 1.8e-6 to 1.7e-7 of
// the result's rms (3 bits: 3.7e-6 to 2.7e-7), for a shift more per eight codes, 1 .. 4 % of the time above 64 rows (256 rows 4096 ->
// 12288 39.7 / 41.3 us).  It serves the calls that the rescaling GEMM had, whose error grows with K and reaches that of 128 + q at 4096
// (groups, 1.8e-6), 5600 (3 bits) and 7200 (per channel).
#include <type_traits>

#include "half_codes.hpp"
#include "lds_loads.hpp"
#include "mid_plan.hpp"
#include "rows_plan.hpp"
#include "w3_unpack.hpp"

namespace dmr {

namespace {

constexpr uint32_t kOnes = 0x3F803F80u;    // bf16 pair (1.0, 1.0)
constexpr int kWaves = 8, kLanes = 2, R = 4;

template <int MT, int WM, int S>
struct Geo {
    static constexpr int BM = 16 * MT * WM, COLS = 16 * R * kLanes;
    static constexpr int ROWB = S * 256;                     // bytes of a panel row
    static constexpr int PANEL = BM * ROWB;
    static constexpr int XL = PANEL / 1024 / kWaves;         // 1 KiB pieces of a panel per wave
    static constexpr int LD = COLS + 4;
    static constexpr size_t RED = (size_t)S * BM * LD * 4;
    static constexpr size_t LDS = 2 * PANEL > RED ? 2 * PANEL : RED;
    static_assert(WM * kLanes * S == kWaves && PANEL % (1024 * kWaves) == 0, "eight waves share a panel's pieces");
    static_assert(COLS == kTileCols, "the planner assumes this shape");
};

struct Item {
    u32x4_t w[R];          // 3-bit layout: .x .y .z hold the lane's three words
    uint32_t s[R];
};

// out_mode: 0 = fp32 y, 1 = bf16 y, 2 = fp32 partial [split][M][N].  No __restrict__ on what the ring loads from: the loads must
// stay between the barriers they are written between, which the waits count on.
template <int MT, int WM, int S, int BITS, bool HALF>
__global__ __launch_bounds__(64 * kWaves) void w4_tile_kernel(const void *wt, const uint32_t *sz, const uint16_t *x, void *y, int M,
                                                              int64_t K, int64_t N, int groups, int tiles, int gps, int out_mode,
                                                              int szs, const uint16_t *res) {
    using G = Geo<MT, WM, S>;
    // Whether requests past the end of a split read its last group again.  Up to 64 rows they ask for no bytes: 17 / 32 / 64 rows 1024 ->
    // 28672 8.17 / 8.49 / 11.2 us reading, 7.70 / 8.04 / 10.9 not (two chunks to a workgroup, as many again behind them).  Above, the
    // selects cost what the reads do at short K and up to 1 % at K = 14336.
    constexpr bool TAIL = WM > 1;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = wave % S, tw = wave / S % kLanes, wm = wave / (S * kLanes);
    const int c = lane >> 4, j = lane & 15;
    const int gA = (int)blockIdx.y * gps;
    const int gE = min(groups, gA + gps), last = gE - 1;
    const int nch = (gE - gA + S - 1) / S;
    const int m0 = (int)blockIdx.z * G::BM, rows = min(G::BM, M - m0);
    const int tile0 = ((int)blockIdx.x * kLanes + tw) * R;

    // panel staging: piece p = wave XL + u is bytes [1024 p, 1024 p + 1024) of the panel; 16-byte chunk q of a group's 256 bytes
    // of a row lies at q ^ (row & 15)
    constexpr int RPP = 1024 / G::ROWB;               // rows per piece
    const uint16_t *xm = x + (int64_t)m0 * K;
    const uint32_t rowb = (uint32_t)K * 2u, xbytes = (uint32_t)rows * rowb;      // (the launcher checks that a block stays below 4 GiB)
    const int gl_lane = (lane % (S * 16)) >> 4;       // the group of the panel and the row of the piece that a lane fetches
    const int row_lane = lane / (S * 16);
    const uint32_t lane16 = (uint32_t)((lane & 15) ^ row_lane) * 16u;
    uint32_t xrow[G::XL], vrow[G::XL];                // byte offsets of a piece's first row (uniform) and of the lane's row behind it
#pragma unroll
    for (int u = 0; u < G::XL; ++u) {
        const int row0 = (wave * G::XL + u) * RPP;
        xrow[u] = (uint32_t)min(row0, rows - 1) * rowb;
        vrow[u] = RPP == 1 ? 0u : (uint32_t)(min(row0 + row_lane, rows - 1) - min(row0, rows - 1)) * rowb;
    }
    auto panel_offset = [&](int ch) { return (uint32_t)min(gA + ch * S + gl_lane, last) * 256u + lane16; };
    auto fetch_piece = [&](int u, uint32_t koff, uint32_t bytes, int buf) {
        const uint32_t swizzled = koff ^ (uint32_t)(((wave * G::XL + u) * RPP & 15) * 16);
        load16_to_lds(xm, bytes, smem + buf * G::PANEL + (wave * G::XL + u) * 1024, vrow[u] + swizzled, xrow[u]);
    };

    // codes and scale words of the wave's tiles (those past the layer's last tile: copies of it)
    constexpr uint32_t BLOCK = BITS == 4 ? 1024 : 768;
    const int tileb = min(tile0, tiles - 1), spare = tiles - 1 - tileb;
    const int sz_row = szs * (groups - 1) + 1;        // scale words of a tile, in units of 16
    const void *wbuf = static_cast<const uint8_t *>(wt) + (int64_t)tileb * groups * BLOCK;
    const void *sbuf = sz + (int64_t)tileb * sz_row * kTileRows;
    const uint32_t mytiles = (uint32_t)min(R - 1, spare) + 1u;
    const uint32_t wbytes = mytiles * (uint32_t)groups * BLOCK, sbytes = mytiles * (uint32_t)sz_row * 64u;
    const uint32_t wvoff = (uint32_t)lane * (BLOCK / 64), svoff = (uint32_t)j * 4u;
    Item ring[2];
    auto fetch_codes = [&](Item &dst, int r, int g, uint32_t bytes) {
        dst.w[r] = load_codes<BITS>(wbuf, bytes, wvoff, ((uint32_t)min(r, spare) * (uint32_t)groups + (uint32_t)g) * BLOCK);
    };
    auto fetch_scale = [&](Item &dst, int r, int g) {
        dst.s[r] = load_word(sbuf, sbytes, svoff, ((uint32_t)min(r, spare) * (uint32_t)sz_row + (uint32_t)(g * szs)) * 64u);
    };
    constexpr int ITEM_LOADS = R * 2;

    f32x4 acc[R][MT];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[r][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    Frag ones;
    ones.u = make_uint4(kOnes, kOnes, kOnes, kOnes);
    const int abase = (wm * MT * 16 + j) * G::ROWB + s * 256 + (((c * 4) ^ j) * 16);

    // One chunk: the wave's group from buffer and ring slot `buf` (a constant where this is expanded), then the next panel into the
    // other buffer and the group after the next one into the same slot.
    auto chunk_step = [&](int ch, int buf) {
        Item &it = ring[buf];
        const int g = gA + ch * S + s, next = min(g + 2 * S, last);
        const uint32_t koff = panel_offset(ch + 1);
        // past the end of the split: its last group's addresses, and no bytes up to 64 rows
        const uint32_t xb = TAIL || ch + 1 < nch ? xbytes : 0u, wb = TAIL || g + 2 * S < gE ? wbytes : 0u;
        float sc[R], cz[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            sc[r] = g < gE ? __uint_as_float(it.s[r] << 16) : 0.f;
            cz[r] = __uint_as_float(it.s[r] & 0xFFFF0000u);   // -(128 + z)
            if constexpr (HALF) cz[r] = fmaf(cz[r], 0.5f, 56.f);                    // -(16 + z) / 2, exact
        }
        __builtin_amdgcn_sched_barrier(0);
        Frag a[4][MT];
        f32x4 xs[MT], d[2][MT];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint8_t *p = smem + buf * G::PANEL + (abase ^ (t << 4));
            read_frags<MT, 16 * G::ROWB>(p, p, a[t]);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                xs[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t][mt].v, ones.v, t ? xs[mt] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        auto fold = [&](int r) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[r][mt][q] = fmaf(sc[r], fmaf(cz[r], xs[mt][q], d[r & 1][mt][q]), acc[r][mt][q]);
        };
        int u = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                Frag b;
                if constexpr (HALF && BITS == 4) {
                    unpack4_word(it.w[r][t], b);
                } else if constexpr (HALF) {
                    unpack3_chunk(it.w[r], t, b);
                } else if constexpr (BITS == 4) {
                    unpack_word(it.w[r][t], b.w);
                } else {
                    if (t == 0) unpack3_step<0>(it.w[r].x, it.w[r].y, it.w[r].z, b.w);
                    if (t == 1) unpack3_step<1>(it.w[r].x, it.w[r].y, it.w[r].z, b.w);
                    if (t == 2) unpack3_step<2>(it.w[r].x, it.w[r].y, it.w[r].z, b.w);
                    if (t == 3) unpack3_step<3>(it.w[r].x, it.w[r].y, it.w[r].z, b.w);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    d[r & 1][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t][mt].v, b.v, t ? d[r & 1][mt] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            }
            if (r > 0) fold(r - 1);
            // The old codes' last use lies above the fence, so the new ones go to the same registers; without it the compiler
            // keeps both and copies at the end of the loop, which waits for the loads.
            __builtin_amdgcn_sched_barrier(0);
            if (r < R / 2) {
#pragma unroll
                for (; u < (r + 1) * G::XL / (R / 2); ++u) fetch_piece(u, koff, xb, buf ^ 1);
            } else {
                fetch_codes(it, 2 * r - R, next, wb);
                fetch_codes(it, 2 * r - R + 1, next, wb);
            }
        }
        fold(R - 1);
        __builtin_amdgcn_sched_barrier(0);            // likewise the scale words
#pragma unroll
        for (int r = 0; r < R; ++r) fetch_scale(it, r, next);
        __builtin_amdgcn_sched_barrier(0);
        wait_loads<ITEM_LOADS>();                     // the next panel has landed; the group requested behind it may be in flight
        wait_lds();
        bare_barrier();
    };

    {
        const uint32_t koff = panel_offset(0);
#pragma unroll
        for (int u = 0; u < G::XL; ++u) fetch_piece(u, koff, xbytes, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            fetch_codes(ring[p], r, min(gA + p * S + s, last), TAIL || gA + p * S + s < gE ? wbytes : 0u);
            fetch_scale(ring[p], r, min(gA + p * S + s, last));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    wait_loads<ITEM_LOADS>();
    bare_barrier();
    for (int ch = 0; ch + 1 < nch; ch += 2) {         // (an exit in the middle instead of the odd chunk behind costs the ring its registers)
        chunk_step(ch, 0);
        chunk_step(ch + 1, 1);
    }
    if (nch & 1) chunk_step(nch - 1, 0);

    // red[s][row][LD]
    wait_loads<0>();
    bare_barrier();                                   // every wave's last loads into the panels have landed
    float *red = reinterpret_cast<float *>(smem);
    {
        float *dst = red + ((size_t)s * G::BM + wm * MT * 16 + c * 4) * G::LD + tw * R * 16 + j;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int q = 0; q < 4; ++q) dst[(mt * 16 + q) * G::LD + r * 16] = acc[r][mt][q];
    }
    __syncthreads();
    constexpr int QC = G::COLS / 4, QUADS = G::BM * QC, THREADS = 64 * kWaves;
    const int64_t part = out_mode == 2 ? (int64_t)blockIdx.y * M * N : 0;
#pragma unroll
    for (int q0 = 0; q0 < QUADS; q0 += THREADS) {
        const int qi = q0 + tid, row = qi / QC, col = (qi % QC) * 4;
        const int64_t n = (int64_t)blockIdx.x * G::COLS + col;
        if (row >= rows || n >= N) continue;
        const float *src = red + (size_t)row * G::LD + col;
        f32x4 v = *reinterpret_cast<const f32x4 *>(src);
#pragma unroll
        for (int k = 1; k < S; ++k) {
            const f32x4 u = *reinterpret_cast<const f32x4 *>(src + (size_t)k * G::BM * G::LD);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += u[e];
        }
        if constexpr (HALF)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] *= 2.f;
        store_quad(v, y, (int64_t)(m0 + row) * N + n, part, out_mode, res);
    }
}

template <int MT, int WM, int S, int BITS, bool HALF>
hipError_t launch_cfg(const void *wt, const uint32_t *sz, int szs, int64_t K, int64_t N, const uint16_t *x, int M, void *y,
                      int out_mode, const uint16_t *res, const RowsPlan &p, hipStream_t stream) {
    using G = Geo<MT, WM, S>;
    // once per process and kernel instantiation (thread-safe static initialisation)
    static const hipError_t attr_status = hipFuncSetAttribute(reinterpret_cast<const void *>(&w4_tile_kernel<MT, WM, S, BITS, HALF>),
                                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::LDS);
    if (attr_status != hipSuccess) return attr_status;
    const int groups = (int)(K / kGroup), tiles = (int)(N / kTileRows);
    const dim3 grid((unsigned)((N + G::COLS - 1) / G::COLS), (unsigned)p.SK, (unsigned)((M + G::BM - 1) / G::BM));
    hipLaunchKernelGGL((w4_tile_kernel<MT, WM, S, BITS, HALF>), grid, dim3(64 * kWaves), G::LDS, stream, wt, sz, x, y, M, K, N, groups,
                       tiles, p.gps, out_mode, szs, out_mode == 2 ? nullptr : res);
    return hipGetLastError();
}

template <int BITS>
hipError_t launch_tile(const void *wt, const uint32_t *sz, int szs, int64_t K, int64_t N, const uint16_t *x, int64_t M, void *y,
                       bool out_f32, const uint16_t *res, void *ws, const RowsPlan &p, hipStream_t stream) {
    const bool split = p.SK > 1;
    if (split && !ws) return hipErrorInvalidValue;
    void *dst = split ? ws : y;
    const int out_mode = split ? 2 : (out_f32 ? 0 : 1);
    const int iM = (int)M;
    hipError_t e = hipErrorInvalidValue;
    auto go = [&](auto half) {
        constexpr bool HALF = decltype(half)::value;
        if (p.WM == 2) {
            if (p.MT == 3) e = launch_cfg<3, 2, 2, BITS, HALF>(wt, sz, szs, K, N, x, iM, dst, out_mode, res, p, stream);
            if (p.MT == 4) e = launch_cfg<4, 2, 2, BITS, HALF>(wt, sz, szs, K, N, x, iM, dst, out_mode, res, p, stream);
            return;
        }
        if constexpr (!HALF)
            if (p.MT == 2) e = launch_cfg<2, 1, 4, BITS, HALF>(wt, sz, szs, K, N, x, iM, dst, out_mode, res, p, stream);
        if (p.MT == 3) e = launch_cfg<3, 1, 4, BITS, HALF>(wt, sz, szs, K, N, x, iM, dst, out_mode, res, p, stream);
        if (p.MT == 4) e = launch_cfg<4, 1, 4, BITS, HALF>(wt, sz, szs, K, N, x, iM, dst, out_mode, res, p, stream);
    };
    if (p.half) go(std::true_type{});
    else go(std::false_type{});
    if (e != hipSuccess || !split) return e;
    return launch_splitk_reduce(static_cast<const float *>(ws), y, M * N, p.SK, out_f32, res, stream);
}

}  // namespace

hipError_t launch_w4_tile(const LayerView &L, const uint16_t *x, int64_t M, void *y, bool out_f32, const uint16_t *res, void *ws,
                          const RowsPlan &p, hipStream_t stream) {
    return launch_tile<4>(L.wt, L.sz, L.szs, L.K, L.N, x, M, y, out_f32, res, ws, p, stream);
}

hipError_t launch_w3_tile(const LayerView3 &L, const uint16_t *x, int64_t M, void *y, bool out_f32, const uint16_t *res, void *ws,
                          const RowsPlan &p, hipStream_t stream) {
    return launch_tile<3>(L.wt, L.sz, 1, L.K, L.N, x, M, y, out_f32, res, ws, p, stream);
}

}  // namespace dmr
