// W4A16 / W3A16 for 17 rows up to several hundred where the workgroups of the staged-panel kernel would be few: eight wavefronts
// of a workgroup share 16 R columns and split K between them, so nothing is shared and there is no barrier until the partial
// tiles meet.
//
// A wave owns a run of groups.  It stages its group of x (16 MT rows x 256 bytes) in an LDS slot of its own by buffer loads into
// LDS (16-byte pieces XOR-swizzled with the row), takes all 4 MT A fragments into registers, and requests the next group into
// the same slot while it works: the sums of x from MFMAs against all-ones, then tile by tile unpacking, MFMAs, the fold
// acc += s (D - (128 + z) X) of the tile before, and the request for the tile's next codes, into the registers they are used
// from.  The scale words of four groups come into LDS with one 256-byte load per tile.  Requests past a wave's last group go to
// a resource of no bytes, so the counts that the waits rest on never change.  The eight partial tiles are added in ascending
// order; quads of lanes transpose 4 x 4 so that a lane stores four columns.  Rows beyond the last are copies of it.
// blockIdx.y splits K (fp32 partials for the shared reduction kernel), blockIdx.z takes blocks of 16 MT rows.
//
// What bounds it (64 rows 4096 -> 6144, R = 2, 12.9 us): 512 KiB of x per CU at about 35 bytes a clock, then launch, first loads
// and the final sum, 6 us.  Against the kernels it replaced (one or two tiles per wave, K split over workgroups, fp32 partials
// and a second launch), us at 64 / 32 rows: 4096 -> 6144 16.7 / 12.9 and 12.1 / 9.5; 14336 -> 4096 (R = 4, K in four) 24.1 / 19.7
// and 17.6 / 15.0; 8192 -> 8192 25.1 / 21.5 and 18.3 / 15.0.  Wide layers are the staged-panel kernel's: 4096 -> 28672, 64 rows 33.9
// here (448 workgroups, one to a CU).
#include "lds_loads.hpp"
#include "mid_plan.hpp"
#include "rows_plan.hpp"
#include "w3_unpack.hpp"
#include "wave_share.hpp"

namespace dmr {

namespace {

constexpr uint32_t kOnes = 0x3F803F80u;    // bf16 pair (1.0, 1.0)
constexpr int kWaves = kSharingWaves;      // all along k

template <int MT, int R>
struct Geo {
    static constexpr int XB = MT * 16 * 256;                 // a wave's slot: one group of x, rows of 256 bytes
    static constexpr int SB = R * 256;                       // scale words of four groups
    static constexpr int SLOT = XB + 2 * SB;
    static constexpr size_t RED = (size_t)R * MT * kWaves * 1024;
    static constexpr size_t LDS = (size_t)kWaves * SLOT > RED ? (size_t)kWaves * SLOT : RED;
    static_assert(LDS <= 160 * 1024, "");
};

template <int MT, int R, int BITS>
__global__ __launch_bounds__(64 * kWaves, MT == 2 && R <= 2 ? 4 : 2) void w4_slices_kernel(const void *wt, const uint32_t *sz, const uint16_t *x, void *y, int M,
                                                              int64_t K, int64_t N, int groups, int tiles, int gps, int out_mode,
                                                              int szs, const uint16_t *res) {
    using G = Geo<MT, R>;
    constexpr int XL = MT * 4;                        // 1 KiB pieces of a group of x: four rows each
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane >> 4, j = lane & 15;
    const WaveShare mine = wave_share(groups, gps, (int)blockIdx.y, wave);
    const int g0 = mine.g0, n = mine.n;
    const int tileb = (int)blockIdx.x * R;            // the last workgroup may have fewer than R tiles of its own
    uint8_t *slot = smem + wave * G::SLOT;

    // piece u of a group: rows 4 u + lane / 16; 16-byte chunk q of a row lies at q ^ (row & 15)
    const int m0 = (int)blockIdx.z * MT * 16, rows = min(MT * 16, M - m0);
    const uint16_t *xm = x + (int64_t)m0 * K;
    const uint32_t rowb = (uint32_t)K * 2u, xbytes = (uint32_t)rows * rowb;      // (the launcher checks that a block stays below 4 GiB)
    uint32_t voff[XL];
#pragma unroll
    for (int u = 0; u < XL; ++u)
        voff[u] = (uint32_t)min(4 * u + c, rows - 1) * rowb + (uint32_t)((j ^ c) ^ (4 * (u & 3))) * 16u;
    auto fetch_x = [&](int u, uint32_t goff, uint32_t bytes) { load16_to_lds(xm, bytes, slot + u * 1024, voff[u], goff); };

    constexpr uint32_t BLOCK = BITS == 4 ? 1024 : 768;
    const int sz_row = szs * (groups - 1) + 1;        // scale words of a tile, in units of 16
    const void *wbuf = static_cast<const uint8_t *>(wt) + (int64_t)tileb * groups * BLOCK;
    const void *sbuf = sz + (int64_t)tileb * sz_row * kTileRows;
    const uint32_t mytiles = (uint32_t)min(R, tiles - tileb);
    const uint32_t wbytes = mytiles * (uint32_t)groups * BLOCK, sbytes = mytiles * (uint32_t)sz_row * 64u;
    const uint32_t wvoff = (uint32_t)lane * (BLOCK / 64);
    u32x4_t code[R];
    auto fetch_codes = [&](int r, int g, uint32_t bytes) {
        code[r] = load_codes<BITS>(wbuf, bytes, wvoff, ((uint32_t)min(r, (int)mytiles - 1) * (uint32_t)groups + (uint32_t)g) * BLOCK);
    };
    // scale words of groups [g, g + 4), lane = (group, row), those past the last group copies of its own
    auto fetch_scales = [&](int g, int buf, uint32_t bytes) {
        const uint32_t v = (uint32_t)min(g + c, groups - 1) * (uint32_t)szs * 64u + (uint32_t)j * 4u;
#pragma unroll
        for (int r = 0; r < R; ++r)
            load4_to_lds(sbuf, bytes, slot + G::XB + buf * G::SB + r * 256, v, (uint32_t)min(r, (int)mytiles - 1) * (uint32_t)sz_row * 64u);
    };

    f32x4 acc[R][MT];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[r][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    Frag ones;
    ones.u = make_uint4(kOnes, kOnes, kOnes, kOnes);
    const int abase = j * 256 + (((c * 4) ^ j) * 16);

    if (n > 0) {
        fetch_scales(g0, 0, sbytes);
#pragma unroll
        for (int u = 0; u < XL; ++u) fetch_x(u, (uint32_t)g0 * 256u, xbytes);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < R; ++r) fetch_codes(r, g0, wbytes);
        __builtin_amdgcn_sched_barrier(0);
    }
    for (int b = 0, sbuf_i = 0; b < n; b += 4, sbuf_i ^= 1) {
        wait_lds();                                   // nothing of the buffer's old words is still to be read
        fetch_scales(g0 + b + 4, sbuf_i ^ 1, b + 4 < n ? sbytes : 0u);
        const uint8_t *sw = slot + G::XB + sbuf_i * G::SB;
        const int in_block = min(4, n - b);
        for (int i = 0; i < in_block; ++i) {
            const int next = requested_group(mine, b + i + 1, groups);
            const bool more = b + i + 1 < n;
            __builtin_amdgcn_sched_barrier(0);
            if (i == 0)
                wait_loads<R + R>();                  // (the scale words of the next four groups were requested behind the codes)
            else
                wait_loads<R>();                      // x of this group has landed; codes requested behind it may be in flight
            Frag a[4][MT];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const uint8_t *p = slot + (abase ^ (t << 4));
                read_frags<MT, 16 * 256>(p, p, a[t]);
            }
            wait_lds();                               // the slot is free
            __builtin_amdgcn_sched_barrier(0);
            f32x4 xs[MT];
            const uint32_t xb = more ? xbytes : 0u, goff = (uint32_t)next * 256u;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    xs[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t][mt].v, ones.v, t ? xs[mt] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    fetch_x(t * MT + mt, goff, xb);
                    __builtin_amdgcn_sched_barrier(0);
                }
            f32x4 d[2][MT];
            float sc[2], cz[2];
            auto fold = [&](int r) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        acc[r][mt][q] = fmaf(sc[r & 1], fmaf(cz[r & 1], xs[mt][q], d[r & 1][mt][q]), acc[r][mt][q]);
            };
            const uint32_t wb = more ? wbytes : 0u;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint8_t *sp = sw + r * 256 + i * 64 + j * 4;
                const uint32_t word = read_word(sp, sp);
                sc[r & 1] = __uint_as_float(word << 16);
                cz[r & 1] = __uint_as_float(word & 0xFFFF0000u);      // -(128 + z)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    Frag w;
                    if constexpr (BITS == 4) {
                        unpack_word(code[r][t], w.w);
                    } else {
                        if (t == 0) unpack3_step<0>(code[r].x, code[r].y, code[r].z, w.w);
                        if (t == 1) unpack3_step<1>(code[r].x, code[r].y, code[r].z, w.w);
                        if (t == 2) unpack3_step<2>(code[r].x, code[r].y, code[r].z, w.w);
                        if (t == 3) unpack3_step<3>(code[r].x, code[r].y, code[r].z, w.w);
                    }
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        d[r & 1][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t][mt].v, w.v, t ? d[r & 1][mt] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                }
                if (r > 0) fold(r - 1);
                __builtin_amdgcn_sched_barrier(0);    // the codes' last use lies above: the load goes to the same registers
                fetch_codes(r, next, wb);
            }
            fold(R - 1);
        }
    }

    // the waves' partial tiles meet in LDS: red[unit][wave][lane]
    wait_loads<0>();
    const int64_t part = out_mode == 2 ? (int64_t)blockIdx.y * M * N : 0;
    f32x4 *red = reinterpret_cast<f32x4 *>(smem);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) red[((r * MT + mt) * kWaves + wave) * 64 + lane] = acc[r][mt];
    __syncthreads();
    for (int u = wave; u < R * MT; u += kWaves) {
        const f32x4 *src = red + u * kWaves * 64 + lane;
        f32x4 v = src[0];
#pragma unroll
        for (int k = 1; k < kWaves; ++k) {
            const f32x4 w2 = src[k * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += w2[e];
        }
        // rows 4 c + q of column j -> columns 4 (j / 4) + p of row 4 c + j % 4
        f32x4 o;
        const int jq = j & 3;
        transpose_quad(v, o, jq);
        const int row = (u % MT) * 16 + c * 4 + jq, tile = tileb + u / MT;
        if (row < rows && tile < tiles)
            store_quad(o, y, (int64_t)(m0 + row) * N + (int64_t)tile * kTileRows + (j & 12), part, out_mode, res);
    }
}

template <int MT, int R, int BITS>
hipError_t launch_cfg(const void *wt, const uint32_t *sz, int szs, int64_t K, int64_t N, const uint16_t *x, int M, void *y,
                      int out_mode, const uint16_t *res, const RowsPlan &p, hipStream_t stream) {
    using G = Geo<MT, R>;
    // once per process and kernel instantiation (thread-safe static initialisation)
    static const hipError_t attr_status = hipFuncSetAttribute(reinterpret_cast<const void *>(&w4_slices_kernel<MT, R, BITS>),
                                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::LDS);
    if (attr_status != hipSuccess) return attr_status;
    const int groups = (int)(K / kGroup), tiles = (int)(N / kTileRows);
    const dim3 grid((unsigned)((tiles + R - 1) / R), (unsigned)p.SK, (unsigned)((M + MT * 16 - 1) / (MT * 16)));
    hipLaunchKernelGGL((w4_slices_kernel<MT, R, BITS>), grid, dim3(64 * kWaves), G::LDS,
                       stream, wt, sz, x, y, M, K, N, groups, tiles, p.gps, out_mode, szs, out_mode == 2 ? nullptr : res);
    return hipGetLastError();
}

template <int MT, int BITS>
hipError_t launch_r(const void *wt, const uint32_t *sz, int szs, int64_t K, int64_t N, const uint16_t *x, int M, void *y,
                    int out_mode, const uint16_t *res, const RowsPlan &p, hipStream_t stream) {
    switch (p.R) {
        case 1: return launch_cfg<MT, 1, BITS>(wt, sz, szs, K, N, x, M, y, out_mode, res, p, stream);
        case 2: return launch_cfg<MT, 2, BITS>(wt, sz, szs, K, N, x, M, y, out_mode, res, p, stream);
        case 4: return launch_cfg<MT, 4, BITS>(wt, sz, szs, K, N, x, M, y, out_mode, res, p, stream);
    }
    return hipErrorInvalidValue;
}

template <int BITS>
hipError_t launch_slices(const void *wt, const uint32_t *sz, int szs, int64_t K, int64_t N, const uint16_t *x, int64_t M, void *y,
                         bool out_f32, const uint16_t *res, void *ws, const RowsPlan &p, hipStream_t stream) {
    const bool split = p.SK > 1;
    if (split && !ws) return hipErrorInvalidValue;
    void *dst = split ? ws : y;
    const int out_mode = split ? 2 : (out_f32 ? 0 : 1);
    const int iM = (int)M;
    hipError_t e = hipErrorInvalidValue;
    if (p.MT == 2) e = launch_r<2, BITS>(wt, sz, szs, K, N, x, iM, dst, out_mode, res, p, stream);
    if (p.MT == 3) e = launch_r<3, BITS>(wt, sz, szs, K, N, x, iM, dst, out_mode, res, p, stream);
    if (p.MT == 4) e = launch_r<4, BITS>(wt, sz, szs, K, N, x, iM, dst, out_mode, res, p, stream);
    if (e != hipSuccess || !split) return e;
    return launch_splitk_reduce(static_cast<const float *>(ws), y, M * N, p.SK, out_f32, res, stream);
}

}  // namespace

hipError_t launch_w4_slices(const LayerView &L, const uint16_t *x, int64_t M, void *y, bool out_f32, const uint16_t *res, void *ws,
                            const RowsPlan &p, hipStream_t stream) {
    return launch_slices<4>(L.wt, L.sz, L.szs, L.K, L.N, x, M, y, out_f32, res, ws, p, stream);
}

hipError_t launch_w3_slices(const LayerView3 &L, const uint16_t *x, int64_t M, void *y, bool out_f32, const uint16_t *res, void *ws,
                            const RowsPlan &p, hipStream_t stream) {
    return launch_slices<3>(L.wt, L.sz, 1, L.K, L.N, x, M, y, out_f32, res, ws, p, stream);
}

}  // namespace dmr
