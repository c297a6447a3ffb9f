// bf16 twin for 2..64 rows: the activations stay in registers, the weights stream past them.
//
// Eight wavefronts split the K (or the split of K) of a workgroup; a wave takes the A fragments of its at most GPW groups of 128 k
// once (MT GPW 16 registers) and then walks a run of 16-row weight tiles with them.  An item is 16 rows x 256 bytes; it goes
// into the wave's own ring of NS LDS slots by buffer loads (four per item: four rows each, 256 contiguous bytes of a row,
// 16-byte pieces XOR-swizzled with the row), is read back as MFMA operands and replaced by the item NS further on: up to 128 KiB
// per CU in flight, no barrier in the stream.  The first items of the ring are the activations themselves, in the same shape.
// At the end of a tile the eight partial tiles meet in one of two LDS buffers (one barrier); MT waves add them in ascending order,
// transpose 4 x 4 within quads of lanes, add the residual (requested when the tile began) and store, the others go on.  Rows
// beyond M are copies of row M - 1; a wave without a group in a place of its sequence asks for no bytes there and skips it.
//
// What bounds it: HBM, 5.6 TB/s at 32 rows 4096 -> 28672.  Against the kernels it replaced (weights from global memory straight
// into registers, 64 bytes of a row per instruction, or through LDS with one barrier per step), us, weights from memory:
//   4096 -> 28672   8 rows 56.9 / 39.8   16 rows 46.3 / 40.5   32 rows 71.6 / 42.1   64 rows 75.7 / 52.5 (K in two)
//   14336 -> 4096   16 rows 35.8 / 25.1   32 rows 36.4 / 26.9   64 rows 39.3 / 30.0 (K in two, four, seven)
//   4096 -> 4096    8 rows 15.1 / 10.0   32 rows 18.2 / 11.6      1024 -> 4096   8 rows 6.7 / 6.3
// The activations read as fragments from global memory (64 bytes of a row per instruction) cost 3.5 us more at 32 rows.
#include <type_traits>

#include "lds_loads.hpp"
#include "mid_plan.hpp"
#include "bf16_rows_plan.hpp"
#include "wave_share.hpp"

namespace dmr {

namespace {

constexpr int kWaves = kSharingWaves;
constexpr int kItem = 4096;          // bytes of an item: 16 rows x 128 bf16

template <int MT>
struct Ring {
    static constexpr int NS = MT <= 2 ? 4 : 3;                // slots of a wave
    static constexpr int RED = kWaves * MT * 1024;
    static constexpr size_t LDS = (size_t)kWaves * NS * kItem + 2 * RED;
    static_assert(LDS <= 160 * 1024, "");
};

// out_mode: 0 = fp32 y, 1 = bf16 y, 2 = fp32 partial [split][M][N]
template <int MT, int GPW>
__global__ __launch_bounds__(64 * kWaves) void bf16_rows_kernel(const uint16_t *w, const uint16_t *x, void *y, int M, int64_t K,
                                                                int64_t N, int groups, int tiles, int gps, int tpw, int out_mode,
                                                                const uint16_t *res) {
    using L = Ring<MT>;
    constexpr int NS = L::NS;
    // Up to 16 rows a wave adds its groups up in two chains, sixteen to a workgroup as the kernels it replaced had: with one the error
    // against fp64 was larger than theirs (8 rows 4096 -> 6144 1.15e-7 of the rms, one chain 1.37e-7, two 1.07e-7), and the time is
    // the same.  Above, one chain has less error than the kernel before it (32 rows 1.37e-7 and 1.89e-7).
    constexpr int CHAINS = MT == 1 && GPW > 1 ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane >> 4, j = lane & 15;
    const WaveShare mine = wave_share(groups, gps, (int)blockIdx.y, wave);
    const int n = mine.n;
    // this workgroup's tiles: [t0, t0 + nt)
    const int t0 = (int)blockIdx.x * tpw, nt = min(tpw, tiles - t0);

    const uint32_t rowb = (uint32_t)K * 2u;
    const uint16_t *wb = w + (int64_t)t0 * kTileRows * K;
    const uint32_t wbytes = (uint32_t)nt * kTileRows * rowb;       // (the launcher checks that a run of tiles stays below 4 GiB)
    uint32_t voff[4];                 // piece p of an item: rows 4 p + c; 16-byte piece q of a row lies at q ^ row
#pragma unroll
    for (int p = 0; p < 4; ++p) voff[p] = (uint32_t)(4 * p + c) * rowb + (uint32_t)(j ^ (4 * p + c)) * 16u;
    uint8_t *ring = smem + wave * NS * kItem;
    // item i of the wave: group i % GPW of tile i / GPW
    auto request = [&](int slot, int tile, int gi) {
        const uint32_t soff = (uint32_t)min(tile, nt - 1) * kTileRows * rowb + (uint32_t)requested_group(mine, gi, groups) * 256u;
        const uint32_t bytes = tile < nt && gi < n ? wbytes : 0u;
#pragma unroll
        for (int p = 0; p < 4; ++p) stream16_to_lds(wb, bytes, ring + slot * kItem + p * 1024, voff[p], soff);
    };

    // The ring's first items are the activations, an item to a row tile and group, in the same shape.
    constexpr int NX = GPW * MT;
    const uint32_t xbytes = (uint32_t)M * rowb;
    uint32_t vlast[4];                // the last row tile: rows beyond M are copies
#pragma unroll
    for (int p = 0; p < 4; ++p)
        vlast[p] = (uint32_t)min(4 * p + c, M - 1 - 16 * (MT - 1)) * rowb + (uint32_t)(j ^ (4 * p + c)) * 16u;
    auto request_item = [&](int i) {                  // item i of the wave's whole sequence; i < NX + NS
        const int slot = i % NS;
        if (i >= NX) {
            request(slot, (i - NX) / GPW, (i - NX) % GPW);
            return;
        }
        const int gi = i / MT, mt = i % MT;
        const uint32_t soff = (uint32_t)mt * kTileRows * rowb + (uint32_t)requested_group(mine, gi, groups) * 256u, bytes = gi < n ? xbytes : 0u;
#pragma unroll
        for (int p = 0; p < 4; ++p) load16_to_lds(x, bytes, ring + slot * kItem + p * 1024, mt == MT - 1 ? vlast[p] : voff[p], soff);
    };
    const int fbase = j * 256 + ((c ^ j) * 16);       // k step t: fbase ^ (64 t)
    auto read_item = [&](int slot, Frag (&f)[4]) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint8_t *p = ring + slot * kItem + (fbase ^ (t << 6));
            read_frag(p, p, f[t]);
        }
    };
    Frag a[GPW][MT][4];
#pragma unroll
    for (int i = 0; i < NS; ++i) request_item(i);
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        wait_loads<(NS - 1) * 4>();
        read_item(i % NS, a[i / MT][i % MT]);
        wait_lds();
        __builtin_amdgcn_sched_barrier(0);
        request_item(i + NS);
    }

    // a lane's four results of a tile (waves 0..MT-1) and their residual, requested when the tile begins: behind the stream's
    // requests it would wait for all of them
    const int orow = wave * 16 + c * 4 + (j & 3);
    // (without a residual: no bytes, and no offset either)
    const uint32_t rvoff = res ? ((uint32_t)min(orow, M - 1) * (uint32_t)N + (uint32_t)(j & 12)) * 2u : 0u;
    const uint32_t rstep = res ? kTileRows * 2u : 0u, rbytes = res ? (uint32_t)M * (uint32_t)N * 2u : 0u;
    uint2 rv;
    auto reduce = [&](int tile, int buf) {            // waves 0..MT-1
        const f32x4 *src = reinterpret_cast<const f32x4 *>(smem + kWaves * NS * kItem + buf * L::RED) + wave * 64 + lane;
        f32x4 v = src[0];
#pragma unroll
        for (int k = 1; k < kWaves; ++k) {
            const f32x4 u = src[k * MT * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += u[e];
        }
        f32x4 o;
        transpose_quad(v, o, j & 3);
        if (res) add_quad(o, rv);
        if (orow < M)
            store_quad(o, y, (int64_t)orow * N + (int64_t)(t0 + tile) * kTileRows + (j & 12), out_mode == 2 ? (int64_t)blockIdx.y * M * N : 0,
                       out_mode, nullptr);
    };
    auto tile_step = [&](int tile, int buf, auto phase) {       // phase: ring slot of the tile's first item
        constexpr int P = decltype(phase)::value;
        f32x4 acc[CHAINS][MT];
#pragma unroll
        for (int ch = 0; ch < CHAINS; ++ch)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[ch][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        rv = load_pair(res, rbytes, rvoff, (uint32_t)(t0 + tile) * rstep);
#pragma unroll
        for (int gi = 0; gi < GPW; ++gi) {
            const int slot = (P + gi) % NS;
            __builtin_amdgcn_sched_barrier(0);
            wait_loads<(NS - 1) * 4>();
            Frag b[4];
            read_item(slot, b);
            wait_lds();                               // the slot is free
            __builtin_amdgcn_sched_barrier(0);
            request(slot, tile + (gi + NS) / GPW, (gi + NS) % GPW);
            if (gi < n) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        f32x4 &sum = acc[gi % CHAINS][mt];
                        sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[gi][mt][t].v, b[t].v, sum, 0, 0, 0);
                    }
            }
        }
        f32x4 *dst = reinterpret_cast<f32x4 *>(smem + kWaves * NS * kItem + buf * L::RED) + wave * MT * 64 + lane;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            f32x4 v = acc[0][mt];
            if constexpr (CHAINS > 1)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += acc[1][mt][e];
            dst[mt * 64] = v;
        }
        wait_lds();
        bare_barrier();
        if (wave < MT) reduce(tile, buf);
    };
    // the slot of a tile's first item advances by GPW % NS per tile
    constexpr int STEP = GPW % NS, START = NX % NS, CYCLE = STEP == 0 ? 1 : NS % STEP == 0 ? NS / STEP : NS;
    for (int tile = 0; tile < nt; ) {
        tile_step(tile, tile & 1, std::integral_constant<int, START>{});
        if (++tile >= nt) break;
        if constexpr (CYCLE > 1) {
            tile_step(tile, tile & 1, std::integral_constant<int, (START + STEP) % NS>{});
            if (++tile >= nt) break;
        }
        if constexpr (CYCLE > 2) {
            tile_step(tile, tile & 1, std::integral_constant<int, (START + 2 * STEP) % NS>{});
            if (++tile >= nt) break;
        }
        if constexpr (CYCLE > 3) {
            tile_step(tile, tile & 1, std::integral_constant<int, (START + 3 * STEP) % NS>{});
            if (++tile >= nt) break;
        }
    }
    wait_loads<0>();      // nothing may still be landing when the LDS is given to another workgroup
}

template <int MT, int GPW>
hipError_t launch_cfg(const uint16_t *w, const uint16_t *x, int M, int64_t K, int64_t N, void *y, int out_mode, const uint16_t *res,
                      const Bf16RowsPlan &p, hipStream_t stream) {
    // once per process and kernel instantiation (thread-safe static initialisation)
    static const hipError_t attr_status = hipFuncSetAttribute(reinterpret_cast<const void *>(&bf16_rows_kernel<MT, GPW>),
                                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)Ring<MT>::LDS);
    if (attr_status != hipSuccess) return attr_status;
    const int groups = (int)(K / kGroup), tiles = (int)(N / kTileRows);
    hipLaunchKernelGGL((bf16_rows_kernel<MT, GPW>), dim3((unsigned)((tiles + p.tpw - 1) / p.tpw), (unsigned)p.SK), dim3(64 * kWaves),
                       Ring<MT>::LDS, stream, w, x, y, M, K, N, groups, tiles, p.gps, p.tpw, out_mode, out_mode == 2 ? nullptr : res);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_bf16_rows(const uint16_t *w, const uint16_t *x, int64_t M, int64_t K, int64_t N, void *y, bool out_f32,
                            const uint16_t *res, void *ws, const Bf16RowsPlan &p, hipStream_t stream) {
    const bool split = p.SK > 1;
    if (split && !ws) return hipErrorInvalidValue;
    void *dst = split ? ws : y;
    const int out_mode = split ? 2 : (out_f32 ? 0 : 1), iM = (int)M;
    hipError_t e = hipErrorInvalidValue;
#define DMR_BF16_ROWS(MT_, GPW_) \
    if (p.MT == MT_ && p.GPW == GPW_) e = launch_cfg<MT_, GPW_>(w, x, iM, K, N, dst, out_mode, res, p, stream)
    DMR_BF16_ROWS(1, 1);
    DMR_BF16_ROWS(1, 2);
    DMR_BF16_ROWS(1, 3);
    DMR_BF16_ROWS(1, 4);
    DMR_BF16_ROWS(1, 5);
    DMR_BF16_ROWS(1, 6);
    DMR_BF16_ROWS(1, 7);
    DMR_BF16_ROWS(1, 8);
    DMR_BF16_ROWS(2, 1);
    DMR_BF16_ROWS(2, 2);
    DMR_BF16_ROWS(2, 3);
    DMR_BF16_ROWS(2, 4);
    DMR_BF16_ROWS(3, 1);
    DMR_BF16_ROWS(3, 2);
    DMR_BF16_ROWS(4, 1);
    DMR_BF16_ROWS(4, 2);
#undef DMR_BF16_ROWS
    if (e != hipSuccess || !split) return e;
    return launch_splitk_reduce(static_cast<const float *>(ws), y, M * N, p.SK, out_f32, res, stream);
}

}  // namespace dmr
