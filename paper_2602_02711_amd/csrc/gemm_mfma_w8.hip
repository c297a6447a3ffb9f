// 256 x 256 tiles (or 192 or 128 rows by 256 columns) on eight wavefronts: the direct-to-LDS pipeline of the tiled GEMMs with two waves per SIMD that take
// turns at the matrix pipe.
//
// y[M][N] = x[M][K] . W[N][K]^T, bf16 operands, fp32 accumulation.  A workgroup of 8 wavefronts (2 x 4) owns a
// 256 x 256 tile, every wave a 128 x 64 patch = 4 x 2 tiles of v_mfma_f32_32x32x16_bf16: 128 accumulator registers,
// which together with the operand fragments fit the 256 registers a wave has at two waves per SIMD, so the
// accumulators stay in ordinary vector registers.  (With tiles of 192 or 128 rows a wave has 3 x 2 or 2 x 2 MFMA tiles: more
// operand traffic per MFMA, but a grid that fills its rounds better, see gemm_big_tile_rows.)  The two waves of a SIMD alternate between a multiply phase (the 16
// MFMAs of a k step, operands already in registers) and a fetch phase (the step's 12 fragment reads from LDS, the wave's
// share of the global -> LDS loads), so that one of them always has MFMAs to issue: measured 3-9 % ahead of eight waves
// that all run the same software pipeline, which in turn was 3-7 % ahead of four waves with 128 x 128 patches.
// Data movement and LDS layout: `global_load_lds_dwordx4` (every lane names its own 16 global bytes, the wave's
// 64 x 16 bytes land contiguously at a wave-uniform LDS address), four LDS stages of 32 k, rows of 64 bytes with the
// 16-byte chunks XOR-swizzled on the global side, bare barriers, loads three to four steps ahead.
#include <cstdint>
#include <type_traits>

#include "common.hpp"

namespace dmr {

namespace {

constexpr int BK = 32, NS = 4;
constexpr int ROW_BYTES = BK * 2;                          // 64
constexpr int TN = 2;                                      // MFMA tiles per wave along n
constexpr int WM = 2, WN = 4;                              // waves per workgroup
constexpr int BN = 32 * TN * WN;                           // 256
constexpr int B_BYTES = BN * ROW_BYTES;
constexpr int LB = BN / 16 / (WM * WN);                    // weight load instructions per wave and step: 2

// TM MFMA tiles per wave along m: tiles of 256, 192 or 128 rows.  A step's 4 TM activation load instructions (16 rows each)
// divide over the eight waves as LA0 each for waves 0..3 and LA1 each for waves 4..7.
template <int TM>
struct Geo {
    static constexpr int BM = 32 * TM * WM;
    static constexpr int A_BYTES = BM * ROW_BYTES, STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr size_t LDS_BYTES = (size_t)NS * STAGE_BYTES;          // 128, 112 or 96 KiB
    static constexpr int LA0 = (TM + 1) / 2, LA1 = TM - LA0;
    static constexpr int L0 = LA0 + LB, L1 = LA1 + LB;
};

typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void global_void;

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
}

__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ ((row >> 2) & 3); }

template <int TM>
__device__ __forceinline__ void load_frags(const uint8_t *__restrict__ As, const uint8_t *__restrict__ Bs, int ks,
                                           Frag (&a)[TM], Frag (&b)[TN], int lane, int wm, int wn) {
    const int chunk = ks * 2 + (lane >> 5);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int ra = wm * 32 * TM + i * 32 + (lane & 31);
        a[i].u = *reinterpret_cast<const uint4 *>(As + ra * ROW_BYTES + swz(ra, chunk) * 16);
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int rb = wn * 32 * TN + j * 32 + (lane & 31);
        b[j].u = *reinterpret_cast<const uint4 *>(Bs + rb * ROW_BYTES + swz(rb, chunk) * 16);
    }
}

template <int TM>
__device__ __forceinline__ void mfma_all(const Frag (&a)[TM], const Frag (&b)[TN], f32x16 (&acc)[TM][TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i].v, b[j].v, acc[i][j], 0, 0, 0);
}

// The two waves of a SIMD alternate roles.  Waves 0..3 (rows 0..127 of the tile) multiply step kt (16 MFMAs on fragments
// already in registers, nothing to wait for) while waves 4..7 fetch their fragments of step kt from LDS and issue their
// loads; then the roles swap.  Two barriers per k step, the same number on both paths.  A wave's fragments of a whole k
// step (both sub-steps, 48 registers) live in registers from its fetch phase to its multiply phase.
template <int TM, bool OUT_F32, bool RES>
__global__ __launch_bounds__(512) void gemm_w8_kernel(const uint16_t *__restrict__ w, const uint16_t *__restrict__ x,
                                                         typename OutPtr<RES>::type y, int64_t M, int64_t K, int64_t N, int nbm, int nbn, int lg_xm,
                                                         const uint16_t *res) {
    using G = Geo<TM>;
    constexpr int BM = G::BM, A_BYTES = G::A_BYTES, STAGE_BYTES = G::STAGE_BYTES;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const bool first = wm == 0;                      // role group: waves 0..3 multiply in the even phases
    int tm, tn;
    if (lg_xm < 0) {
        // any other grid: every XCD (linear index mod 8) takes a contiguous share of the tiles, walked in bands of four
        // tile rows, so that the 32 tiles it runs at a time still form about a 4 x 8 patch
        const int total = nbm * nbn, xcd = (int)blockIdx.x & 7, share = total >> 3, rest = total & 7;
        const int t = xcd * share + min(xcd, rest) + ((int)blockIdx.x >> 3);
        const int band = t / (4 * nbn), r = t - band * 4 * nbn;
        const int rows = min(4, nbm - band * 4);
        tm = band * 4 + r % rows;
        tn = r / rows;
    } else {
        const int region = (int)blockIdx.x >> 8, r = (int)blockIdx.x & 255;
        const int xcd = r & 7, q = r >> 3;
        const int xn = 8 >> lg_xm;
        const int regions_n = nbn / (8 * xn);
        tm = (region / regions_n) * (4 << lg_xm) + (xcd / xn) * 4 + (q >> 3);
        tn = (region % regions_n) * 8 * xn + (xcd % xn) * 8 + (q & 7);
    }
    const int64_t n0 = (int64_t)tn * BN;
    const int64_t m0 = (int64_t)tm * BM;
    const int steps = (int)(K / BK);

    const int arow0 = first ? wave * 16 * G::LA0 : 64 * G::LA0 + (wave - 4) * 16 * G::LA1;     // first activation row this wave loads
    const uint16_t *gp[G::L0];
#pragma unroll
    for (int i = 0; i < G::LA0; ++i) {                 // (where LA1 < LA0 the last pointer of the second group is not used)
        const int row = min(arow0 + i * 16, BM - 16) + (lane >> 2);
        const int64_t m = m0 + row < M ? m0 + row : M - 1;
        gp[i] = x + m * K + swz(row, lane & 3) * 8;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int row = wave * 16 * LB + i * 16 + (lane >> 2);
        const int64_t n = n0 + row < N ? n0 + row : N - 1;
        gp[G::LA0 + i] = w + n * K + swz(row, lane & 3) * 8;
    }
    int at = 0;
    auto issue = [&](auto la, int step) {                     // this wave's share of a step's loads, into stage step % 4
        uint8_t *stage = lds + (step & 3) * STAGE_BYTES;
        const int target = step < steps ? step : steps - 1;
        const int adv = (target - at) * BK;
        at = target;
#pragma unroll
        for (int i = 0; i < decltype(la)::value; ++i) {
            gp[i] += adv;
            __builtin_amdgcn_global_load_lds((global_void *)gp[i], (lds_void *)(stage + (arow0 + i * 16) * ROW_BYTES), 16, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            gp[G::LA0 + i] += adv;
            __builtin_amdgcn_global_load_lds((global_void *)gp[G::LA0 + i],
                                             (lds_void *)(stage + A_BYTES + (wave * 16 * LB + i * 16) * ROW_BYTES), 16, 0, 0);
        }
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    Frag fa[2][TM], fb[2][TN];
    auto fetch = [&](int step) {
        const uint8_t *st = lds + (step & 3) * STAGE_BYTES;
        load_frags(st, st + A_BYTES, 0, fa[0], fb[0], lane, wm, wn);
        load_frags(st, st + A_BYTES, 1, fa[1], fb[1], lane, wm, wn);
    };
    auto multiply = [&]() {        // (raising the wave's priority around this block measured 1-2 % slower)
        mfma_all(fa[0], fb[0], acc);
        mfma_all(fa[1], fb[1], acc);
    };

    // Prologue.  Every wave issues its shares of steps 0..2, the first group also of step 3 (in the loop the first group
    // issues step kt + 4 in the odd phase, the second group step kt + 3 in the even phase).
    constexpr std::integral_constant<int, G::LA0> la0{};
    constexpr std::integral_constant<int, G::LA1> la1{};
    constexpr int L0 = G::L0, L1 = G::L1;
    if (first) {
        issue(la0, 0);
        issue(la0, 1);
        issue(la0, 2);
        issue(la0, 3);
        wait_vmcnt<3 * L0>();      // step 0 landed
    } else {
        issue(la1, 0);
        issue(la1, 1);
        issue(la1, 2);
        wait_vmcnt<2 * L1>();
    }
    bare_barrier();
    if (first) fetch(0);
    wait_vmcnt<3 * L0>();          // own LDS reads done (the load count is already satisfied)
    bare_barrier();

    // Two loops, one per role group, with the same number of barriers (two per k step): a single loop with the roles
    // behind branches makes the compiler spill the accumulators at the joins.
    if (first) {
        for (int kt = 0; kt < steps; ++kt) {
            multiply();                // even phase: step kt
            __builtin_amdgcn_sched_barrier(0);
            wait_vmcnt<2 * L0>();      // shares of step kt + 1 landed (two younger shares may be in flight)
            bare_barrier();
            fetch(kt + 1);             // odd phase (past the end: the clamped stage, never used)
            __builtin_amdgcn_sched_barrier(0);
            issue(la0, kt + 4);
            __builtin_amdgcn_sched_barrier(0);
            wait_vmcnt<3 * L0>();      // own LDS reads done; no new share is needed yet
            bare_barrier();
        }
    } else {
        for (int kt = 0; kt < steps; ++kt) {
            fetch(kt);                 // even phase
            __builtin_amdgcn_sched_barrier(0);
            issue(la1, kt + 3);
            __builtin_amdgcn_sched_barrier(0);
            wait_vmcnt<2 * L1>();      // shares of step kt + 1 landed, own LDS reads done
            bare_barrier();
            multiply();                // odd phase: step kt
            __builtin_amdgcn_sched_barrier(0);
            wait_vmcnt<3 * L1>();
            bare_barrier();
        }
    }
    wait_vmcnt<0>();

#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t n = n0 + wn * 32 * TN + j * 32 + (lane & 31);
            float rv[16];
            if constexpr (RES) {      // unconditional loads, a tile's all in flight (with the branch at run time, no template
                // flag, the calls without a residual ran 5-7 % slower)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t m = min(m0 + wm * 32 * TM + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), M - 1);
                    rv[r] = bf16_bits_to_f32(res[m * N + min(n, N - 1)]);
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t m = m0 + wm * 32 * TM + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (m < M && n < N) {
                    const float v = RES ? acc[i][j][r] + rv[r] : acc[i][j][r];
                    if (OUT_F32)
                        reinterpret_cast<float *>(y)[m * N + n] = v;
                    else
                        reinterpret_cast<uint16_t *>(y)[m * N + n] = f32_to_bf16(v);
                }
            }
        }
}

template <int TM, bool OUT_F32, bool RES>
hipError_t launch_one(const uint16_t *w, const uint16_t *x, int64_t M, int64_t K, int64_t N, void *y, const uint16_t *res,
                      hipStream_t stream) {
    if (K / BK < 4) return hipErrorInvalidValue;
    static const hipError_t attr_status = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_w8_kernel<TM, OUT_F32, RES>),
                                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)Geo<TM>::LDS_BYTES);
    if (attr_status != hipSuccess) return attr_status;
    // Workgroups go to the 8 XCDs round-robin by linear index and each XCD has its own L2.  When the
    // grid of tiles divides evenly, the index is decoded so that the 32 workgroups an XCD runs at
    // a time form a compact 4 x 8 patch of tiles (12 operand panels instead of ~17) and the 8 patches of a
    // round tile a compact region; otherwise each XCD walks a contiguous share of the tiles in bands of four
    // tile rows (a padded region would leave XCDs idle).
    // Measured at (4096, 28672), M = 8192: L2 hit rate 53 % -> 79 %, time -7 %.  (Walking k in a different
    // order per tile was measured too and is slower: tiles in step share operand panels.)
    const int nbm = (int)((M + Geo<TM>::BM - 1) / Geo<TM>::BM), nbn = (int)((N + BN - 1) / BN);
    int lg_xm = 2;
    while (lg_xm >= 0 && (nbm % (4 << lg_xm) != 0 || nbn % (8 * (8 >> lg_xm)) != 0)) --lg_xm;
    hipLaunchKernelGGL((gemm_w8_kernel<TM, OUT_F32, RES>), dim3((unsigned)(nbm * nbn)), dim3(512), Geo<TM>::LDS_BYTES, stream, w, x, y, M, K, N, nbm, nbn,
                       lg_xm, res);
    return hipGetLastError();
}

}  // namespace

// Rows of the tile (256, 192 or 128; 256 columns each), or 0 where the 128 x 128 kernel with two workgroups per CU is to be
// preferred.  One workgroup of this kernel is resident per CU, so a launch runs in rounds of 256 tiles, and what a ragged
// last round wastes decides: 3000 rows x 4096 outputs are 192 tiles of 256 rows (three quarters of a round), 256 tiles of
// 192 rows (exactly one) or 768 blocks of 128 x 128 (one and a half rounds).  The time of a launch is taken as
// (full rounds) * full + (a last round filled to f: base + slope * f), the numbers in us at K = 4096.  Against all four kernels
// on five K of 1024 .. 14336, nine N of 1024 .. 28672 and 150 .. 8192 rows (774 points, weights from memory) the choice is
// 0.1 % behind the fastest on average; at five rounds and more 192 and 256 rows lie within 6 % of each other with no order that
// holds over K.
//     3000 rows, us with 256 rows or 128 x 128 only / now:  4096 -> 6144  210 / 165;  4096 -> 4096  122 / 93;  14336 -> 4096  464 / 310
// One and a half rounds of 128 x 128 blocks or less do better than that where the column blocks divide by the eight XCDs: each
// XCD then keeps to its own columns and reads the weights once, which pays while they are the larger operand (us, 128 x 128 / 128
// rows: 1400 x 4096 -> 3072 62 / 73, 700 x 4096 -> 6144 66 / 73, 600 x 8192 -> 8192 129 / 149; but 900 x 4096 -> 6000, 47 column
// blocks, 6 % behind, 4300 x 4096 -> 1024 86 / 71, and with three or four row blocks 1 .. 18 % behind); a little less of a round
// if the last row block is half empty, which the taller tiles feel less (1436 x 8192 -> 4096, 384 blocks: 7 % behind).
// Below K = 1024 (not measured) the former rule stands: 256 rows from 1.5 tiles per CU on, or for one round that is at least
// 80 % full.
int gemm_big_tile_rows(int64_t M, int64_t K, int64_t N) {
    const int forced = env_int("DMR_W8_BM", -1);
    if (forced >= 0) return forced;
    if (K < 1024) {
        const int64_t wgs = ((M + 255) / 256) * ((N + 255) / 256);
        return (wgs >= 384 || (wgs >= 208 && wgs <= 256)) ? 256 : 0;
    }
    struct Shape {
        int rows, full, base, slope;
    };
    const Shape shapes[3] = {{256, 114, 65, 49}, {192, K >= 8192 ? 93 : 90, 52, 40}, {128, 74, 40, 29}};
    // 128 x 128 blocks: 512 at a time, up to half of that one workgroup per CU
    const int64_t nbm = (M + 127) / 128, nbn = (N + 127) / 128, blocks = nbm * nbn, left = blocks % 512;
    const int64_t limit = (M - 1) % 128 < 64 ? 360 : 400;
    if (blocks <= limit && nbn % 8 == 0 && nbm >= 5 && nbm <= nbn) return 0;
    int64_t best = 82 * (blocks / 512) * 256 + (left == 0 ? 0 : left <= 256 ? 36 * 256 + 12 * left : 62 * 256 + 20 * (left - 256));
    if (nbn > 1 && ((M + 255) / 256) * ((N + 255) / 256) >= 384) best = INT64_MAX;      // 100000 x 4096 -> 384: 480, 256 rows 439
    int rows = 0;
    for (const Shape &s : shapes) {
        const int64_t tiles = ((M + s.rows - 1) / s.rows) * ((N + 255) / 256), last = tiles % 256;
        const int64_t t = s.full * (tiles / 256) * 256 + (last ? s.base * 256 + s.slope * last : 0);
        if (t < best) {
            best = t;
            rows = s.rows;
        }
    }
    return rows;
}

hipError_t launch_bf16_gemm_w8(const uint16_t *w, const uint16_t *x, int64_t M, int64_t K, int64_t N, void *y, bool out_f32,
                               const uint16_t *res, hipStream_t stream) {
    auto go = [&](auto tm) {
        constexpr int TM = decltype(tm)::value;
        if (res)
            return out_f32 ? launch_one<TM, true, true>(w, x, M, K, N, y, res, stream) : launch_one<TM, false, true>(w, x, M, K, N, y, res, stream);
        return out_f32 ? launch_one<TM, true, false>(w, x, M, K, N, y, res, stream) : launch_one<TM, false, false>(w, x, M, K, N, y, res, stream);
    };
    switch (gemm_big_tile_rows(M, K, N)) {
        case 128: return go(std::integral_constant<int, 2>{});
        case 192: return go(std::integral_constant<int, 3>{});
        default: return go(std::integral_constant<int, 4>{});
    }
}

}  // namespace dmr
