// W4A16 for up to 16 rows (per row block) where neither the rows nor a slice of them fit LDS: 2..16 rows of a K whose group
// count does not slice, 3-bit decode rows beyond the GEMV's budget, and rows too long for 32-bit offsets inside a block.
//
// The streaming layout already is MFMA B-operand order, so the weights never touch LDS: a wave loads its 1 KiB blocks
// straight into registers (nontemporal, requested four groups ahead), unpacks them with the bf16 magic number and feeds
// v_mfma_f32_16x16x32_bf16.  Only the activations go through LDS: the workgroup's 16 x 128 slice of x for the current group,
// double buffered (and requested three groups ahead into registers), rows padded to 272 bytes so that the 16-byte A-operand
// reads of 8 consecutive lanes fall in distinct banks.  A wave owns R weight tiles.  The group sums of x come from one more MFMA
// against an all-ones operand, already in accumulator layout, and a group contributes
//     acc += s (D - (128 + z) X)                                  (exact codes, fp32 scale)
// as in the decode kernels, so this path has their accuracy.
//
// K is split over blockIdx.z where the columns leave CUs idle: each split writes an fp32 partial tile to the caller's workspace
// and a second kernel adds the partials in ascending split order (deterministic, no atomics).
//
// BITS = 3 runs the same kernel on the 3-bit streaming layout (768-byte blocks, three words per lane).
#include <algorithm>

#include "mid_plan.hpp"
#include "w3_unpack.hpp"

namespace dmr {

namespace {

constexpr int ROW_BYTES = 272;   // one activation row of a group in LDS: 128 bf16 + 16 bytes of padding
constexpr int NW = 4, BM = 16;    // waves (columns) and rows of a workgroup


// out: 0 = fp32 y, 1 = bf16 y, 2 = fp32 partial [split][M][N]; kResidualInPlace
template <int R, int BITS>
__global__ __launch_bounds__(64 * NW, 2) void w4_mid_kernel(
    const void *__restrict__ wt, const uint32_t *__restrict__ sz, const uint16_t *__restrict__ x,
    void *__restrict__ y, int M, int64_t K, int64_t N, int groups, int tiles, int gps, int out, int szs,
    const uint16_t *__restrict__ res) {
    constexpr int THREADS = 64 * NW;
    constexpr int ROWS_PER_PASS = THREADS / 16;
    constexpr int XL = BM / ROWS_PER_PASS;          // 16-byte pieces of x per thread and group
    static_assert(BM % ROWS_PER_PASS == 0, "activation rows must divide over the threads");
    extern __shared__ __attribute__((aligned(16))) uint8_t xl[];   // [2][BM][ROW_BYTES]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane >> 4, j = lane & 15;
    const int m0 = (int)blockIdx.y * BM;
    const int gA = (int)blockIdx.z * gps;
    const int gB = min(groups, gA + gps);

    const int tile0 = ((int)blockIdx.x * NW + wave) * R;
    int64_t wbase[R];          // block index of (tile, group 0); ragged last column block re-reads the last tile
    int64_t sbase[R];          // its first scale / zero word (wave-uniform, like wbase)
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
        wbase[rt] = (int64_t)min(tile0 + rt, tiles - 1) * groups;
        sbase[rt] = sz_index(min(tile0 + rt, tiles - 1), 0, groups, szs, 0);
    }
    const uint32_t *szj = sz + j;
    const int sstep = szs * kTileRows;

    struct Slot {
        uint4 w[R];            // BITS == 3: .x .y .z hold the lane's three words
        uint32_t s[R];
    };
    Slot ring[4];
    auto fetch_w = [&](Slot &s, int g) {
#pragma unroll
        for (int rt = 0; rt < R; ++rt) {
            const int64_t block = wbase[rt] + g;
            if constexpr (BITS == 4) {
                s.w[rt] = load_stream(static_cast<const uint4 *>(wt) + block * 64 + lane);
            } else {
                const uint32_t *pw = static_cast<const uint32_t *>(wt) + (block * 64 + lane) * 3;
                s.w[rt].x = load_stream(pw);
                s.w[rt].y = load_stream(pw + 1);
                s.w[rt].z = load_stream(pw + 2);
            }
            s.s[rt] = szj[sbase[rt] + (int64_t)g * sstep];
        }
    };

    // activations: thread -> (row, 16-byte piece) of the BM x 128 slice.  Rows beyond M wrap around to
    // rows m mod M: MFMA rows are independent and those outputs are never stored, so no zero fill
    // (whose per-lane select would make the loads conditional) is needed.
    u32x4_t xr[2][XL];     // two groups in flight (a plain vector type: the array has to stay in registers)
    const int xrow = tid >> 4, xpiece = tid & 15;
    const uint16_t *xsrc[XL];
#pragma unroll
    for (int p = 0; p < XL; ++p) {
        const int m = m0 + p * ROWS_PER_PASS + xrow;
        xsrc[p] = x + (int64_t)(m < M ? m : m % M) * K + xpiece * 8;
    }
    auto fetch_x = [&](int set, int g) {
#pragma unroll
        for (int p = 0; p < XL; ++p)
            xr[set][p] = *reinterpret_cast<const u32x4_t *>(xsrc[p] + (int64_t)g * kGroup);
    };
    auto put_x = [&](int set, int buf) {
        uint8_t *dst = xl + buf * (BM * ROW_BYTES);
#pragma unroll
        for (int p = 0; p < XL; ++p)
            *reinterpret_cast<u32x4_t *>(dst + (p * ROWS_PER_PASS + xrow) * ROW_BYTES + xpiece * 16) = xr[set][p];
    };

    f32x4 acc[R];
#pragma unroll
    for (int rt = 0; rt < R; ++rt) acc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};

    Frag ones;
    ones.w[0] = ones.w[1] = ones.w[2] = ones.w[3] = 0x3F803F80u;

    auto compute = [&](const Slot &s, int buf, bool valid) {
        const uint8_t *src = xl + buf * (BM * ROW_BYTES) + j * ROW_BYTES + c * 64;
        f32x4 d[R], xs = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int rt = 0; rt < R; ++rt) d[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            Frag a;
            a.u = *reinterpret_cast<const uint4 *>(src + t * 16);
            xs = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, ones.v, xs, 0, 0, 0);
#pragma unroll
            for (int rt = 0; rt < R; ++rt) {
                Frag b;
                if constexpr (BITS == 4) {
                    const uint32_t word = t == 0 ? s.w[rt].x : t == 1 ? s.w[rt].y : t == 2 ? s.w[rt].z : s.w[rt].w;
                    unpack_word(word, b.w);
                } else {
                    if (t == 0) unpack3_step<0>(s.w[rt].x, s.w[rt].y, s.w[rt].z, b.w);
                    if (t == 1) unpack3_step<1>(s.w[rt].x, s.w[rt].y, s.w[rt].z, b.w);
                    if (t == 2) unpack3_step<2>(s.w[rt].x, s.w[rt].y, s.w[rt].z, b.w);
                    if (t == 3) unpack3_step<3>(s.w[rt].x, s.w[rt].y, s.w[rt].z, b.w);
                }
                d[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, d[rt], 0, 0, 0);
            }
        }
#pragma unroll
        for (int rt = 0; rt < R; ++rt) {
            // a slot past the end of this split's k range re-reads its last group with scale 0
            const float sc = valid ? __uint_as_float(s.s[rt] << 16) : 0.f;
            const float cz = __uint_as_float(s.s[rt] & 0xFFFF0000u);   // -(128 + z)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[rt][q] = fmaf(sc, fmaf(cz, xs[q], d[rt][q]), acc[rt][q]);
        }
    };

    // Software pipeline, one group of 128 k per phase: the weights of a phase were requested four
    // phases earlier, its activations three phases earlier into registers and written to the other
    // LDS buffer one phase earlier.  Phases come in fours (static register indices); a phase past the
    // end of this split's k range re-reads the last group with scale 0, so that every wave passes the
    // same barriers and every load is unconditional.  (Walking the groups in a different order per
    // workgroup was measured and is slower: workgroups in step share the activations in cache.)
    const int last = gB - 1;
    fetch_x(0, gA);          // ahead of the weights: a wave's loads return in order, and this one is needed first
#pragma unroll
    for (int u = 0; u < 4; ++u) fetch_w(ring[u], min(gA + u, last));
    put_x(0, 0);
    fetch_x(1, min(gA + 1, last));
    fetch_x(0, min(gA + 2, last));
    __syncthreads();
    for (int g = gA; g < gB; g += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            compute(ring[u], u & 1, g + u < gB);
            fetch_w(ring[u], min(g + u + 4, last));
            put_x((u + 1) & 1, (u + 1) & 1);                 // group g + u + 1
            fetch_x((u + 1) & 1, min(g + u + 3, last));
            __syncthreads();
        }
    }

    const int out_mode = out & 3;
    const uint16_t *from = residual_source(y, res, out);
    if (from && out_mode != 2) {      // clamped, unconditional loads: all of them in flight at once
#pragma unroll
        for (int rt = 0; rt < R; ++rt)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int m = min(m0 + c * 4 + q, M - 1);
                acc[rt][q] += bf16_bits_to_f32(from[(int64_t)m * N + (int64_t)min(tile0 + rt, tiles - 1) * kTileRows + j]);
            }
    }
    const int64_t part = out_mode == 2 ? (int64_t)blockIdx.z * M * N : 0;
#pragma unroll
    for (int rt = 0; rt < R; ++rt) {
        const int tile = tile0 + rt;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int m = m0 + c * 4 + q;
            if (m < M && tile < tiles) {
                const int64_t o = (int64_t)m * N + (int64_t)tile * kTileRows + j;
                if (out_mode == 1)
                    reinterpret_cast<uint16_t *>(y)[o] = f32_to_bf16(acc[rt][q]);
                else
                    reinterpret_cast<float *>(y)[part + o] = acc[rt][q];
            }
        }
    }
}

// y = sum over splits of part[split], four outputs per thread, splits in ascending order; an optional residual is added
// to the fp32 sum (a launch of its own for it cost 2-4 us and two more passes over M x N fp32).  A launch is short and waits for
// memory: with the number of splits known (SK; 0: any) a thread has all its loads under way at once, where a loop waited for each
// in turn.  us in a chain of launches, loop / this: 8 x 4096 of 4
// splits 2.63 / 2.46, of 8 3.12 / 2.57, 64 x 4096 of 7 3.17 / 2.74, 200 x 4096 of 4 level; six layers of 64 rows 412 / 398.
template <int SK>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float *__restrict__ part, void *y,
                                                            int64_t total, int splits, int out_f32,
                                                            const uint16_t *res) {
    const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i >= total) return;
    // (without a residual any address: behind a branch the load would be waited for at once)
    const uint2 r = *reinterpret_cast<const uint2 *>((res ? res : reinterpret_cast<const uint16_t *>(part)) + i);
    f32x4 v;
    if constexpr (SK > 0) {
        f32x4 u[SK];
#pragma unroll
        for (int s = 0; s < SK; ++s) u[s] = *reinterpret_cast<const f32x4 *>(part + (int64_t)s * total + i);
        v = u[0];
#pragma unroll
        for (int s = 1; s < SK; ++s)
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] += u[s][k];
    } else {
        v = *reinterpret_cast<const f32x4 *>(part + i);
        for (int s0 = 1; s0 < splits; s0 += 4) {
            f32x4 u[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) u[s] = *reinterpret_cast<const f32x4 *>(part + (int64_t)min(s0 + s, splits - 1) * total + i);
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (s0 + s < splits)
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] += u[s][k];
        }
    }
    if (res) {
        v[0] += __uint_as_float(r.x << 16);
        v[1] += __uint_as_float(r.x & 0xFFFF0000u);
        v[2] += __uint_as_float(r.y << 16);
        v[3] += __uint_as_float(r.y & 0xFFFF0000u);
    }
    if (out_f32) {
        *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(y) + i) = v;
    } else {
        uint2 o;
        o.x = pack_bf16x2(v[0], v[1]);
        o.y = pack_bf16x2(v[2], v[3]);
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(y) + i) = o;
    }
}

template <int R, int BITS>
hipError_t launch_cfg(const void *wt, const uint32_t *sz, int szs, int64_t K, int64_t N, const uint16_t *x, int M, void *dst,
                      int out_mode, const uint16_t *res, const MidPlan &p, hipStream_t stream) {
    constexpr size_t lds = 2ull * BM * ROW_BYTES;
    // once per process and kernel instantiation (thread-safe static initialisation)
    static const hipError_t attr_status = hipFuncSetAttribute(
        reinterpret_cast<const void *>(&w4_mid_kernel<R, BITS>), hipFuncAttributeMaxDynamicSharedMemorySize,
        (int)lds);
    if (attr_status != hipSuccess) return attr_status;
    const int groups = (int)(K / kGroup), tiles = (int)(N / kTileRows);
    const dim3 grid((unsigned)((tiles + NW * R - 1) / (NW * R)), (unsigned)((M + BM - 1) / BM), (unsigned)p.SK);
    hipLaunchKernelGGL((w4_mid_kernel<R, BITS>), grid, dim3(64 * NW), lds, stream, wt, sz, x, dst, M,
                       K, N, groups, tiles, p.gps, out_mode, szs, res);
    return hipGetLastError();
}

template <int BITS>
hipError_t launch_r(const void *wt, const uint32_t *sz, int szs, int64_t K, int64_t N, const uint16_t *x, int M, void *dst,
                    int out_mode, const uint16_t *res, const MidPlan &p, hipStream_t stream) {
    return p.R == 2 ? launch_cfg<2, BITS>(wt, sz, szs, K, N, x, M, dst, out_mode, res, p, stream)
                    : launch_cfg<1, BITS>(wt, sz, szs, K, N, x, M, dst, out_mode, res, p, stream);
}

template <int BITS>
hipError_t launch_mid(const void *wt, const uint32_t *sz, int szs, int64_t K, int64_t N, const uint16_t *x, int64_t M, void *y,
                      bool out_f32, const uint16_t *res, void *ws, hipStream_t stream) {
    const MidPlan p = plan_mid(M, K, N);
    const bool split = p.SK > 1;
    if (split && !ws) return hipErrorInvalidValue;
    void *dst = split ? ws : y;
    const int out_mode = split ? 2 : (out_f32 ? 0 : 1) | residual_in_place(y, res);
    const hipError_t e = launch_r<BITS>(wt, sz, szs, K, N, x, (int)M, dst, out_mode, res, p, stream);
    if (e != hipSuccess || !split) return e;
    return launch_splitk_reduce(static_cast<const float *>(ws), y, M * N, p.SK, out_f32, res, stream);
}

}  // namespace

hipError_t launch_splitk_reduce(const float *part, void *y, int64_t total, int splits, bool out_f32, const uint16_t *res,
                                hipStream_t stream) {
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((total / 4 + 255) / 256)), dim3(256), 0, stream, part, y, total, splits,
                           out_f32 ? 1 : 0, res);
    };
    switch (splits) {
        case 2: go(&splitk_reduce_kernel<2>); break;
        case 3: go(&splitk_reduce_kernel<3>); break;
        case 4: go(&splitk_reduce_kernel<4>); break;
        case 5: go(&splitk_reduce_kernel<5>); break;
        case 6: go(&splitk_reduce_kernel<6>); break;
        case 7: go(&splitk_reduce_kernel<7>); break;
        case 8: go(&splitk_reduce_kernel<8>); break;
        default: go(&splitk_reduce_kernel<0>);
    }
    return hipGetLastError();
}

hipError_t launch_w4_mid(const LayerView &L, const uint16_t *x, int64_t M, void *y, bool out_f32, const uint16_t *res,
                         void *ws, hipStream_t stream) {
    return launch_mid<4>(L.wt, L.sz, L.szs, L.K, L.N, x, M, y, out_f32, res, ws, stream);
}

hipError_t launch_w3_mid(const LayerView3 &L, const uint16_t *x, int64_t M, void *y, bool out_f32, const uint16_t *res,
                         void *ws, hipStream_t stream) {
    return launch_mid<3>(L.wt, L.sz, 1, L.K, L.N, x, M, y, out_f32, res, ws, stream);
}

}  // namespace dmr
