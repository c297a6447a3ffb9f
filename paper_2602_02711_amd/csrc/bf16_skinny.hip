// Weight-streaming bf16 kernel for up to 16 rows: the high-precision twin of the W4A16 decode path.
// Same work split as the INT4 kernel (one workgroup per 16 weight rows, S wavefronts along k,
// deterministic LDS reduction); the B operand of each 16x16x32 MFMA is loaded straight from the
// row-major bf16 weight matrix: lane l = 16 c + j reads W[16 T + j][k0 + 32 t + 8 c .. + 7].
#include "common.hpp"

namespace dmr {

namespace {

constexpr int kMaxWaves = 16;

struct StepRegs {
    Frag b[4], a[4];
};

__device__ __forceinline__ void load_step(StepRegs &r, const uint16_t *__restrict__ wrow, const uint16_t *__restrict__ x, int lane,
                                          int64_t M, int64_t K, int64_t k0) {
    const int c = lane >> 4, j = lane & 15;
#pragma unroll
    for (int t = 0; t < 4; ++t)
        r.b[t].u = *reinterpret_cast<const uint4 *>(wrow + k0 + t * 32 + c * 8);
    if (j < M) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
            r.a[t].u = *reinterpret_cast<const uint4 *>(x + j * K + k0 + t * 32 + c * 8);
    } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) r.a[t].u = make_uint4(0, 0, 0, 0);
    }
}

template <bool OUT_F32>
__global__ __launch_bounds__(kMaxWaves * 64) void bf16_skinny_kernel(
    const uint16_t *__restrict__ w, const uint16_t *__restrict__ x, void *y, int64_t M,
    int64_t K, int64_t N, const uint16_t *res) {
    extern __shared__ float red[];   // [S][4][64]
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int S = blockDim.x >> 6;
    const int64_t T = blockIdx.x;
    const int steps = (int)(K / 128);
    const int s0 = (int)(((int64_t)steps * wave) / S);
    const int s1 = (int)(((int64_t)steps * (wave + 1)) / S);
    const uint16_t *wrow = w + (T * kTileRows + (lane & 15)) * K;

    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int U = 2;
    int st = s0;
    for (; st + U <= s1; st += U) {
        StepRegs regs[U];
#pragma unroll
        for (int u = 0; u < U; ++u) load_step(regs[u], wrow, x, lane, M, K, (int64_t)(st + u) * 128);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(regs[u].a[t].v, regs[u].b[t].v, acc, 0, 0, 0);
    }
    for (; st < s1; ++st) {
        StepRegs regs;
        load_step(regs, wrow, x, lane, M, K, (int64_t)st * 128);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(regs.a[t].v, regs.b[t].v, acc, 0, 0, 0);
    }

#pragma unroll
    for (int q = 0; q < 4; ++q) red[(wave * 4 + q) * 64 + lane] = acc[q];
    __syncthreads();

    for (int e = threadIdx.x; e < 4 * 64; e += blockDim.x) {
        float sum = 0.f;
        for (int s = 0; s < S; ++s) sum += red[s * (4 * 64) + e];
        const int l = e & 63, q = e >> 6;
        const int64_t m = (l >> 4) * 4 + q;
        const int64_t n = T * kTileRows + (l & 15);
        if (m < M) {
            sum = plus_residual(sum, res, m * N + n);
            if (OUT_F32)
                reinterpret_cast<float *>(y)[m * N + n] = sum;
            else
                reinterpret_cast<uint16_t *>(y)[m * N + n] = f32_to_bf16(sum);
        }
    }
}

int pick_waves(int64_t tiles, int steps) {
    int s = 1;
    while (s < kMaxWaves && tiles * s < 4096 && s * 2 <= steps) s *= 2;
    return s;
}

}  // namespace

hipError_t launch_bf16_skinny(const uint16_t *w, const uint16_t *x, int64_t M, int64_t K, int64_t N,
                              void *y, bool out_f32, const uint16_t *res, hipStream_t stream) {
    if (M > 16) return hipErrorInvalidValue;
    const int64_t tiles = N / kTileRows;
    const int S = pick_waves(tiles, (int)(K / 128));
    const size_t lds = (size_t)S * 4 * 64 * sizeof(float);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(S * 64), lds, stream, w, x, y, M, K, N, res);
    };
    if (out_f32) go(&bf16_skinny_kernel<true>);
    else go(&bf16_skinny_kernel<false>);
    return hipGetLastError();
}

}  // namespace dmr
