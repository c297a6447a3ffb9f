// One-off, integer-mostly kernels around the streaming layout: re-tile at create time,
// dequantize (the parity anchor of the layout), and the round-to-nearest quantiser that
// produces canonical inputs on the device.
#include "convert.hpp"

namespace dmr {

// ---- re-tile: canonical [N][K/8] words + [N][K/128] scales/zeros -> streaming blocks ----------
// One thread per 16-byte lane slot (T, G, l): its four words are canonical words 16G+4c..+3 of
// row 16T+j, which are contiguous, so the read and the write are both one 128-bit access.
__global__ __launch_bounds__(256) void retile_kernel(int64_t K, int64_t N,
                                                     const uint32_t *__restrict__ qweight,
                                                     const uint16_t *__restrict__ scales,
                                                     const uint16_t *__restrict__ zeros,
                                                     uint4 *__restrict__ wt,
                                                     uint32_t *__restrict__ sz, int per_channel) {
    const int64_t groups = K / kGroup;
    const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t slots = N * K / 32;
    if (slot >= slots) return;
    const int l = (int)(slot & 63);
    const auto [T, G] = block_pos(slot >> 6, groups);
    const int c = l >> 4, j = l & 15;
    const int64_t n = T * kTileRows + j;
    const uint4 src = *reinterpret_cast<const uint4 *>(qweight + n * (K / 8) + G * 16 + c * 4);
    const uint32_t in[4] = {src.x, src.y, src.z, src.w};
    uint32_t out[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        uint32_t w = 0;
#pragma unroll
        for (int p = 0; p < 8; ++p)
            w |= ((in[t] >> (4 * p)) & 0xFu) << (4 * nibble_of_position(p));
        out[t] = w;
    }
    wt[slot] = make_uint4(out[0], out[1], out[2], out[3]);
    if (c == 0 && (!per_channel || G == 0)) {
        // per-channel symmetric layers carry one scale per row and the fixed zero point 8: one word per row
        const uint32_t s_bits = per_channel ? scales[n] : scales[n * groups + G];
        const float z = per_channel ? 8.0f : bf16_bits_to_f32(zeros[n * groups + G]);
        const uint32_t cz_bits = __float_as_uint(-(128.0f + z)) >> 16;   // exact in bf16
        sz[sz_index(T, G, groups, per_channel ? 0 : 1, j)] = s_bits | (cz_bits << 16);
    }
}

hipError_t launch_retile(int64_t K, int64_t N, const uint32_t *qweight, const uint16_t *scales,
                         const uint16_t *zeros, uint4 *wt, uint32_t *sz, bool per_channel,
                         hipStream_t stream) {
    const int64_t slots = N * K / 32;
    const unsigned blocks = (unsigned)((slots + 255) / 256);
    hipLaunchKernelGGL(retile_kernel, dim3(blocks), dim3(256), 0, stream, K, N, qweight, scales, zeros,
                       wt, sz, per_channel ? 1 : 0);
    return hipGetLastError();
}

// ---- dequantize: streaming blocks -> bf16 [N][K] = RNE_bf16((q - z) * s) ----------------------
__global__ __launch_bounds__(256) void dequantize_kernel(int64_t K, int64_t N,
                                                         const uint4 *__restrict__ wt,
                                                         const uint32_t *__restrict__ sz,
                                                         uint16_t *__restrict__ w_bf16, int szs) {
    __shared__ __attribute__((aligned(16))) uint32_t turn[4][kTurnWords];
    const int64_t groups = K / kGroup;
    const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = slot < N * K / 32;         // whole wavefronts: a block is 64 slots
    const auto [T, G] = block_pos(live ? slot >> 6 : 0, groups);
    const uint4 src = live ? wt[slot] : make_uint4(0, 0, 0, 0);
    const uint32_t szw = sz[sz_index(T, G, groups, szs, (int)(slot & 15))];
    store_dequantized<true>(turn[threadIdx.x >> 6], src, szw, live, T, G, K, w_bf16);
}

hipError_t launch_dequantize(const LayerView &L, uint16_t *w_bf16, hipStream_t stream) {
    const int64_t slots = L.N * L.K / 32;
    const unsigned blocks = (unsigned)((slots + 255) / 256);
    hipLaunchKernelGGL(dequantize_kernel, dim3(blocks), dim3(256), 0, stream, L.K, L.N, L.wt, L.sz,
                       w_bf16, L.szs);
    return hipGetLastError();
}

// ---- quantise: fp32 [N][K] -> canonical codes, scales, zero points (round to nearest) --------
// 16 consecutive lanes share one group of 128 weights (8 each): range over the 16 lanes, then every lane derives the
// same scale and zero point and packs its own word.
__global__ __launch_bounds__(256) void quantize_kernel(int64_t K, int64_t N,
                                                       const float *__restrict__ w,
                                                       uint32_t *__restrict__ qweight,
                                                       uint16_t *__restrict__ scales,
                                                       uint16_t *__restrict__ zeros) {
    const int64_t word = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // canonical word index
    const bool live = word < N * K / 8;
    float v[8];
    float lo = 0.0f, hi = 0.0f;
    if (live) {
        load_weights(w + word * 8, v);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            lo = fminf(lo, v[i]);
            hi = fmaxf(hi, v[i]);
        }
    }
    row16_range(lo, hi);
    if (!live) return;
    const float s32 = (float)(((double)hi - (double)lo) / 15.0);
    uint32_t s_bits = f32_to_bf16(s32);
    if ((s_bits & 0x7FFFu) == 0) s_bits = 0x3F80u;
    float z;
    const uint32_t packed = quantize_codes<15, 4>(v, bf16_bits_to_f32(s_bits), lo, z);
    qweight[word] = packed;
    if ((word & 15) == 0) {
        const int64_t group = word >> 4;     // (n, G) flattened: rows hold K/128 groups each
        scales[group] = (uint16_t)s_bits;
        zeros[group] = f32_to_bf16(z);
    }
}

hipError_t launch_quantize(int64_t K, int64_t N, const float *w, uint32_t *qweight, uint16_t *scales,
                           uint16_t *zeros, hipStream_t stream) {
    const int64_t words = N * K / 8;
    const unsigned blocks = (unsigned)((words + 255) / 256);
    hipLaunchKernelGGL(quantize_kernel, dim3(blocks), dim3(256), 0, stream, K, N, w, qweight, scales,
                       zeros);
    return hipGetLastError();
}

}  // namespace dmr
