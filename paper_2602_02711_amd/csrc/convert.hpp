// Device pieces shared by the 4-bit and 3-bit conversion kernels: code rounding, group ranges, and the store of one
// dequantised weight block.
#pragma once
#include "common.hpp"

namespace dmr {

// (row tile, group) of a weight block.  A layer that fits memory has fewer than 2^32 blocks of 384 or more bytes, so the
// division is one of 32 bits (one of 64 bits is a loop's worth of VALU instructions per thread).
struct BlockPos {
    int64_t T, G;
};
__device__ __forceinline__ BlockPos block_pos(int64_t block, int64_t groups) {
    const uint32_t b = (uint32_t)block, g = (uint32_t)groups, t = b / g;
    return {(int64_t)t, (int64_t)(b - t * g)};
}

// Eight consecutive fp32 weights, read once: past the caches, which the codes that the re-tiling reads next can then keep
// (28672 x 4096 and three narrower layers, 4 bits: quantise 54.4 -> 49.9, re-tile 13.1 -> 12.2 us on average).
__device__ __forceinline__ void load_weights(const float *__restrict__ w, float (&v)[8]) {
    const uint4 a = load_stream(reinterpret_cast<const uint4 *>(w)), b = load_stream(reinterpret_cast<const uint4 *>(w + 4));
    const uint32_t bits[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = __uint_as_float(bits[i]);
}

// Minimum / maximum over each aligned group of 16 lanes, in every lane: four rotations on the VALU, no LDS round trip.
__device__ __forceinline__ void row16_range(float &lo, float &hi) {
    lo = fminf(lo, dpp_move<0x128>(lo)); hi = fmaxf(hi, dpp_move<0x128>(hi));
    lo = fminf(lo, dpp_move<0x124>(lo)); hi = fmaxf(hi, dpp_move<0x124>(hi));
    lo = fminf(lo, dpp_move<0x122>(lo)); hi = fmaxf(hi, dpp_move<0x122>(hi));
    lo = fminf(lo, dpp_move<0x121>(lo)); hi = fmaxf(hi, dpp_move<0x121>(hi));
}

// 1 / s for rounded_quotient, or NaN where s or its reciprocal could leave the normal range (then nothing it says is used).
__device__ __forceinline__ float quotient_rcp(float s) {
    return s > 0x1p-100f && s < 0x1p100f ? __builtin_amdgcn_rcpf(s) : __uint_as_float(0x7FC00000u);
}

// rint(v / s) from v * (1 / s).  The product is off by at most 2^-22 of itself (one ulp of the reciprocal, half an ulp of the
// product), less than 2^-18 below 16, so it rounds as the quotient does unless it lies within 2^-16 of a tie: `sure` is
// cleared there, and for |v / s| >= 16, infinities and NaN, and the caller divides in 64 bits.
__device__ __forceinline__ float rounded_quotient(float v, float rcp, bool &sure) {
    const float q = v * rcp, r = rintf(q);
    sure = sure && fabsf(q) < 16.0f && fabsf(fabsf(q - r) - 0.5f) > 0x1p-16f;
    return r;
}

// Codes of eight weights against bf16 scale s and zero point z of their group, `bits` apart in the result: clamp(rint(v / s)
// + z, 0, top), the quotient as 64 bits have it; z is rint(-lo / s) clamped the same way.  Eight 64-bit divisions a thread
// kept the quantiser off memory speed; now about one wave in 60 divides so.  28672 x 4096 weights, 4 bits: 128 -> 108 us.
template <int TOP, int BITS>
__device__ __forceinline__ uint32_t quantize_codes(const float (&v)[8], float s, float lo, float &z_out) {
    const float rcp = quotient_rcp(s);
    bool sure = true;
    float z = rounded_quotient(-lo, rcp, sure);
    z = z > 0.0f ? fminf(z, (float)TOP) : 0.0f;        // code 0 is +0 also when -lo / s is -0
    uint32_t packed = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float c = fminf(fmaxf(rounded_quotient(v[i], rcp, sure) + z, 0.0f), (float)TOP);
        packed |= (uint32_t)(int)c << (BITS * i);
    }
    if (!sure) {
        const double sd = (double)s;
        double zd = rint(-(double)lo / sd);
        zd = (zd > 0.0) ? fmin(zd, (double)TOP) : 0.0;
        z = (float)zd;
        packed = 0;
#pragma unroll 1
        for (int i = 0; i < 8; ++i) {
            float x = v[0];
#pragma unroll
            for (int k = 1; k < 8; ++k) x = i == k ? v[k] : x;
            const double c = fmin(fmax(rint((double)x / sd) + zd, 0.0), (double)TOP);
            packed |= (uint32_t)(int)c << (BITS * i);
        }
    }
    z_out = z;
    return packed;
}

// Dequantised store of one block by one wavefront: lane 16 c + j brings its 32 codes as four words of eight nibbles
// (position p of a word in nibble SHUFFLED ? nibble_of_position(p) : p) and its row's scale word.  Through LDS the wave turns
// them so that 16 lanes store the 256 contiguous bytes of a row; straight from the lane each store instruction was 64
// pieces of 16 bytes, 64 bytes apart (28672 x 4096 weights, 4 bits: 83 -> 50 us, 5.9 TB/s of codes and bf16).  Rows of 64
// words are padded by 16: the four c of a read then use different banks.
// The stores go past the caches too: 24.5 -> 21.2 us on average over four layers, 5.8 -> 6.6 TB/s on the largest.
// Every thread of the workgroup calls this (it synchronises); `live` is uniform over the wave.
constexpr int kTurnWords = 3 * 80 + 64;
template <bool SHUFFLED>
__device__ __forceinline__ void store_dequantized(uint32_t *turn, uint4 words, uint32_t szw, bool live, int64_t T, int64_t G,
                                                  int64_t K, uint16_t *__restrict__ w_bf16) {
    const int l = threadIdx.x & 63;
    *reinterpret_cast<uint4 *>(turn + 80 * (l >> 4) + 4 * (l & 15)) = words;
    __syncthreads();
    if (!live) return;
    const int u = l & 15;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int j = 4 * r + (l >> 4);
        const uint32_t in = turn[80 * (u >> 2) + 4 * j + (u & 3)];
        const uint32_t sw = __shfl(szw, j, 64);
        const float s = bf16_bits_to_f32(sw & 0xFFFFu);
        const float z = -bf16_bits_to_f32(sw >> 16) - 128.0f;
        uint32_t o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n0 = SHUFFLED ? nibble_of_position(2 * i) : 2 * i;
            const int n1 = SHUFFLED ? nibble_of_position(2 * i + 1) : 2 * i + 1;
            // (q - z) * s: a 5-bit integer times an 8-bit significand, exact in fp32
            const float lo = ((float)((in >> (4 * n0)) & 0xFu) - z) * s;
            const float hi = ((float)((in >> (4 * n1)) & 0xFu) - z) * s;
            o[i] = pack_bf16x2(lo, hi);
        }
        const u32x4_t ov = {o[0], o[1], o[2], o[3]};
        __builtin_nontemporal_store(ov, reinterpret_cast<u32x4_t *>(w_bf16 + (T * kTileRows + j) * K + G * kGroup) + u);
    }
}

}  // namespace dmr
