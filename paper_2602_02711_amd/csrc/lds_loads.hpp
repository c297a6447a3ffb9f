// Loads through buffer resources, shared by the W4 / W3 kernels that stage activations straight into LDS: a lane's part of an
// address is 32 bits and rarely changes, the rest is scalar, and nothing is read beyond `bytes`.  (The plain
// global_load_lds form is taken for a flat access by the compiler's wait-count pass, which then waits for every load in
// flight, the weights requested ahead included, whenever one result is needed.)
#pragma once
#include "common.hpp"

namespace dmr {

typedef __attribute__((address_space(3))) void lds_void;

template <int N>
__device__ __forceinline__ void wait_loads() {      // until at most N vector loads of the wave are in flight
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4)); }

// 16 or 4 bytes per lane from base + voff + soff, lane after lane to `dst`.
__device__ __forceinline__ void load16_to_lds(const void *base, uint32_t bytes, uint8_t *dst, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000),
                                             (lds_void *)dst, 16, (int)voff, (int)soff, 0, 0);
}
// The same past the caches, for weights that are read once.
__device__ __forceinline__ void stream16_to_lds(const void *base, uint32_t bytes, uint8_t *dst, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000),
                                             (lds_void *)dst, 16, (int)voff, (int)soff, 0, 2);
}
__device__ __forceinline__ void load4_to_lds(const void *base, uint32_t bytes, uint8_t *dst, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000),
                                             (lds_void *)dst, 4, (int)voff, (int)soff, 0, 0);
}

// A lane's codes of one group (16 bytes, 3-bit layout 12), past the caches like every weight that is read once.
template <int BITS>
__device__ __forceinline__ u32x4_t load_codes(const void *base, uint32_t bytes, uint32_t voff, uint32_t soff) {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
    if constexpr (BITS == 4) {
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)voff, (int)soff, 2);
    } else {
        const auto v = __builtin_amdgcn_raw_buffer_load_b96(rsrc, (int)voff, (int)soff, 2);
        return u32x4_t{v[0], v[1], v[2], 0u};
    }
}
__device__ __forceinline__ uint32_t load_word(const void *base, uint32_t bytes, uint32_t voff, uint32_t soff) {
    return __builtin_amdgcn_raw_buffer_load_b32(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000),
                                                (int)voff, (int)soff, 0);
}
__device__ __forceinline__ uint2 load_pair(const void *base, uint32_t bytes, uint32_t voff, uint32_t soff) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000),
                                                        (int)voff, (int)soff, 0);
    return make_uint2(v[0], v[1]);
}

// MFMA A operands of MT row tiles, STRIDE bytes apart in LDS.  Restrict pointers: their alias scopes keep the wait-count pass
// from tying the reads to the loads into LDS in flight, whose completion the kernels wait for explicitly.  (A scope only
// appears for a restrict parameter that has another one to be distinct from, and only survives on a load of a vector type.)
template <int MT, int STRIDE>
__device__ __forceinline__ void read_frags(const uint8_t *__restrict__ p, const uint8_t *__restrict__ q, Frag (&a)[MT]) {
    static_assert(MT >= 2, "half of the tiles through each pointer");
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const u32x4_t v = *reinterpret_cast<const u32x4_t *>((i & 1 ? q : p) + i * STRIDE);
        a[i].u = make_uint4(v[0], v[1], v[2], v[3]);
    }
}
__device__ __forceinline__ void read_frag(const uint8_t *__restrict__ p, const uint8_t *__restrict__ q, Frag &a) {
    typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
    const u32x2_t lo = *reinterpret_cast<const u32x2_t *>(p);
    const u32x2_t hi = *reinterpret_cast<const u32x2_t *>(q + 8);
    a.u = make_uint4(lo[0], lo[1], hi[0], hi[1]);
}
__device__ __forceinline__ uint32_t read_word(const uint8_t *__restrict__ p, const uint8_t *__restrict__ q) {
    const uint32_t lo = *reinterpret_cast<const uint16_t *>(p);
    const uint32_t hi = *reinterpret_cast<const uint16_t *>(q + 2);
    return lo | (hi << 16);
}

// 4 x 4 transpose within the quads of lanes: v[q] of lane jq = 0..3 holds element (q, jq); o[p] becomes element (jq, p).
__device__ __forceinline__ void transpose_quad(const f32x4 &v, f32x4 &o, int jq) {
    auto pick = [&](float e0, float e1, float e2, float e3) {
        const float lo = jq & 1 ? e1 : e0, hi = jq & 1 ? e3 : e2;
        return jq & 2 ? hi : lo;
    };
    o[0] = pick(dpp_move<0x00>(v[0]), dpp_move<0x00>(v[1]), dpp_move<0x00>(v[2]), dpp_move<0x00>(v[3]));
    o[1] = pick(dpp_move<0x55>(v[0]), dpp_move<0x55>(v[1]), dpp_move<0x55>(v[2]), dpp_move<0x55>(v[3]));
    o[2] = pick(dpp_move<0xAA>(v[0]), dpp_move<0xAA>(v[1]), dpp_move<0xAA>(v[2]), dpp_move<0xAA>(v[3]));
    o[3] = pick(dpp_move<0xFF>(v[0]), dpp_move<0xFF>(v[1]), dpp_move<0xFF>(v[2]), dpp_move<0xFF>(v[3]));
}

__device__ __forceinline__ void add_quad(f32x4 &v, uint2 r) {
    v[0] += __uint_as_float(r.x << 16);
    v[1] += __uint_as_float(r.x & 0xFFFF0000u);
    v[2] += __uint_as_float(r.y << 16);
    v[3] += __uint_as_float(r.y & 0xFFFF0000u);
}

// Four consecutive results of a row, at element `at` of y, of a partial (fp32, from element `part` on), or of y with a bf16
// residual added before rounding.  N is a multiple of 16, so four columns are whole and aligned.
__device__ __forceinline__ void store_quad(f32x4 v, void *y, int64_t at, int64_t part, int out_mode, const uint16_t *res) {
    if (res) add_quad(v, *reinterpret_cast<const uint2 *>(res + at));
    if (out_mode == 1)
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(y) + at) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
    else
        *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(y) + part + at) = v;
}

}  // namespace dmr
