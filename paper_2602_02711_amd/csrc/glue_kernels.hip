// Stand-alone decoder glue kernels (any M): RMSNorm, SwiGLU, residual add.  At M == 1 the forwards
// fuse the same arithmetic into their activation staging instead (glue.hpp).
#include "glue.hpp"

namespace dmr {

namespace {

// One workgroup per row: pieces round-robin over 256 threads, sum of squares through DPP / LDS.  A rollout batch is a few
// rows and waits for memory, so a thread asks for its first kHeld pieces of x and gamma at once and keeps them: one trip to
// memory where loading x piece by piece and again with gamma after the sum was three (rows up to 8192 wide; longer ones go
// on in loops).  Same pieces to a thread and the same order of the sum as those loops, hence the same bits.  With the 32-bit
// division below, four decoder layers of 8 rows 205.6 -> 202.0 us, of 16 rows (3 bits) 227.7 -> 222.9; from 32 rows on level.
constexpr int kHeld = 4;
__global__ __launch_bounds__(256) void rmsnorm_kernel(const uint16_t *__restrict__ x,
                                                      const uint16_t *__restrict__ gamma, float eps, int64_t K,
                                                      uint16_t *__restrict__ out) {
    __shared__ float part[4];
    const int64_t row = blockIdx.x;
    const u32x4_t *src = reinterpret_cast<const u32x4_t *>(x + row * K);
    const u32x4_t *gsrc = reinterpret_cast<const u32x4_t *>(gamma);
    uint4 *dst = reinterpret_cast<uint4 *>(out + row * K);
    const int pieces = (int)(K / 8), tid = (int)threadIdx.x;
    auto piece = [](const u32x4_t &v) { return make_uint4(v.x, v.y, v.z, v.w); };
    u32x4_t v[kHeld], g[kHeld];
#pragma unroll
    for (int u = 0; u < kHeld; ++u)
        if (256 * u < pieces) v[u] = src[min(tid + 256 * u, pieces - 1)];
#pragma unroll
    for (int u = 0; u < kHeld; ++u)
        if (256 * u < pieces) g[u] = gsrc[min(tid + 256 * u, pieces - 1)];
    float ss = 0.f;
#pragma unroll
    for (int u = 0; u < kHeld; ++u)
        if (tid + 256 * u < pieces) ss += sumsq_piece(piece(v[u]));
    for (int i = tid + 256 * kHeld; i < pieces; i += 256) ss += sumsq_piece(piece(src[i]));
    ss = wave64_sum(ss);
    if ((tid & 63) == 0) part[tid >> 6] = ss;
    __syncthreads();
    const float scale = rms_scale((part[0] + part[1]) + (part[2] + part[3]), 1.0f / (float)K, eps);
#pragma unroll
    for (int u = 0; u < kHeld; ++u)
        if (tid + 256 * u < pieces) dst[tid + 256 * u] = rmsnorm_piece(piece(v[u]), piece(g[u]), scale);
    for (int i = tid + 256 * kHeld; i < pieces; i += 256) dst[i] = rmsnorm_piece(piece(src[i]), piece(gsrc[i]), scale);
}

// (A launch has fewer than 2^32 threads, so the row of a slot is a 32-bit division.)
__global__ __launch_bounds__(256) void swiglu_kernel(const uint16_t *__restrict__ in, int64_t M, int64_t I,
                                                     uint16_t *__restrict__ out) {
    const uint32_t pieces_per_row = (uint32_t)(I / 8);
    const int64_t slot = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (slot >= M * pieces_per_row) return;
    const uint32_t m = (uint32_t)slot / pieces_per_row, i = (uint32_t)slot - m * pieces_per_row;
    const uint4 *row = reinterpret_cast<const uint4 *>(in + (int64_t)m * 2 * I);
    reinterpret_cast<uint4 *>(out + (int64_t)m * I)[i] = swiglu_piece(row[i], row[pieces_per_row + i]);
}

__global__ __launch_bounds__(256) void add_residual_kernel(const float *__restrict__ acc,
                                                           const uint16_t *res, int64_t count,
                                                           void *out, int out_f32) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= count) return;
    const f32x4 a = *reinterpret_cast<const f32x4 *>(acc + i);
    const uint2 r = *reinterpret_cast<const uint2 *>(res + i);
    f32x4 v;
    v[0] = a[0] + __uint_as_float(r.x << 16);
    v[1] = a[1] + __uint_as_float(r.x & 0xFFFF0000u);
    v[2] = a[2] + __uint_as_float(r.y << 16);
    v[3] = a[3] + __uint_as_float(r.y & 0xFFFF0000u);
    if (out_f32) {
        *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(out) + i) = v;
    } else {
        uint2 o;
        o.x = pack_bf16x2(v[0], v[1]);
        o.y = pack_bf16x2(v[2], v[3]);
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(out) + i) = o;
    }
}

}  // namespace

hipError_t launch_rmsnorm(const uint16_t *x, const uint16_t *gamma, float eps, int64_t M, int64_t K, uint16_t *out,
                          hipStream_t stream) {
    hipLaunchKernelGGL(rmsnorm_kernel, dim3((unsigned)M), dim3(256), 0, stream, x, gamma, eps, K, out);
    return hipGetLastError();
}

hipError_t launch_swiglu(const uint16_t *in, int64_t M, int64_t I, uint16_t *out, hipStream_t stream) {
    const int64_t slots = M * (I / 8);
    hipLaunchKernelGGL(swiglu_kernel, dim3((unsigned)((slots + 255) / 256)), dim3(256), 0, stream, in, M, I, out);
    return hipGetLastError();
}

hipError_t launch_add_residual(const float *acc, const uint16_t *res, int64_t count, void *out, bool out_f32,
                               hipStream_t stream) {
    hipLaunchKernelGGL(add_residual_kernel, dim3((unsigned)((count / 4 + 255) / 256)), dim3(256), 0, stream, acc, res,
                       count, out, out_f32 ? 1 : 0);
    return hipGetLastError();
}

}  // namespace dmr
