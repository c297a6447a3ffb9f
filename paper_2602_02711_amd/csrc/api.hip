// C ABI of dmr_qlinear.h: argument checks (all before the first HIP call), the host handle, and
// the choice of kernel by M.  No device memory is allocated here or anywhere in the library.
#include <new>

#include "bf16_rows_plan.hpp"
#include "glue.hpp"
#include "mid_plan.hpp"
#include "panel_plan.hpp"
#include "row_splits.hpp"

struct dmr_qlinear {
    int64_t K, N;
    int32_t g;
    int32_t bits;           // 4, or 3 for the W3A16 variant
    const uint4 *wt;        // 4-bit streaming blocks
    const uint32_t *wt3;    // 3-bit streaming blocks
    const uint32_t *sz;
    int32_t szs;            // 1: a scale / zero word per (row, group); 0: one per row (per-channel layers)
};

namespace {

constexpr int64_t kSkinnyMaxM = 64;

// Which INT4 kernel serves M rows of a (K, N) layer (measured crossovers, 256 CUs).  The workspace
// query and the forward call both go through this.  Rows: the tile or the slices kernel, as rows_call says.  Mid: what neither of
// these nor the streaming kernels take, up to 16 rows and rows of 2^24 and more.
enum class W4Path { Gemv, Stream, Panel, Rows, Mid, Gemm, GemmRescale };
size_t mid_workspace_bytes(int64_t M, int64_t K, int64_t N) {
    const int sk = dmr::plan_mid(M, K, N).SK;
    return sk > 1 ? (size_t)sk * (size_t)M * (size_t)N * sizeof(float) : 0;
}
W4Path w4_path(int64_t M, int64_t K, int64_t N) {
    if (M == 1) return W4Path::Gemv;
    if (M <= 16) {
        if (dmr::w4_stream_fits(M, K, N)) return W4Path::Stream;
        // long rows: k-sliced panels of x in LDS (measured 10-15 % ahead of the rollout-batch kernel)
        return dmr::w4_panel_applies(M, K, N) ? W4Path::Panel : W4Path::Mid;
    }
    if (M <= kSkinnyMaxM || dmr::rows_beat_tiled(M, K, N)) return dmr::rows_kernels_fit(M, K) ? W4Path::Rows : W4Path::Mid;
    return dmr::w4_gemm_rescale_applies(M, N) ? W4Path::GemmRescale : W4Path::Gemm;
}

// 3-bit layers: the 4-bit size classes on the native 3-bit kernels; a decode row too long for the GEMV's LDS
// budget takes the rollout-batch kernel (which slices K).  The workspace query and the forward call both go
// through this.
enum class W3Path { Gemv, Stream, Panel, Rows, Mid, Gemm, GemmRescale };
W3Path w3_path(int64_t M, int64_t K, int64_t N) {
    if (M == 1) return dmr::w3_gemv_fits(K, N) ? W3Path::Gemv : W3Path::Mid;
    if (M <= 16) {
        if (dmr::w4_stream_fits(M, K, N)) return W3Path::Stream;
        return dmr::w4_panel_applies(M, K, N) ? W3Path::Panel : W3Path::Mid;
    }
    if (M <= kSkinnyMaxM || dmr::rows_beat_tiled(M, K, N)) return dmr::rows_kernels_fit(M, K) ? W3Path::Rows : W3Path::Mid;
    return dmr::w4_gemm_rescale_applies(M, N) ? W3Path::GemmRescale : W3Path::Gemm;
}

// The bf16 twin: GEMV, up to 64 rows the kernel that keeps its activations in registers wherever its plan applies (bf16_rows_plan),
// else the classes Skinny (no workspace: 2..8 rows, and 9..16 of short rows on wide layers) and Mid (fp32 partials).
enum class Bf16Path { Gemv, Skinny, Mid, GemmBig, Gemm };

// M > 64, K >= 1024: whether the direct-to-LDS kernels beat the rollout-batch kernel.  While one round covers the layer they
// take the same time whatever its width; the other kernel's time grows with its blocks (its own row blocks times 128 columns)
// in the steps of its plan.  From 24 values of K, 56 .. 168 blocks and nine row counts in 90 .. 1000, weights from memory; us
// at 200 rows, rollout-batch / tiled:
//   up to 64 blocks (its workgroups fit one round)   K = 2048 24 / 29   K = 4096 38 / 50   K = 8192 58 / 88   K = 14336 93 / 160
//   65 .. 95, K split four ways or more                                 4096, 72 48 / 50   8192, 72 76 / 85   14336, 72 126 / 161
//   65 .. 128, fewer splits                   2048, 96 blocks 36 / 30   4096, 96 56 / 51   8192, 96 96 / 89   14336, 96 163 / 164
//   above 128                                 2048, 132       49 / 31   4096, 132 77 / 53  8192, 132 136 / 95 14336, 132 237 / 174
// The third class changes hands between K = 5120 (0.95 .. 1.09 of the tiled time over the row counts) and 6144 (0.91 .. 1.06)
// and is the rollout-batch kernel's from there on, but for K = 8192 (0.96 .. 1.11; 7936 and 8704 0.91 .. 1.07) and for a K
// whose groups do not split on its plan (8064, 96 blocks: 115 / 93).
bool tiled_beats_rollout(int64_t M, int64_t K, int64_t N) {
    const dmr::MidPlan m = dmr::plan_mid(M, K, N);
    const int64_t blocks = m.mblocks * ((N + 127) / 128);
    if (blocks <= 64 || blocks > 128) return blocks > 128;
    return m.SK < 4 && (K < 5632 || K == 8192 || m.SK == 1);
}
Bf16Path bf16_path(int64_t M, int64_t K, int64_t N) {
    if (M == 1) return Bf16Path::Gemv;
    if (M <= 8 || (M <= 16 && N / dmr::kTileRows > 1024 && M * (K / 8 + 1) <= 9216)) return Bf16Path::Skinny;
    if (M <= 64) return Bf16Path::Mid;
    if (K < 1024) {                  // no direct-to-LDS kernel there
        if (((M + 127) / 128) * ((N + 127) / 128) <= 128) return Bf16Path::Mid;
    } else if (!tiled_beats_rollout(M, K, N)) {
        return Bf16Path::Mid;
    }
    return dmr::gemm_big_tile_rows(M, K, N) != 0 ? Bf16Path::GemmBig : Bf16Path::Gemm;
}

// The rollout-batch kernel keeps 33..64 rows where its plan is one full round of one-tile workgroups with four splits of K and this one's
// has two, whose last round of tiles is ragged: K = 4096 and 3700 .. 4096 outputs (us, that kernel / this one: 48 rows 4096 -> 4096 13.0 /
// 14.2, -> 3968 0.81 of its time, -> 3712 0.87, -> 3840 0.99; level at 3072 and 3584, 1.4 x behind from 4112 on).  With three splits and
// more here it is 8 .. 25 % behind over K = 4608 .. 8192 and the same widths.
dmr::Bf16RowsPlan bf16_rows_plan(int64_t M, int64_t K, int64_t N) {
    const bool mid = bf16_path(M, K, N) == Bf16Path::Mid;
    const dmr::MidPlan m = dmr::plan_mid(M, K, N);
    dmr::Bf16RowsPlan p = dmr::plan_bf16_rows(M, K, N, mid ? m.SK : 1);
    if (mid && M > 32 && p.SK == 2 && m.R == 1 && m.SK == 4 && m.wgs > dmr::kCus * 7 / 8 && m.wgs <= dmr::kCus) p.ok = false;
    return p;
}

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// Workspace of a fused forward that falls back to glue kernel + plain forward: the glue output
// (bf16 [M][K]), the fp32 result awaiting its residual ([M][N]), then the plain forward's own.
size_t fused_extra_bytes(int64_t M, int64_t K, int64_t N, int pro, bool has_res) {
    return (pro != DMR_PRO_NONE ? align256((size_t)M * (size_t)K * 2) : 0) +
           (has_res ? align256((size_t)M * (size_t)N * 4) : 0);
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

dmr_status_t check_shape(int64_t K, int64_t N, int32_t g) {
    if (K <= 0 || N <= 0 || g <= 0) return DMR_ERR_SHAPE;
    if (g != dmr::kGroup) return (K % g == 0) ? DMR_ERR_UNSUPPORTED : DMR_ERR_SHAPE;
    if (K % dmr::kGroup != 0 || N % dmr::kTileRows != 0) return DMR_ERR_SHAPE;
    // block and element indices are formed in 64 bits; the grid's x dimension is 32 bits
    if (N / dmr::kTileRows > 0x7FFFFFFF || K > (int64_t(1) << 31) || N > (int64_t(1) << 31))
        return DMR_ERR_SHAPE;
    return DMR_OK;
}

dmr_status_t hip_status(hipError_t e) { return e == hipSuccess ? DMR_OK : DMR_ERR_HIP; }

}  // namespace

namespace {

// What M rows of this layer take: what the query says for the shape, less for the tiled kernels of a per-channel layer, which keep the
// sums of the activation rows alone there.
size_t layer_workspace_bytes(const dmr_qlinear_t *layer, int64_t M) {
    if (layer->bits == 3) return dmr_qlinear_w3_workspace_bytes(M, layer->K, layer->N);
    if (layer->szs == 0 && w4_path(M, layer->K, layer->N) == W4Path::GemmRescale) return (size_t)M * sizeof(float2);
    return dmr_qlinear_workspace_bytes(M, layer->K, layer->N);
}

// The forwards with an optional bf16 residual added where the result is stored.
dmr_status_t forward_quant(const dmr_qlinear_t *layer, const uint16_t *d_x, int64_t M, void *d_y, dmr_out_t out,
                           const uint16_t *res, void *d_ws, size_t ws_bytes, hipStream_t s) {
    if (!layer) return DMR_ERR_NULL;
    if (M < 0 || M > (int64_t(1) << 22)) return DMR_ERR_SHAPE;
    if (out != DMR_OUT_BF16 && out != DMR_OUT_FP32) return DMR_ERR_UNSUPPORTED;
    if (M == 0) return DMR_OK;
    if (!d_x || !d_y) return DMR_ERR_NULL;
    if (!aligned16(d_x) || !aligned16(d_y) || (d_ws && !aligned16(d_ws))) return DMR_ERR_ALIGN;
    const bool f32 = out == DMR_OUT_FP32;
    if (layer->bits == 3) {
        const dmr::LayerView3 L3{layer->K, layer->N, layer->wt3, layer->sz};
        const size_t need3 = layer_workspace_bytes(layer, M);
        if (need3 > 0 && (!d_ws || ws_bytes < need3)) {
            if (!dmr::runs_unsplit(M, layer->K, layer->N)) return DMR_ERR_WORKSPACE;
            d_ws = nullptr;
        }
        switch (w3_path(M, layer->K, layer->N)) {
            case W3Path::Gemv: return hip_status(dmr::launch_w3_gemv(L3, d_x, d_y, f32, res, s));
            case W3Path::Stream: return hip_status(dmr::launch_w3_stream(L3, d_x, M, d_y, f32, res, s));
            case W3Path::Panel: return hip_status(dmr::launch_w3_panel(L3, d_x, M, d_y, f32, res, d_ws, s));
            case W3Path::Rows:
                return hip_status(dmr::launch_w3_rows(L3, d_x, M, d_y, f32, res, d_ws, dmr::rows_call(M, L3.K, L3.N, d_ws), s));
            case W3Path::Mid: return hip_status(dmr::launch_w3_mid(L3, d_x, M, d_y, f32, res, d_ws, s));
            case W3Path::Gemm: return hip_status(dmr::launch_w3_gemm(L3, d_x, M, d_y, f32, res, s));
            case W3Path::GemmRescale: return hip_status(dmr::launch_w3_gemm_rescale(L3, d_x, M, d_y, f32, res, d_ws, s));
        }
        return DMR_ERR_UNSUPPORTED;
    }
    const size_t need = layer_workspace_bytes(layer, M);
    if (need > 0 && (!d_ws || ws_bytes < need)) {
        if (!dmr::runs_unsplit(M, layer->K, layer->N)) return DMR_ERR_WORKSPACE;
        d_ws = nullptr;
    }
    const dmr::LayerView L{layer->K, layer->N, layer->wt, layer->sz, layer->szs};
    const W4Path path = w4_path(M, layer->K, layer->N);
    dmr::Fusion f;
    f.res = res;
    if (path == W4Path::Gemv) {
        const hipError_t e = dmr::launch_w4_gemv_fused(L, d_x, d_y, f32, f, s);
        if (e != hipErrorInvalidValue) return hip_status(e);   // else: shape outside its range
    }
    if (path == W4Path::Stream) {
        const hipError_t e = dmr::launch_w4_stream_fused(L, d_x, M, d_y, f32, f, s);
        if (e != hipErrorInvalidValue) return hip_status(e);   // else: activations do not fit LDS
    }
    if (path == W4Path::Panel) return hip_status(dmr::launch_w4_panel(L, d_x, M, d_y, f32, res, d_ws, s));
    if (path == W4Path::Rows)
        return hip_status(dmr::launch_w4_rows(L, d_x, M, d_y, f32, res, d_ws, dmr::rows_call(M, L.K, L.N, d_ws), s));
    if (path == W4Path::Mid) return hip_status(dmr::launch_w4_mid(L, d_x, M, d_y, f32, res, d_ws, s));
    if (M <= kSkinnyMaxM) return hip_status(dmr::launch_w4_skinny(L, d_x, M, d_y, f32, s));
    if (path == W4Path::GemmRescale) return hip_status(dmr::launch_w4_gemm_rescale(L, d_x, M, d_y, f32, res, d_ws, s));
    // Not reached with the present crossovers (the rescaling kernel takes every tiled shape and calls this kernel
    // itself for the column blocks it declines): 128 x 128 tiles on the exact integer codes q - z, the group's scale
    // applied to the group's partial sums in fp32.  (No tiled kernel rounds the weights to bf16 on their way into
    // LDS, what dmr_qlinear_dequantize returns: that leaves an error of about 1.7e-3 rms(y) standard deviation per
    // output, so that the largest of 10^7 .. 10^8 outputs lands at 0.8 .. 1.1 times the 1e-2 rms bound.)
    return hip_status(dmr::launch_w4_gemm(L, d_x, M, d_y, f32, res, s));
}

dmr_status_t forward_bf16(const uint16_t *d_w, const uint16_t *d_x, int64_t M, int64_t K, int64_t N, void *d_y,
                          dmr_out_t out, const uint16_t *res, void *d_ws, size_t ws_bytes, hipStream_t s) {
    const dmr_status_t shape = check_shape(K, N, dmr::kGroup);
    if (shape != DMR_OK) return shape;
    if (M < 0 || M > (int64_t(1) << 22)) return DMR_ERR_SHAPE;
    if (out != DMR_OUT_BF16 && out != DMR_OUT_FP32) return DMR_ERR_UNSUPPORTED;
    if (M == 0) return DMR_OK;
    if (!d_w || !d_x || !d_y) return DMR_ERR_NULL;
    if (!aligned16(d_w) || !aligned16(d_x) || !aligned16(d_y) || (d_ws && !aligned16(d_ws)))
        return DMR_ERR_ALIGN;
    const size_t need = dmr_qlinear_bf16_workspace_bytes(M, K, N);
    if (need > 0 && (!d_ws || ws_bytes < need)) return DMR_ERR_WORKSPACE;
    const bool f32 = out == DMR_OUT_FP32;
    const Bf16Path path = bf16_path(M, K, N);
    if (path == Bf16Path::Gemv) {
        dmr::Fusion fusion;
        fusion.res = res;
        const hipError_t e = dmr::launch_bf16_gemv_fused(d_w, d_x, K, N, d_y, f32, fusion, s);
        if (e != hipErrorInvalidValue) return hip_status(e);   // else: K outside its range
        return hip_status(dmr::launch_bf16_skinny(d_w, d_x, M, K, N, d_y, f32, res, s));
    }
    const dmr::Bf16RowsPlan rows = bf16_rows_plan(M, K, N);
    if (rows.ok) return hip_status(dmr::launch_bf16_rows(d_w, d_x, M, K, N, d_y, f32, res, d_ws, rows, s));
    switch (path) {
        case Bf16Path::Skinny: return hip_status(dmr::launch_bf16_skinny(d_w, d_x, M, K, N, d_y, f32, res, s));
        case Bf16Path::Mid: return hip_status(dmr::launch_bf16_mid(d_w, d_x, M, K, N, d_y, f32, res, d_ws, s));
        case Bf16Path::GemmBig: return hip_status(dmr::launch_bf16_gemm_w8(d_w, d_x, M, K, N, d_y, f32, res, s));
        default: {
            // 128 x 128 tiles: the direct-to-LDS kernel where its pipeline has room to pay (25-30 % ahead at 256 workgroups;
            // grids of more than a few hundred get here only where one column block is the whole layer, and there the two are
            // level: 200000 x 4096 -> 128 429 / 458 us, 100000 rows 242 / 233)
            if (K >= 1024) return hip_status(dmr::launch_bf16_gemm_dma128(d_w, d_x, M, K, N, d_y, f32, res, s));
            return hip_status(dmr::launch_bf16_gemm(d_w, d_x, M, K, N, d_y, f32, res, s));
        }
    }
}

}  // namespace

extern "C" {

size_t dmr_qlinear_storage_bytes(int64_t K, int64_t N, int32_t g) {
    if (check_shape(K, N, g) != DMR_OK) return 0;
    return dmr::weight_region_bytes(K, N) + dmr::sz_region_bytes(K, N);
}

size_t dmr_qlinear_workspace_bytes(int64_t M, int64_t K, int64_t N) {
    if (M <= 0 || K <= 0 || K % dmr::kGroup != 0 || N <= 0 || N % dmr::kTileRows != 0) return 0;
    switch (w4_path(M, K, N)) {
        case W4Path::Mid: return mid_workspace_bytes(M, K, N);    // fp32 partials when K is split
        case W4Path::Panel: return dmr::w4_panel_workspace_bytes(M, K, N);    // likewise
        case W4Path::Rows: return dmr::rows_workspace_bytes(M, K, N);         // likewise
        case W4Path::GemmRescale: return dmr::w4_gemm_rescale_workspace_bytes(M, K, N);   // zero-point operands, factors
        default: return 0;
    }
}

size_t dmr_qlinear_bf16_workspace_bytes(int64_t M, int64_t K, int64_t N) {
    if (M <= 0 || K <= 0 || K % dmr::kGroup != 0 || N <= 0 || N % dmr::kTileRows != 0) return 0;
    const dmr::Bf16RowsPlan rows = bf16_rows_plan(M, K, N);
    if (rows.ok) return rows.SK > 1 ? (size_t)rows.SK * (size_t)M * (size_t)N * sizeof(float) : 0;
    return bf16_path(M, K, N) == Bf16Path::Mid ? dmr::bf16_mid_workspace_bytes(M, K, N) : 0;
}

dmr_status_t dmr_qlinear_create(dmr_qlinear_t **out, int64_t K, int64_t N, int32_t g,
                                const uint32_t *d_qweight, const uint16_t *d_scales,
                                const uint16_t *d_zeros, void *d_storage, size_t storage_bytes,
                                void *stream) {
    if (!out) return DMR_ERR_NULL;
    *out = nullptr;
    const dmr_status_t shape = check_shape(K, N, g);
    if (shape != DMR_OK) return shape;
    if (!d_qweight || !d_scales || !d_zeros || !d_storage) return DMR_ERR_NULL;
    if (!aligned16(d_qweight) || !aligned16(d_scales) || !aligned16(d_zeros) || !aligned16(d_storage))
        return DMR_ERR_ALIGN;
    if (storage_bytes < dmr_qlinear_storage_bytes(K, N, g)) return DMR_ERR_WORKSPACE;

    dmr_qlinear *h = new (std::nothrow) dmr_qlinear;
    if (!h) return DMR_ERR_NULL;
    h->K = K;
    h->N = N;
    h->g = g;
    h->bits = 4;
    h->szs = 1;
    h->wt3 = nullptr;
    uint8_t *base = static_cast<uint8_t *>(d_storage);
    h->wt = reinterpret_cast<const uint4 *>(base);
    h->sz = reinterpret_cast<const uint32_t *>(base + dmr::weight_region_bytes(K, N));
    const hipError_t e = dmr::launch_retile(K, N, d_qweight, d_scales, d_zeros,
                                            reinterpret_cast<uint4 *>(base),
                                            reinterpret_cast<uint32_t *>(base + dmr::weight_region_bytes(K, N)),
                                            false, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) {
        delete h;
        return DMR_ERR_HIP;
    }
    *out = h;
    return DMR_OK;
}

size_t dmr_qlinear_per_channel_storage_bytes(int64_t K, int64_t N) {
    if (check_shape(K, N, dmr::kGroup) != DMR_OK) return 0;
    return dmr::weight_region_bytes(K, N) + dmr::sz_region_bytes_per_channel(N);
}

dmr_status_t dmr_qlinear_create_per_channel(dmr_qlinear_t **out, int64_t K, int64_t N,
                                            const uint32_t *d_qweight, const uint16_t *d_scales,
                                            void *d_storage, size_t storage_bytes, void *stream) {
    if (!out) return DMR_ERR_NULL;
    *out = nullptr;
    const dmr_status_t shape = check_shape(K, N, dmr::kGroup);
    if (shape != DMR_OK) return shape;
    if (!d_qweight || !d_scales || !d_storage) return DMR_ERR_NULL;
    if (!aligned16(d_qweight) || !aligned16(d_scales) || !aligned16(d_storage)) return DMR_ERR_ALIGN;
    if (storage_bytes < dmr_qlinear_per_channel_storage_bytes(K, N)) return DMR_ERR_WORKSPACE;
    dmr_qlinear *h = new (std::nothrow) dmr_qlinear;
    if (!h) return DMR_ERR_NULL;
    h->K = K;
    h->N = N;
    h->g = (int32_t)K;      // one group spans the whole row
    h->bits = 4;
    h->szs = 0;             // one scale word per row behind the weights: 0.5 byte per weight + 4 bytes per row
    h->wt3 = nullptr;
    uint8_t *base = static_cast<uint8_t *>(d_storage);
    h->wt = reinterpret_cast<const uint4 *>(base);
    h->sz = reinterpret_cast<const uint32_t *>(base + dmr::weight_region_bytes(K, N));
    const hipError_t e = dmr::launch_retile(K, N, d_qweight, d_scales, nullptr, reinterpret_cast<uint4 *>(base),
                                            reinterpret_cast<uint32_t *>(base + dmr::weight_region_bytes(K, N)),
                                            true, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) {
        delete h;
        return DMR_ERR_HIP;
    }
    *out = h;
    return DMR_OK;
}

size_t dmr_qlinear_w3_storage_bytes(int64_t K, int64_t N, int32_t g) {
    if (check_shape(K, N, g) != DMR_OK) return 0;
    return dmr::weight3_region_bytes(K, N) + dmr::sz_region_bytes(K, N);
}

size_t dmr_qlinear_w3_workspace_bytes(int64_t M, int64_t K, int64_t N) {
    if (M <= 0 || K <= 0 || K % dmr::kGroup != 0 || N <= 0 || N % dmr::kTileRows != 0) return 0;
    switch (w3_path(M, K, N)) {
        case W3Path::Panel: return dmr::w4_panel_workspace_bytes(M, K, N);   // fp32 partials of the k slices
        case W3Path::Mid: return mid_workspace_bytes(M, K, N);       // fp32 partials when K is split
        case W3Path::Rows: return dmr::rows_workspace_bytes(M, K, N);        // likewise
        case W3Path::GemmRescale: return dmr::w4_gemm_rescale_workspace_bytes(M, K, N);   // zero-point operands, factors
        default: return 0;
    }
}

dmr_status_t dmr_qlinear_w3_create(dmr_qlinear_t **out, int64_t K, int64_t N, int32_t g,
                                   const uint32_t *d_qweight3, const uint16_t *d_scales,
                                   const uint16_t *d_zeros, void *d_storage, size_t storage_bytes,
                                   void *stream) {
    if (!out) return DMR_ERR_NULL;
    *out = nullptr;
    const dmr_status_t shape = check_shape(K, N, g);
    if (shape != DMR_OK) return shape;
    if (!d_qweight3 || !d_scales || !d_zeros || !d_storage) return DMR_ERR_NULL;
    if (!aligned16(d_qweight3) || !aligned16(d_scales) || !aligned16(d_zeros) || !aligned16(d_storage))
        return DMR_ERR_ALIGN;
    if (storage_bytes < dmr_qlinear_w3_storage_bytes(K, N, g)) return DMR_ERR_WORKSPACE;
    dmr_qlinear *h = new (std::nothrow) dmr_qlinear;
    if (!h) return DMR_ERR_NULL;
    h->K = K;
    h->N = N;
    h->g = g;
    h->bits = 3;
    h->szs = 1;
    h->wt = nullptr;
    uint8_t *base = static_cast<uint8_t *>(d_storage);
    h->wt3 = reinterpret_cast<const uint32_t *>(base);
    h->sz = reinterpret_cast<const uint32_t *>(base + dmr::weight3_region_bytes(K, N));
    const hipError_t e = dmr::launch_retile3(K, N, d_qweight3, d_scales, d_zeros,
                                             reinterpret_cast<uint32_t *>(base),
                                             reinterpret_cast<uint32_t *>(base + dmr::weight3_region_bytes(K, N)),
                                             static_cast<hipStream_t>(stream));
    if (e != hipSuccess) {
        delete h;
        return DMR_ERR_HIP;
    }
    *out = h;
    return DMR_OK;
}

dmr_status_t dmr_qlinear_quantize_w3(int64_t K, int64_t N, int32_t g, const float *d_w, uint32_t *d_qweight3,
                                     uint16_t *d_scales, uint16_t *d_zeros, void *stream) {
    const dmr_status_t shape = check_shape(K, N, g);
    if (shape != DMR_OK) return shape;
    if (!d_w || !d_qweight3 || !d_scales || !d_zeros) return DMR_ERR_NULL;
    if (!aligned16(d_w) || !aligned16(d_qweight3) || !aligned16(d_scales) || !aligned16(d_zeros))
        return DMR_ERR_ALIGN;
    return hip_status(dmr::launch_quantize3(K, N, d_w, d_qweight3, d_scales, d_zeros,
                                            static_cast<hipStream_t>(stream)));
}

dmr_status_t dmr_qlinear_dequantize(const dmr_qlinear_t *layer, uint16_t *d_w_bf16, void *stream) {
    if (!layer || !d_w_bf16) return DMR_ERR_NULL;
    if (!aligned16(d_w_bf16)) return DMR_ERR_ALIGN;
    if (layer->bits == 3) {
        const dmr::LayerView3 L3{layer->K, layer->N, layer->wt3, layer->sz};
        return hip_status(dmr::launch_dequantize3(L3, d_w_bf16, static_cast<hipStream_t>(stream)));
    }
    const dmr::LayerView L{layer->K, layer->N, layer->wt, layer->sz, layer->szs};
    return hip_status(dmr::launch_dequantize(L, d_w_bf16, static_cast<hipStream_t>(stream)));
}

dmr_status_t dmr_qlinear_forward(const dmr_qlinear_t *layer, const uint16_t *d_x, int64_t M, void *d_y,
                                 dmr_out_t out, void *d_ws, size_t ws_bytes, void *stream) {
    return forward_quant(layer, d_x, M, d_y, out, nullptr, d_ws, ws_bytes, static_cast<hipStream_t>(stream));
}

dmr_status_t dmr_qlinear_bf16_forward(const uint16_t *d_w, const uint16_t *d_x, int64_t M, int64_t K,
                                      int64_t N, void *d_y, dmr_out_t out, void *d_ws, size_t ws_bytes,
                                      void *stream) {
    return forward_bf16(d_w, d_x, M, K, N, d_y, out, nullptr, d_ws, ws_bytes, static_cast<hipStream_t>(stream));
}

dmr_status_t dmr_glue_rmsnorm(const uint16_t *d_x, const uint16_t *d_gamma, float eps, int64_t M, int64_t K,
                              uint16_t *d_out, void *stream) {
    if (M < 0 || M > (int64_t(1) << 22) || K <= 0 || K % 8 != 0 || K > (int64_t(1) << 31)) return DMR_ERR_SHAPE;
    if (!(eps >= 0.f)) return DMR_ERR_UNSUPPORTED;
    if (M == 0) return DMR_OK;
    if (!d_x || !d_gamma || !d_out) return DMR_ERR_NULL;
    if (!aligned16(d_x) || !aligned16(d_gamma) || !aligned16(d_out)) return DMR_ERR_ALIGN;
    return hip_status(dmr::launch_rmsnorm(d_x, d_gamma, eps, M, K, d_out, static_cast<hipStream_t>(stream)));
}

dmr_status_t dmr_glue_swiglu(const uint16_t *d_in, int64_t M, int64_t I, uint16_t *d_out, void *stream) {
    if (M < 0 || M > (int64_t(1) << 22) || I <= 0 || I % 8 != 0 || I > (int64_t(1) << 30)) return DMR_ERR_SHAPE;
    if (M == 0) return DMR_OK;
    if (!d_in || !d_out) return DMR_ERR_NULL;
    if (!aligned16(d_in) || !aligned16(d_out)) return DMR_ERR_ALIGN;
    return hip_status(dmr::launch_swiglu(d_in, M, I, d_out, static_cast<hipStream_t>(stream)));
}

size_t dmr_qlinear_fused_workspace_bytes(const dmr_qlinear_t *layer, int64_t M, dmr_prologue_t pro,
                                         int32_t has_residual) {
    if (!layer || M <= 0) return 0;
    return fused_extra_bytes(M, layer->K, layer->N, pro, has_residual != 0) + layer_workspace_bytes(layer, M);
}

size_t dmr_qlinear_bf16_fused_workspace_bytes(int64_t M, int64_t K, int64_t N, dmr_prologue_t pro,
                                              int32_t has_residual) {
    if (M <= 0 || K <= 0 || N <= 0) return 0;
    return fused_extra_bytes(M, K, N, pro, has_residual != 0) + dmr_qlinear_bf16_workspace_bytes(M, K, N);
}

}  // extern "C"

namespace {

// Argument checks shared by the two fused forwards; DMR_OK means "go on".
dmr_status_t check_fused(dmr_prologue_t pro, const uint16_t *d_in, const uint16_t *d_gamma, float eps,
                         const uint16_t *d_residual, int64_t M, const void *d_y, dmr_out_t out, const void *d_ws) {
    if (M < 0 || M > (int64_t(1) << 22)) return DMR_ERR_SHAPE;
    if (out != DMR_OUT_BF16 && out != DMR_OUT_FP32) return DMR_ERR_UNSUPPORTED;
    if (pro != DMR_PRO_NONE && pro != DMR_PRO_RMSNORM && pro != DMR_PRO_SWIGLU) return DMR_ERR_UNSUPPORTED;
    if (pro == DMR_PRO_RMSNORM && !(eps >= 0.f)) return DMR_ERR_UNSUPPORTED;
    if (M == 0) return DMR_OK;
    if (!d_in || !d_y || (pro == DMR_PRO_RMSNORM && !d_gamma)) return DMR_ERR_NULL;
    if (!aligned16(d_in) || !aligned16(d_y) || (d_gamma && !aligned16(d_gamma)) ||
        (d_residual && !aligned16(d_residual)) || (d_ws && !aligned16(d_ws)))
        return DMR_ERR_ALIGN;
    return DMR_OK;
}

// Whether the kernel that serves M rows of this layer adds a residual where it stores the result (the direct-from-L2 kernel does
// not).
bool quant_adds_residual(const dmr_qlinear_t *layer, int64_t M) {
    if (layer->bits == 3) return true;
    const W4Path path = w4_path(M, layer->K, layer->N);
    return !(path == W4Path::Gemv && !dmr::w4_gemv_fits(layer->K, layer->N, true));
}

bool overlap(const void *a, size_t na, const void *b, size_t nb) {
    const uintptr_t pa = reinterpret_cast<uintptr_t>(a), pb = reinterpret_cast<uintptr_t>(b);
    return pa < pb + nb && pb < pa + na;
}

// The composition for more rows than the kernels that fuse the prologue take: glue kernel into the workspace, then the
// forward, which adds the residual where it stores the result.  (That replaced an fp32 result [M][N] in the workspace and a
// launch that added the residual to it: same sums, one launch and two passes over M x N less; rollout of eight rows
// 214 -> 209 us for four decoder layers, prefill chunk of 1000 rows 972 -> 950 us for two.)  The fp32 detour is left for
// the kernels without a residual and for an output over the activations that the forward still reads.  `forward` runs the
// plain forward on (x, y, out type, residual, inner workspace).
template <typename Forward>
dmr_status_t run_unfused(dmr_prologue_t pro, const uint16_t *d_in, const uint16_t *d_gamma, float eps,
                         const uint16_t *d_residual, bool adds_residual, int64_t M, int64_t K, int64_t N, void *d_y,
                         dmr_out_t out, void *d_ws, size_t ws_bytes, hipStream_t s, Forward forward) {
    uint8_t *ws = static_cast<uint8_t *>(d_ws);
    size_t used = 0;
    const uint16_t *x = d_in;
    if (pro != DMR_PRO_NONE) {
        uint16_t *xg = reinterpret_cast<uint16_t *>(ws);
        used += align256((size_t)M * (size_t)K * 2);
        const hipError_t e = pro == DMR_PRO_RMSNORM ? dmr::launch_rmsnorm(d_in, d_gamma, eps, M, K, xg, s)
                                                     : dmr::launch_swiglu(d_in, M, K, xg, s);
        if (e != hipSuccess) return DMR_ERR_HIP;
        x = xg;
    }
    const size_t y_bytes = (size_t)M * (size_t)N * (out == DMR_OUT_FP32 ? 4 : 2);
    if (!d_residual || (adds_residual && !overlap(d_y, y_bytes, x, (size_t)M * (size_t)K * 2) &&
                        (d_y == d_residual ? out == DMR_OUT_BF16 : !overlap(d_y, y_bytes, d_residual, (size_t)M * (size_t)N * 2))))
        return forward(x, d_y, out, d_residual, ws + used, ws_bytes - used);
    float *acc = reinterpret_cast<float *>(ws + used);
    used += align256((size_t)M * (size_t)N * 4);
    const dmr_status_t st = forward(x, acc, DMR_OUT_FP32, nullptr, ws + used, ws_bytes - used);
    if (st != DMR_OK) return st;
    return hip_status(dmr::launch_add_residual(acc, d_residual, M * N, d_y, out == DMR_OUT_FP32, s));
}

}  // namespace

extern "C" {

dmr_status_t dmr_qlinear_forward_fused(const dmr_qlinear_t *layer, dmr_prologue_t pro, const uint16_t *d_in,
                                       const uint16_t *d_gamma, float eps, const uint16_t *d_residual, int64_t M,
                                       void *d_y, dmr_out_t out, void *d_ws, size_t ws_bytes, void *stream) {
    if (!layer) return DMR_ERR_NULL;
    const dmr_status_t chk = check_fused(pro, d_in, d_gamma, eps, d_residual, M, d_y, out, d_ws);
    if (chk != DMR_OK || M == 0) return chk;
    const size_t need = dmr_qlinear_fused_workspace_bytes(layer, M, pro, d_residual != nullptr);
    if (need > 0 && (!d_ws || ws_bytes < need)) {
        const size_t least = dmr::runs_unsplit(M, layer->K, layer->N) ? fused_extra_bytes(M, layer->K, layer->N, pro, d_residual != nullptr) : need;
        if (least > 0 && (!d_ws || ws_bytes < least)) return DMR_ERR_WORKSPACE;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (M == 1 && layer->bits == 4) {
        const dmr::LayerView L{layer->K, layer->N, layer->wt, layer->sz, layer->szs};
        dmr::Fusion f;
        f.pro = (int)pro;
        f.aux = d_gamma;
        f.eps = eps;
        f.res = d_residual;
        const hipError_t e = dmr::launch_w4_gemv_fused(L, d_in, d_y, out == DMR_OUT_FP32, f, s);
        if (e != hipErrorInvalidValue) return hip_status(e);   // else: shape outside the GEMV's range
    }
    return run_unfused(pro, d_in, d_gamma, eps, d_residual, quant_adds_residual(layer, M), M, layer->K, layer->N, d_y, out,
                       d_ws, ws_bytes, s,
                       [&](const uint16_t *x, void *y, dmr_out_t o, const uint16_t *res, void *ws, size_t wsb) {
                           return forward_quant(layer, x, M, y, o, res, ws, wsb, s);
                       });
}

dmr_status_t dmr_qlinear_bf16_forward_fused(const uint16_t *d_w, dmr_prologue_t pro, const uint16_t *d_in,
                                            const uint16_t *d_gamma, float eps, const uint16_t *d_residual,
                                            int64_t M, int64_t K, int64_t N, void *d_y, dmr_out_t out, void *d_ws,
                                            size_t ws_bytes, void *stream) {
    const dmr_status_t shape = check_shape(K, N, dmr::kGroup);
    if (shape != DMR_OK) return shape;
    const dmr_status_t chk = check_fused(pro, d_in, d_gamma, eps, d_residual, M, d_y, out, d_ws);
    if (chk != DMR_OK || M == 0) return chk;
    if (!d_w) return DMR_ERR_NULL;
    if (!aligned16(d_w)) return DMR_ERR_ALIGN;
    const size_t need = dmr_qlinear_bf16_fused_workspace_bytes(M, K, N, pro, d_residual != nullptr);
    if (need > 0 && (!d_ws || ws_bytes < need)) return DMR_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (M == 1) {
        dmr::Fusion f;
        f.pro = (int)pro;
        f.aux = d_gamma;
        f.eps = eps;
        f.res = d_residual;
        const hipError_t e = dmr::launch_bf16_gemv_fused(d_w, d_in, K, N, d_y, out == DMR_OUT_FP32, f, s);
        if (e != hipErrorInvalidValue) return hip_status(e);   // else: K outside its range, or RMSNorm over slices
    }
    return run_unfused(pro, d_in, d_gamma, eps, d_residual, true, M, K, N, d_y, out, d_ws, ws_bytes, s,
                       [&](const uint16_t *x, void *y, dmr_out_t o, const uint16_t *res, void *ws, size_t wsb) {
                           return forward_bf16(d_w, x, M, K, N, y, o, res, ws, wsb, s);
                       });
}

dmr_status_t dmr_qlinear_quantize(int64_t K, int64_t N, int32_t g, const float *d_w, uint32_t *d_qweight,
                                  uint16_t *d_scales, uint16_t *d_zeros, void *stream) {
    const dmr_status_t shape = check_shape(K, N, g);
    if (shape != DMR_OK) return shape;
    if (!d_w || !d_qweight || !d_scales || !d_zeros) return DMR_ERR_NULL;
    if (!aligned16(d_w) || !aligned16(d_qweight) || !aligned16(d_scales) || !aligned16(d_zeros))
        return DMR_ERR_ALIGN;
    return hip_status(dmr::launch_quantize(K, N, d_w, d_qweight, d_scales, d_zeros,
                                           static_cast<hipStream_t>(stream)));
}

dmr_status_t dmr_probe_hbm_read(const void *d_buf, size_t bytes, uint32_t *d_sink, int32_t blocks,
                                void *stream) {
    if (!d_buf || !d_sink) return DMR_ERR_NULL;
    if (bytes == 0 || bytes % 16 != 0 || blocks <= 0 || blocks > (1 << 20)) return DMR_ERR_SHAPE;
    if (!aligned16(d_buf) || !aligned16(d_sink)) return DMR_ERR_ALIGN;
    return hip_status(dmr::launch_hbm_read_probe(d_buf, bytes, d_sink, blocks, static_cast<hipStream_t>(stream)));
}

const char *dmr_qlinear_kernel_path(dmr_format_t format, int64_t M, int64_t K, int64_t N) {
    if (M <= 0 || check_shape(K, N, dmr::kGroup) != DMR_OK) return "none";
    auto bf16_name = [&]() -> const char * {
        if (M <= 64 && bf16_rows_plan(M, K, N).ok) return "bf16_rows";
        switch (bf16_path(M, K, N)) {
            case Bf16Path::Gemv: return dmr::bf16_gemv_fits(K) ? "bf16_gemv" : "bf16_skinny";
            case Bf16Path::Skinny: return "bf16_skinny";
            case Bf16Path::Mid: return "bf16_mid";
            case Bf16Path::GemmBig: {
                const int rows = dmr::gemm_big_tile_rows(M, K, N);
                return rows == 256 ? "bf16_gemm256" : rows == 192 ? "bf16_gemm192x256" : "bf16_gemm128x256";
            }
            default: return K >= 1024 ? "bf16_gemm128_dma" : "bf16_gemm128";
        }
    };
    switch (format) {
        case DMR_FMT_BF16: return bf16_name();
        case DMR_FMT_W3_G128:
            switch (w3_path(M, K, N)) {
                case W3Path::Gemv: return "w3_gemv";
                case W3Path::Stream: return "w3_stream";
                case W3Path::Panel: return "w3_panel";
                case W3Path::Rows: return dmr::rows_call(M, K, N).slices ? "w3_slices" : "w3_tile";
                case W3Path::Mid: return "w3_mid";
                case W3Path::GemmRescale:
                    if (dmr::w4_gemm_rescale_tile_rows(M, N) == 128) return "w3_gemm128_rescale";
                    return dmr::w4_gemm_rescale_wave_columns(M, N) == 4 ? "w3_gemm256_rescale" : "w3_gemm256x128_rescale";
                default: return "w3_gemm128_exact";
            }
        case DMR_FMT_W4_G128:
        case DMR_FMT_W4_PER_CHANNEL:
            switch (w4_path(M, K, N)) {
                case W4Path::Gemv: return dmr::w4_gemv_fits(K, N, false) ? "w4_gemv" : "w4_skinny";
                case W4Path::Stream: return "w4_stream";
                case W4Path::Panel: return "w4_panel";
                case W4Path::Rows: return dmr::rows_call(M, K, N).slices ? "w4_slices" : "w4_tile";
                case W4Path::Mid: return "w4_mid";
                case W4Path::GemmRescale:
                    if (dmr::w4_gemm_rescale_tile_rows(M, N) == 128) return "w4_gemm128_rescale";
                    return dmr::w4_gemm_rescale_wave_columns(M, N) == 4 ? "w4_gemm256_rescale" : "w4_gemm256x128_rescale";
                default: return "w4_gemm128_exact";
            }
    }
    return "none";
}

dmr_status_t dmr_probe_empty_launch(int32_t blocks, int32_t threads, size_t lds_bytes, void *stream) {
    if (blocks <= 0 || blocks > (1 << 20) || threads <= 0 || threads > 1024 || threads % 64 != 0 ||
        lds_bytes > 64 * 1024)
        return DMR_ERR_SHAPE;
    return hip_status(dmr::launch_empty_probe(blocks, threads, lds_bytes, static_cast<hipStream_t>(stream)));
}

void dmr_qlinear_destroy(dmr_qlinear_t *layer) { delete layer; }

int32_t dmr_qlinear_bits(const dmr_qlinear_t *layer) { return layer ? layer->bits : 0; }

dmr_status_t dmr_qlinear_shape(const dmr_qlinear_t *layer, int64_t *K, int64_t *N, int32_t *g) {
    if (!layer) return DMR_ERR_NULL;
    if (K) *K = layer->K;
    if (N) *N = layer->N;
    if (g) *g = layer->g;
    return DMR_OK;
}

const char *dmr_status_string(dmr_status_t status) {
    switch (status) {
        case DMR_OK: return "ok";
        case DMR_ERR_NULL: return "a required pointer is NULL";
        case DMR_ERR_SHAPE: return "bad shape";
        case DMR_ERR_ALIGN: return "device pointer not 16-byte aligned";
        case DMR_ERR_WORKSPACE: return "storage or workspace buffer too small";
        case DMR_ERR_UNSUPPORTED: return "unsupported configuration";
        case DMR_ERR_HIP: return "HIP launch failed";
    }
    return "unknown status";
}

}  // extern "C"
