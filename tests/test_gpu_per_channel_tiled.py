"""Per-channel INT4 layers in the tiled GEMMs: whole outputs against fp64 on the codes, in each of the three tile shapes, with
ragged last row and column blocks, one group of K, scales of zero and below the normal range, and rows of infinities."""
import pytest
import torch

import paper_2602_02711_amd as dmr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("M,K,N,path", [
    (513, 128, 4096, "w4_gemm128_rescale"), (600, 1664, 6160, "w4_gemm128_rescale"), (1000, 4096, 4080, "w4_gemm128_rescale"),
    (700, 384, 6160, "w4_gemm256x128_rescale"), (1025, 2048, 4112, "w4_gemm256x128_rescale"),
    (1000, 4096, 8208, "w4_gemm256_rescale"), (2049, 128, 3856, "w4_gemm256_rescale"),
])
def test_per_channel_tiled(M, K, N, path):
    assert dmr.dmr_qlinear_kernel_path(dmr.DMR_FMT_W4_PER_CHANNEL, M, K, N) == path
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + K + N)
    q, s, _ = dmr.dmr_qlinear_quantize(0.02 * torch.randn((N, K), generator=gen, device=DEV), 128)
    codes = ((q.view(N, K // 8, 1) >> (4 * torch.arange(8, device=DEV, dtype=torch.int32))) & 15).reshape(N, K).double() - 8.0
    s = s[:, 0].contiguous()
    s[0], s[17], s[N - 1] = 0.0, 2.0 ** -130, 2.0 ** 40
    layer = dmr.dmr_qlinear_create_per_channel(q, s)
    x = torch.randn((M, K), generator=gen, device=DEV).to(torch.bfloat16)
    res = torch.randn((M, N), generator=gen, device=DEV).to(torch.bfloat16)
    ref = x.double() @ codes.t()
    ws = torch.full((dmr.dmr_qlinear_workspace_bytes(M, K, N),), 0xFF, dtype=torch.uint8, device=DEV)
    y = dmr.dmr_qlinear_forward(layer, x, out_dtype=torch.float32, workspace=ws)
    assert bool((y[:, 0] == 0).all())
    live = torch.arange(N, device=DEV) != 0
    # each column in units of its scale: fp32 sums of K products in units of 16 + q, some five times the result's own; the bound
    # of the tiled class' parity tests
    err = float((y.double()[:, live] / s.double()[live] - ref[:, live]).abs().max() / ref.square().mean().sqrt())
    print(f"{path} M={M} K={K} N={N}: {err:.2e} rms")
    subnormal = 2.0 ** -149 / 2.0 ** -130 / float(ref.square().mean().sqrt())    # half a step of the column of tiny outputs
    assert err <= 1e-4 + subnormal
    assert torch.equal(dmr.dmr_qlinear_forward(layer, x), y.to(torch.bfloat16))
    # two floats a row are all that such a call writes there
    ws = torch.full((8 * M + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    assert torch.equal(dmr.dmr_qlinear_forward(layer, x, out_dtype=torch.float32, workspace=ws[:8 * M]), y)
    assert bool((ws[8 * M:] == 0xA5).all())
    with pytest.raises(dmr.DmrError):
        dmr.dmr_qlinear_forward(layer, x, workspace=ws[:8 * M - 1])
    out = res.clone()
    dmr.dmr_qlinear_forward_fused(layer, dmr.DMR_PRO_NONE, x, residual=out, out=out)
    assert torch.equal(out, (y + res.float()).to(torch.bfloat16))
    x[M - 1, 3], x[5, K - 1] = float("inf"), float("nan")      # such a row alone loses its outputs
    z = dmr.dmr_qlinear_forward(layer, x, out_dtype=torch.float32)
    hit = torch.zeros(M, dtype=torch.bool, device=DEV)
    hit[M - 1] = hit[5] = True
    assert not bool(torch.isfinite(z[hit]).any())
    assert torch.equal(z[~hit], y[~hit])
