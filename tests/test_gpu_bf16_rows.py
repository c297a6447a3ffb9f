"""The bf16 kernel for 2..64 rows that keeps its activations in registers, whole outputs against fp64: every row-tile count and
number of groups per wave, group counts that leave waves short or idle, ragged rows and runs of tiles, K whole and split."""
import pytest
import torch

import paper_2602_02711_amd as dmr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("M,K,N", [
    # groups per wave 1 to 8; fewer groups than waves; one tile and several to a workgroup
    (8, 896, 8208), (3, 1152, 8208), (8, 2688, 1040), (9, 128, 272), (16, 4096, 4128), (5, 5632, 528), (12, 8192, 528), (16, 4608, 528), (7, 6656, 1040),
    (17, 896, 1040), (32, 1920, 4112), (20, 2944, 8208), (31, 3584, 528), (32, 4096, 12304),
    (33, 1024, 4112), (48, 1152, 272), (49, 896, 4112), (64, 2048, 8208),
    # K split
    (16, 11008, 1040), (32, 14336, 4112), (64, 4096, 6160), (40, 5120, 5136),
])
def test_bf16_rows(M, K, N):
    assert dmr.dmr_qlinear_kernel_path(dmr.DMR_FMT_BF16, M, K, N) == "bf16_rows"
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + K + N)
    w = (0.02 * torch.randn((N, K), generator=gen, device=DEV)).to(torch.bfloat16)
    x = torch.randn((M, K), generator=gen, device=DEV).to(torch.bfloat16)
    res = torch.randn((M, N), generator=gen, device=DEV).to(torch.bfloat16)
    ref = x.double() @ w.double().t()
    ws = torch.full((max(dmr.dmr_qlinear_bf16_workspace_bytes(M, K, N), 16),), 0xFF, dtype=torch.uint8, device=DEV)
    y = dmr.dmr_qlinear_bf16_forward(w, x, out_dtype=torch.float32, workspace=ws)
    # K products in fp32, at most K / 8 of them in one chain: sqrt(K) roundings of 2^-24 of a running sum of the result's size
    assert float((y.double() - ref).abs().max()) <= 1e-5 * float(ref.square().mean().sqrt())
    assert torch.equal(dmr.dmr_qlinear_bf16_forward(w, x), y.to(torch.bfloat16))
    out = res.clone()
    dmr.dmr_qlinear_bf16_forward_fused(w, dmr.DMR_PRO_NONE, x, residual=out, out=out)
    assert torch.equal(out, (y + res.float()).to(torch.bfloat16))


@pytest.mark.parametrize("M,K,N", [(2, 3072, 8208), (8, 4096, 6144), (16, 4096, 28672), (3, 5120, 5120)])
def test_error_up_to_16_rows(M, K, N):
    # rms against fp64, of the result's: sixteen chains of K / 512 MFMAs, measured 1.0e-7 .. 1.17e-7; with eight chains 1.2e-7 .. 1.54e-7
    assert dmr.dmr_qlinear_kernel_path(dmr.DMR_FMT_BF16, M, K, N) == "bf16_rows"
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + K + N)
    w = (0.02 * torch.randn((N, K), generator=gen, device=DEV)).to(torch.bfloat16)
    errs, refs = 0.0, 0.0
    for _ in range(8):
        x = torch.randn((M, K), generator=gen, device=DEV).to(torch.bfloat16)
        ref = x.double() @ w.double().t()
        errs += float((dmr.dmr_qlinear_bf16_forward(w, x, out_dtype=torch.float32).double() - ref).square().mean())
        refs += float(ref.square().mean())
    assert (errs / refs) ** 0.5 <= (1.1e-7 if K == 3072 else 1.25e-7)
