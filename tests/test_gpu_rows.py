"""The two kernels for 17 rows up to several hundred (staged panels, slices of K), whole outputs against fp64 on the dequantised
codes: every shape that the plan can choose with K whole and split (tests/test_row_plans_cpu.py holds the lists to that), edges of
row and column tiles, group counts that do not divide over waves or splits, fewer groups than waves, rows that share a workgroup's
weights and rows in several blocks."""
import pytest
import torch

import paper_2602_02711_amd as dmr
from paper_2602_02711_amd import synth

pytestmark = pytest.mark.gpu
G = synth.GROUP
DEV = "cuda:0"


def make(fmt, w):
    """(layer, exact weights in fp64)"""
    N, K = w.shape
    if fmt == "w3":
        q, s, z = dmr.dmr_qlinear_quantize_w3(w, G)
        layer = dmr.dmr_qlinear_w3_create(q, s, z, G)
        bits = (q.view(N, K // 32, 3, 1) >> torch.arange(32, device=DEV, dtype=torch.int32)) & 1
        bits = bits.view(N, K // 32, 32, 3)
        codes = bits[..., 0] + 2 * bits[..., 1] + 4 * bits[..., 2]
    else:
        q, s, z = dmr.dmr_qlinear_quantize(w, G)
        codes = (q.view(N, K // 8, 1) >> (4 * torch.arange(8, device=DEV, dtype=torch.int32))) & 15
        if fmt == "w4pc":
            s = (w.abs().amax(dim=1) / 7.5).to(torch.bfloat16)
            return dmr.dmr_qlinear_create_per_channel(q, s), (codes.reshape(N, K).double() - 8.0) * s.double()[:, None]
        layer = dmr.dmr_qlinear_create(q, s, z, G)
    exact = (codes.reshape(N, K // G, G).double() - z.double()[..., None]) * s.double()[..., None]
    return layer, exact.view(N, K)


SLICES = [
    # one, two and four tiles; 1..4 row tiles' worth of rows, one group in all, five, eight and 29 over eight waves
    (17, 128, 1024), (33, 640, 272), (48, 3712, 6144), (64, 384, 8208), (65, 1152, 2064), (100, 128, 272),
    (130, 2560, 4096), (250, 512, 1040), (17, 128, 4320), (32, 2560, 8208),
    # K split, two to sixteen ways
    (17, 4096, 272), (17, 16384, 272), (30, 16384, 640), (33, 3328, 272), (65, 8192, 272), (65, 16384, 272), (49, 3328, 272), (196, 4096, 272),
    (196, 8192, 272),
]
TILE = [
    # chunks of four groups (32, 33 and 35 of them; seven splits of 16), then of two in blocks of 96 and 128 rows
    (20, 4224, 16400), (40, 4480, 16400), (64, 4096, 28688), (50, 14336, 4112), (96, 512, 28688), (97, 384, 17936), (128, 1664, 16400),
    (200, 1664, 12304), (400, 640, 6160), (512, 384, 8192),
    # blocks of 33, 48 and 50 rows with chunks of four
    (65, 1024, 16400), (96, 1536, 16384), (200, 4096, 6160),
    # K split on two and three row tiles and on blocks of 96 and 128 rows; codes in smaller units in blocks of 48 and 64
    (17, 6656, 4320), (322, 4608, 1376), (455, 6144, 2112), (343, 14336, 1376), (129, 384, 9392), (259, 384, 6160),
]
CODE = {"w4": dmr.DMR_FMT_W4_G128, "w4pc": dmr.DMR_FMT_W4_PER_CHANNEL, "w3": dmr.DMR_FMT_W3_G128}


@pytest.mark.parametrize("M,K,N,path", [(*c, "slices") for c in SLICES] + [(*c, "tile") for c in TILE])
@pytest.mark.parametrize("fmt", ["w4", "w4pc", "w3"])
def test_rows(fmt, M, K, N, path):
    assert dmr.dmr_qlinear_kernel_path(CODE[fmt], M, K, N) == fmt[:2] + "_" + path
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + K + N)
    layer, exact = make(fmt, 0.02 * torch.randn((N, K), generator=gen, device=DEV))
    x = torch.randn((M, K), generator=gen, device=DEV).to(torch.bfloat16)
    res = torch.randn((M, N), generator=gen, device=DEV).to(torch.bfloat16)
    ref = x.double() @ exact.t()
    need = (dmr.dmr_qlinear_w3_workspace_bytes if fmt == "w3" else dmr.dmr_qlinear_workspace_bytes)(M, K, N)
    ws = torch.full((max(need, 16),), 0xFF, dtype=torch.uint8, device=DEV)        # NaN partials where nothing was written
    y = dmr.dmr_qlinear_forward(layer, x, out_dtype=torch.float32, workspace=ws)
    # fp32 sums of K products in units of (128 + q) ~ 20 times the result's own: the bound of this kernel class' parity tests
    assert float((y.double() - ref).abs().max()) <= 1e-4 * float(ref.square().mean().sqrt())
    # bf16 output, and a residual in the output's own buffer: the same fp32 sums, rounded once
    assert torch.equal(dmr.dmr_qlinear_forward(layer, x), y.to(torch.bfloat16))
    out = res.clone()
    dmr.dmr_qlinear_forward_fused(layer, dmr.DMR_PRO_NONE, x, residual=out, out=out)
    assert torch.equal(out, (y + res.float()).to(torch.bfloat16))
