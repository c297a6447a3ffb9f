"""The eight-wave bf16 kernel on its three tile heights.  Weights and activations are small integers: every product and
every partial sum is exact in fp32 whatever the order (|sum| <= K * 16 * 8 < 2^24), so the result must equal the reference
(the same product in fp32 by the host) bit for bit, ragged last tiles and the store of the residual included."""
import pytest
import torch

import paper_2602_02711_amd as dmr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("K,N,M,path", [
    (1024, 3856, 2890, "bf16_gemm192x256"),      # 16 x 16 tiles, 10 rows and 16 columns in the last ones
    (1152, 4096, 3072, "bf16_gemm192x256"),      # whole tiles, nine groups of 128
    (1024, 4096, 2048, "bf16_gemm128x256"),      # exactly one round of 128-row tiles
    (1152, 3600, 1930, "bf16_gemm128x256"),      # ragged both ways, an odd number of tiles (no XCD-even grid)
    (1024, 4080, 3843, "bf16_gemm256"),          # 16 x 16 tiles, 3 rows in the last row tile
    (1024, 1040, 13000, "bf16_gemm256"),         # 51 x 5 tiles: bands of four tile rows, the last of three
])
def test_exact_integers(K, N, M, path):
    assert dmr.dmr_qlinear_kernel_path(dmr.DMR_FMT_BF16, M, K, N) == path
    gen = torch.Generator().manual_seed(K + N + M)
    w = torch.randint(-16, 17, (N, K), generator=gen).float()
    x = torch.randint(-8, 9, (M, K), generator=gen).float()
    res = torch.randint(-100, 101, (M, N), generator=gen).float()
    want = x @ w.t()
    wd, xd = w.to(torch.bfloat16).to(DEV), x.to(torch.bfloat16).to(DEV)
    assert torch.equal(dmr.dmr_qlinear_bf16_forward(wd, xd, out_dtype=torch.float32).cpu(), want)
    rd = res.to(torch.bfloat16).to(DEV)
    got = dmr.dmr_qlinear_bf16_forward_fused(wd, dmr.DMR_PRO_NONE, xd, residual=rd, out_dtype=torch.float32)
    assert torch.equal(got.cpu(), want + res)
    y = dmr.dmr_qlinear_bf16_forward_fused(wd, dmr.DMR_PRO_NONE, xd, residual=rd)
    assert torch.equal(y.cpu(), (want + res).to(torch.bfloat16))
    dmr.dmr_qlinear_bf16_forward_fused(wd, dmr.DMR_PRO_NONE, xd, residual=rd, out=rd)     # over the residual
    assert torch.equal(rd, y)
