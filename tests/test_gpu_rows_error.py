"""Error of the tile kernel on calls that the rescaling GEMM would have: whole outputs against fp64, rms in units of the result's.  The
group sums are formed on (16 + q) / 2, 8 .. 16, so the fp32 roundings of a group (four MFMAs and the fold, 2^-24 / sqrt(3) of the
running sum each) are sqrt(5) 2^-24 / sqrt(3) 12 / 2.3 = 4e-7 of its result for four bits, whose codes spread by 4.6 / 2, and twice that
for three, and independent over the groups.  On 128 + q they would be 1.8e-6 and 3.7e-6."""
import pytest
import torch

import paper_2602_02711_amd as dmr
from test_gpu_rows import CODE, DEV, make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(129, 128, 8960), (193, 512, 12304), (200, 1024, 10240), (256, 4096, 8976), (400, 384, 6160), (512, 2048, 4608),
                                   (160, 7168, 9216)])
@pytest.mark.parametrize("fmt,bound", [("w4", 4e-7), ("w4pc", 4e-7), ("w3", 8e-7)])
def test_error(fmt, bound, M, K, N):
    assert dmr.dmr_qlinear_kernel_path(CODE[fmt], M, K, N) == fmt[:2] + "_tile"
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + K + N)
    layer, exact = make(fmt, 0.02 * torch.randn((N, K), generator=gen, device=DEV))
    x = torch.randn((M, K), generator=gen, device=DEV).to(torch.bfloat16)
    ref = x.double() @ exact.t()
    y = dmr.dmr_qlinear_forward(layer, x, out_dtype=torch.float32)
    err = float(((y.double() - ref) / ref.square().mean(dim=0).sqrt()).square().mean().sqrt())
    print(f"{fmt} {M} x {K} -> {N}: {err:.2e} rms")
    assert err <= bound
