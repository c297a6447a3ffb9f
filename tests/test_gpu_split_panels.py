"""17..64 rows of layers too narrow to give every CU 128 columns, K split over workgroups or whole as the plan has it: whole outputs
against fp64 on the dequantised codes, uneven last split, ragged rows and columns, every row-tile count."""
import pytest
import torch

import paper_2602_02711_amd as dmr
from paper_2602_02711_amd import synth

pytestmark = pytest.mark.gpu
G = synth.GROUP
DEV = "cuda:0"


@pytest.mark.parametrize("fmt", ["w4", "w3"])
@pytest.mark.parametrize("M,K,N,path", [(17, 14336, 4096, "slices"), (33, 14336, 4112, "tile"), (64, 11264, 2704, "slices"),
                                        (48, 4096, 6144, "slices"), (32, 2560, 8208, "slices")])
def test_split_panels(fmt, M, K, N, path):
    code = dmr.DMR_FMT_W4_G128 if fmt == "w4" else dmr.DMR_FMT_W3_G128
    assert dmr.dmr_qlinear_kernel_path(code, M, K, N) == fmt + "_" + path
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + K + N)
    w = 0.02 * torch.randn((N, K), generator=gen, device=DEV)
    x = torch.randn((M, K), generator=gen, device=DEV).to(torch.bfloat16)
    if fmt == "w4":
        q, s, z = dmr.dmr_qlinear_quantize(w, G)
        layer = dmr.dmr_qlinear_create(q, s, z, G)
        codes = (q.view(N, K // 8, 1) >> (4 * torch.arange(8, device=DEV, dtype=torch.int32))) & 15
    else:
        q, s, z = dmr.dmr_qlinear_quantize_w3(w, G)
        layer = dmr.dmr_qlinear_w3_create(q, s, z, G)
        bits = (q.view(N, K // 32, 3, 1) >> torch.arange(32, device=DEV, dtype=torch.int32)) & 1
        bits = bits.view(N, K // 32, 32, 3)
        codes = bits[..., 0] + 2 * bits[..., 1] + 4 * bits[..., 2]
    exact = (codes.reshape(N, K // G, G).double() - z.double()[..., None]) * s.double()[..., None]
    ref = x.double() @ exact.view(N, K).t()
    need = (dmr.dmr_qlinear_workspace_bytes if fmt == "w4" else dmr.dmr_qlinear_w3_workspace_bytes)(M, K, N)
    assert need <= 8 << 20
    ws = torch.full((max(need, 16),), 0xFF, dtype=torch.uint8, device=DEV)        # NaN partials where nothing was written
    y = dmr.dmr_qlinear_forward(layer, x, out_dtype=torch.float32, workspace=ws)
    # fp32 sums of K products in units of (128 + q) ~ 20 times the result's own: the bound of this kernel class' parity tests
    assert float((y.double() - ref).abs().max()) <= 1e-4 * float(ref.square().mean().sqrt())
