"""Layers of 16384 outputs at 17..64 rows split K in two when the caller brings the partials' workspace, and run unsplit, as
accepted calls, when it does not."""
import pytest
import torch

import paper_2602_02711_amd as dmr
from paper_2602_02711_amd import binding, synth

pytestmark = pytest.mark.gpu
G = synth.GROUP
DEV = "cuda:0"
N = 16384


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("M,K", [(17, 4096), (40, 3072), (64, 4608)])
def test_a_smaller_workspace_is_accepted(bits, M, K):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + K)
    w = 0.02 * torch.randn((N, K), generator=gen, device=DEV)
    x = torch.randn((M, K), generator=gen, device=DEV).to(torch.bfloat16)
    res = torch.randn((M, N), generator=gen, device=DEV).to(torch.bfloat16)
    gamma = torch.rand(K, generator=gen, device=DEV).to(torch.bfloat16)
    layer = dmr.dmr_qlinear_create(*dmr.dmr_qlinear_quantize(w, G), G) if bits == 4 else \
        dmr.dmr_qlinear_w3_create(*dmr.dmr_qlinear_quantize_w3(w, G), G)
    lib = binding.lib()
    want = dmr.dmr_qlinear_forward(layer, x, out_dtype=torch.float32)
    # the two differ in the order of fp32 sums over K products in units of (128 + q), about 20 times the result's own
    bound = 1e-4 * float(want.square().mean().sqrt())
    need = (lib.dmr_qlinear_workspace_bytes if bits == 4 else lib.dmr_qlinear_w3_workspace_bytes)(M, K, N)
    assert need > 0
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device=DEV)
    for ptr, size in ((None, 0), (ws.data_ptr(), 0), (ws.data_ptr(), need - 1)):
        y = torch.full((M, N), float("nan"), device=DEV)
        torch.cuda.synchronize()
        assert lib.dmr_qlinear_forward(layer.handle, x.data_ptr(), M, y.data_ptr(), 1, ptr, size, None) == binding.DMR_OK
        torch.cuda.synchronize()
        assert float((y - want).abs().max()) <= bound

    # fused: what the prologue and the residual take stays required
    full = lib.dmr_qlinear_fused_workspace_bytes(layer.handle, M, 1, 1)
    own = full - need
    ws = torch.full((full,), 0xFF, dtype=torch.uint8, device=DEV)
    ref = dmr.dmr_qlinear_forward_fused(layer, dmr.DMR_PRO_RMSNORM, x, gamma=gamma, eps=1e-6, residual=res, out_dtype=torch.float32)
    y = torch.full((M, N), float("nan"), device=DEV)
    args = (layer.handle, 1, x.data_ptr(), gamma.data_ptr(), 1e-6, res.data_ptr(), M, y.data_ptr(), 1, ws.data_ptr())
    torch.cuda.synchronize()
    assert lib.dmr_qlinear_forward_fused(*args, own - 1, None) == binding.DMR_ERR_WORKSPACE
    assert lib.dmr_qlinear_forward_fused(*args, own, None) == binding.DMR_OK
    torch.cuda.synchronize()
    assert float((y - ref).abs().max()) <= bound


@pytest.mark.parametrize("K,N", [(4096, 6144), (4096, 11008)])
def test_other_split_layers_still_refuse(K, N):
    layer = dmr.dmr_qlinear_create(*dmr.dmr_qlinear_quantize(torch.zeros((N, K), device=DEV), G), G)
    x = torch.zeros((33, K), dtype=torch.bfloat16, device=DEV)
    y = torch.empty((33, N), dtype=torch.bfloat16, device=DEV)
    assert dmr.dmr_qlinear_kernel_path(dmr.DMR_FMT_W4_G128, 33, K, N) == "w4_slices"
    lib = binding.lib()
    assert lib.dmr_qlinear_forward(layer.handle, x.data_ptr(), 33, y.data_ptr(), 0, None, 0, None) == binding.DMR_ERR_WORKSPACE
    assert lib.dmr_qlinear_forward_fused(layer.handle, 0, x.data_ptr(), None, 0.0, None, 33, y.data_ptr(), 0, None, 0,
                                         None) == binding.DMR_ERR_WORKSPACE
