"""Calls of 17..64 rows and their workspace: layers of more than 32768 outputs split K when the caller brings the partials' memory and
run unsplit, as accepted calls, when it does not; layers that stay whole need none; other split layers refuse."""
import pytest
import torch

import paper_2602_02711_amd as dmr
from paper_2602_02711_amd import binding, synth
from test_gpu_rows import make

pytestmark = pytest.mark.gpu
G = synth.GROUP
DEV = "cuda:0"


@pytest.mark.parametrize("fmt", ["w4", "w3"])
@pytest.mark.parametrize("M,K,N", [(33, 6912, 33216), (49, 7936, 33216)])
def test_a_smaller_workspace_is_accepted(fmt, M, K, N):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + K)
    layer, exact = make(fmt, 0.02 * torch.randn((N, K), generator=gen, device=DEV))
    x = torch.randn((M, K), generator=gen, device=DEV).to(torch.bfloat16)
    res = torch.randn((M, N), generator=gen, device=DEV).to(torch.bfloat16)
    gamma = torch.rand(K, generator=gen, device=DEV).to(torch.bfloat16)
    lib = binding.lib()
    ref = x.double() @ exact.t()
    # fp32 sums of K products in units of (128 + q) ~ 20 times the result's own: the bound of this kernel class' parity tests
    bound = 1e-4 * float(ref.square().mean().sqrt())
    need = (lib.dmr_qlinear_workspace_bytes if fmt == "w4" else lib.dmr_qlinear_w3_workspace_bytes)(M, K, N)
    assert need == 2 * 4 * M * N
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device=DEV)
    split = dmr.dmr_qlinear_forward(layer, x, out_dtype=torch.float32, workspace=ws)
    assert float((split.double() - ref).abs().max()) <= bound
    for ptr, size in ((None, 0), (ws.data_ptr(), 0), (ws.data_ptr(), need - 1)):
        y = torch.full((M, N), float("nan"), device=DEV)
        torch.cuda.synchronize()
        assert lib.dmr_qlinear_forward(layer.handle, x.data_ptr(), M, y.data_ptr(), 1, ptr, size, None) == binding.DMR_OK
        torch.cuda.synchronize()
        assert float((y.double() - ref).abs().max()) <= bound
        assert not torch.equal(y, split)              # another order of the sums: K stayed whole

    # fused: what the prologue and the residual take stays required
    full = lib.dmr_qlinear_fused_workspace_bytes(layer.handle, M, 1, 1)
    own = full - need
    ws = torch.full((full,), 0xFF, dtype=torch.uint8, device=DEV)
    xg = dmr.dmr_glue_rmsnorm(x, gamma, 1e-6)
    ref = xg.double() @ exact.t() + res.double()
    y = torch.full((M, N), float("nan"), device=DEV)
    args = (layer.handle, 1, x.data_ptr(), gamma.data_ptr(), 1e-6, res.data_ptr(), M, y.data_ptr(), 1, ws.data_ptr())
    torch.cuda.synchronize()
    assert lib.dmr_qlinear_forward_fused(*args, own - 1, None) == binding.DMR_ERR_WORKSPACE
    assert lib.dmr_qlinear_forward_fused(*args, own, None) == binding.DMR_OK
    torch.cuda.synchronize()
    assert float((y.double() - ref).abs().max()) <= bound


@pytest.mark.parametrize("fmt", ["w4", "w3"])
@pytest.mark.parametrize("M,K,N", [(33, 4096, 6144), (33, 4096, 11008), (40, 3072, 16384), (30, 640, 16400)])
def test_whole_layers_need_none(fmt, M, K, N):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + K)
    layer, exact = make(fmt, 0.02 * torch.randn((N, K), generator=gen, device=DEV))
    x = torch.randn((M, K), generator=gen, device=DEV).to(torch.bfloat16)
    y = torch.full((M, N), float("nan"), device=DEV)
    lib = binding.lib()
    assert (lib.dmr_qlinear_workspace_bytes if fmt == "w4" else lib.dmr_qlinear_w3_workspace_bytes)(M, K, N) == 0
    torch.cuda.synchronize()
    assert lib.dmr_qlinear_forward(layer.handle, x.data_ptr(), M, y.data_ptr(), 1, None, 0, None) == binding.DMR_OK
    torch.cuda.synchronize()
    ref = x.double() @ exact.t()
    assert float((y.double() - ref).abs().max()) <= 1e-4 * float(ref.square().mean().sqrt())


@pytest.mark.parametrize("M,K,N", [(33, 14336, 4096), (50, 14336, 4112)])
def test_other_split_layers_still_refuse(M, K, N):
    layer = dmr.dmr_qlinear_create(*dmr.dmr_qlinear_quantize(torch.zeros((N, K), device=DEV), G), G)
    x = torch.zeros((M, K), dtype=torch.bfloat16, device=DEV)
    y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    lib = binding.lib()
    assert lib.dmr_qlinear_workspace_bytes(M, K, N) > 0
    assert lib.dmr_qlinear_forward(layer.handle, x.data_ptr(), M, y.data_ptr(), 0, None, 0, None) == binding.DMR_ERR_WORKSPACE
    assert lib.dmr_qlinear_forward_fused(layer.handle, 0, x.data_ptr(), None, 0.0, None, M, y.data_ptr(), 0, None, 0,
                                         None) == binding.DMR_ERR_WORKSPACE
