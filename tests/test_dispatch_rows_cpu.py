"""Dispatch of the row kernels, on the host: where their classes begin and end, and what those calls ask for."""
import pytest

from paper_2602_02711_amd import binding

W4, PC, W3, BF16 = (binding.DMR_FMT_W4_G128, binding.DMR_FMT_W4_PER_CHANNEL, binding.DMR_FMT_W3_G128, binding.DMR_FMT_BF16)


@pytest.mark.parametrize("M,K,N,path,asks", [
    (400, 4096, 6144, "tile", False), (512, 4096, 8192, "tile", False),                    # 192 and 256 blocks of 128 x 128: one round
    (513, 4096, 6144, "gemm128_rescale", True), (400, 4096, 16384, "gemm256x128_rescale", True),
])
def test_quantised_rows(M, K, N, path, asks):
    lib = binding.lib()
    for fmt, name in ((W4, "w4_"), (PC, "w4_"), (W3, "w3_")):
        assert lib.dmr_qlinear_kernel_path(fmt, M, K, N).decode() == name + path
    assert (lib.dmr_qlinear_workspace_bytes(M, K, N) > 0) == asks
    assert (lib.dmr_qlinear_w3_workspace_bytes(M, K, N) > 0) == asks


@pytest.mark.parametrize("M,K,N,rows", [
    (1, 4096, 4096, False), (2, 4096, 28672, True), (16, 4096, 28672, True), (17, 4096, 4096, True), (64, 14336, 4096, True),
    (65, 4096, 4096, False), (8, 1024, 1024, False),                                     # a small layer at up to eight rows
])
def test_bf16_rows(M, K, N, rows):
    assert (binding.lib().dmr_qlinear_kernel_path(BF16, M, K, N) == b"bf16_rows") == rows
