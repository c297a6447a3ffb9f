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


@pytest.mark.parametrize("M,K,N,path", [
    # 2..8 rows: short rows on any width, up to 4096 outputs, up to 8192, and 8192 itself at K = 2048 and 4096
    (2, 896, 8208, "skinny"), (2, 1024, 8208, "rows"), (5, 896, 12288, "skinny"), (5, 1024, 12288, "rows"), (7, 768, 9216, "skinny"),
    (7, 896, 9216, "rows"), (8, 640, 8208, "skinny"), (8, 768, 8208, "rows"), (3, 1024, 16384, "skinny"), (3, 1024, 16368, "rows"),
    (4, 2560, 4096, "skinny"), (4, 2688, 4096, "rows"), (6, 1792, 4096, "skinny"), (6, 1920, 4096, "rows"), (8, 1536, 4096, "skinny"),
    (8, 1664, 4096, "rows"), (4, 1536, 8192, "skinny"), (4, 1664, 8192, "rows"), (7, 1280, 4112, "skinny"), (7, 1408, 4112, "rows"),
    (8, 768, 8192, "skinny"), (8, 896, 8192, "rows"), (2, 4096, 8192, "skinny"), (2, 4096, 8128, "rows"), (4, 2048, 8144, "skinny"),
    (4, 2560, 8192, "rows"), (8, 8192, 4096, "rows"), (8, 8320, 4096, "skinny"),          # 64 groups held
    # 9..64 rows up to K = 512
    (16, 512, 4096, "rows"), (16, 512, 4112, "mid"), (16, 512, 16384, "mid"), (16, 512, 16400, "rows"), (16, 640, 8192, "rows"),
    (16, 256, 4096, "rows"), (16, 256, 16400, "skinny"), (32, 256, 4096, "mid"), (33, 256, 4096, "rows"), (64, 256, 20480, "mid"),
    (32, 384, 4096, "rows"), (32, 512, 9216, "mid"), (64, 512, 16400, "rows"), (64, 640, 9216, "rows"),
    # 33..64 rows: one full round of the other kernel with K in four, in two here
    (64, 4096, 4096, "mid"), (33, 4096, 3600, "mid"), (64, 4096, 3584, "rows"), (64, 4096, 4112, "rows"), (64, 4608, 4096, "rows"),
    (32, 4096, 4096, "rows"), (64, 8192, 4096, "rows"), (64, 14336, 28672, "mid"),        # two splits held, seven needed
])
def test_bf16_rows_crossover(M, K, N, path):
    assert binding.lib().dmr_qlinear_kernel_path(BF16, M, K, N).decode() == "bf16_" + path
