"""Which kernel class serves a shape, on both sides of the measured crossovers (host arithmetic only)."""
import pytest

from paper_2602_02711_amd import binding


@pytest.fixture(scope="module")
def lib():
    return binding.lib()


def bf16_path(lib, M, K, N):
    return lib.dmr_qlinear_kernel_path(binding.DMR_FMT_BF16, M, K, N)


@pytest.mark.parametrize("M,K,N,tiled", [
    (200, 2048, 4096, False), (200, 2048, 4224, True),          # 64 / 66 blocks of 128 x 128, K split twice
    (200, 4096, 4608, False), (384, 4096, 3072, False),         # 72 blocks, K split four ways: 48 / 50 us
    (200, 4096, 6144, True), (512, 4096, 4096, True),           # 96 and 128 blocks
    (200, 8192, 4608, False), (384, 8192, 3072, False),         # 72 blocks: 76 / 85 us
    (200, 8192, 6144, True),                                    # 96 blocks
    (200, 6144, 6144, False), (200, 11264, 8192, False),        # 96 and 128 blocks of longer rows
    (200, 6144, 8320, True), (200, 14336, 8320, True),          # 130 blocks
    (450, 4096, 3328, True),                                    # five row blocks of 96 x 26 column blocks
    (200, 8064, 6144, True),                                    # 63 groups: the rollout-batch kernel cannot split K
    (200, 512, 8192, False), (200, 512, 8320, True),            # K < 1024: 128 / 130 blocks
])
def test_bf16_crossover(lib, M, K, N, tiled):
    assert (bf16_path(lib, M, K, N) != b"bf16_mid") == tiled


@pytest.mark.parametrize("K", [512, 1024, 2048, 4096, 5120, 8064, 8192, 11264, 14336])
@pytest.mark.parametrize("M", [70, 128, 200, 450, 512, 1000])
def test_bf16_crossover_has_no_holes(lib, M, K):
    tiled = [bf16_path(lib, M, K, N) != b"bf16_mid" for N in range(128, 24576, 128)]
    assert tiled == sorted(tiled)


@pytest.mark.parametrize("M,K,N,name", [
    (700, 4096, 6144, "bf16_gemm128_dma"), (1400, 4096, 3072, "bf16_gemm128_dma"),     # column blocks divide by the XCDs
    (600, 8192, 8192, "bf16_gemm128_dma"), (1020, 4096, 5120, "bf16_gemm128_dma"),
    (1240, 4096, 5120, "bf16_gemm128_dma"), (1200, 4096, 6144, "bf16_gemm128x256"),    # 400 and 480 blocks
    (1436, 8192, 4096, "bf16_gemm128x256"), (1531, 8192, 4096, "bf16_gemm128_dma"),    # the last row block half empty / full
    (900, 4096, 6000, "bf16_gemm128x256"), (4300, 4096, 1024, "bf16_gemm128x256"),     # 47 column blocks; a tall layer
    (400, 4096, 16384, "bf16_gemm128x256"),                                            # four row blocks
    (1300, 4096, 28672, "bf16_gemm256"), (1642, 8192, 14864, "bf16_gemm256"),
    (4300, 8192, 16384, "bf16_gemm256"), (4300, 4096, 16384, "bf16_gemm192x256"),
    (100000, 4096, 384, "bf16_gemm256"), (200000, 4096, 128, "bf16_gemm128_dma"),
    (3000, 4096, 6144, "bf16_gemm192x256"), (2000, 4096, 4096, "bf16_gemm128x256"),
    (1024, 4096, 4096, "bf16_gemm128_dma"), (8192, 4096, 4096, "bf16_gemm256"),
])
def test_bf16_tile(lib, M, K, N, name):
    assert bf16_path(lib, M, K, N).decode() == name


@pytest.mark.parametrize("M,K,N,rows,splits", [
    (33, 1536, 12288, "slices", 1), (64, 4096, 6144, "slices", 1), (64, 8192, 8192, "slices", 1), (17, 4096, 11008, "slices", 1),
    (17, 12288, 2048, "slices", 4), (64, 12288, 2048, "slices", 4), (33, 7168, 4096, "slices", 4), (64, 14336, 4096, "slices", 4),
    (50, 14336, 4112, "tile", 7), (64, 4096, 28672, "tile", 1), (400, 4096, 6144, "tile", 1),
    # 1024 row tiles and more: whole up to 32768 outputs; those that split also run without the partials
    (17, 11264, 16384, "slices", 1), (17, 11008, 16384, "slices", 1), (33, 4096, 16384, "slices", 1), (64, 14336, 16384, "slices", 1), (33, 6912, 33216, "tile", 2),
])
def test_rows_kernel_and_splits(lib, M, K, N, rows, splits):
    # the workspace is the partials of the splits that the launch makes, nothing where K stays whole
    need = 4 * splits * M * N if splits > 1 else 0
    for fmt, name in ((binding.DMR_FMT_W4_G128, "w4_"), (binding.DMR_FMT_W3_G128, "w3_")):
        assert lib.dmr_qlinear_kernel_path(fmt, M, K, N).decode() == name + rows
    assert lib.dmr_qlinear_workspace_bytes(M, K, N) == need
    assert lib.dmr_qlinear_w3_workspace_bytes(M, K, N) == need


@pytest.mark.parametrize("M,K,N,splits", [
    (32, 4096, 4096, 1), (17, 4096, 28672, 1), (32, 14336, 4096, 4), (64, 4096, 28672, 2), (64, 14336, 4096, 7), (64, 2048, 4096, 1),
])
def test_bf16_rows_splits(lib, M, K, N, splits):
    assert bf16_path(lib, M, K, N) == b"bf16_rows"
    assert lib.dmr_qlinear_bf16_workspace_bytes(M, K, N) == (4 * splits * M * N if splits > 1 else 0)


def test_partials_of_64_rows_fit_the_fixed_scratch(lib):
    for M in (17, 33, 42, 43, 48, 64):
        for K in range(128, 28672, 128):
            for N in (272, 1024, 2704, 4096, 4112, 6144, 8208, 11008, 12288, 16368):
                assert lib.dmr_qlinear_workspace_bytes(M, K, N) <= binding.DMR_STATIC_SCRATCH_BYTES, (M, K, N)
