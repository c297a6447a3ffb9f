"""The residual of a fused forward is added in fp32 where each kernel stores its result (or in the pass that adds the
partial sums of a split K).  The sum is the one of the plain forward's fp32 output and the residual, so the outputs must
agree with that bit for bit, on every kernel class, for ragged sizes, and with an output over the residual's or the
activations' own buffer."""
import pytest
import torch

import paper_2602_02711_amd as dmr
from paper_2602_02711_amd import synth

pytestmark = pytest.mark.gpu
G = synth.GROUP
DEV = "cuda:0"


def weights(N, K, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return 0.02 * torch.randn((N, K), generator=gen, device=DEV)


def acts(shape, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return torch.randn(shape, generator=gen, device=DEV).to(torch.bfloat16)


def forwards(fmt, w):
    """(plain, fused) forwards of one weight matrix in the named format."""
    if fmt == "bf16":
        wb = w.to(torch.bfloat16)
        return (lambda x, **kw: dmr.dmr_qlinear_bf16_forward(wb, x, **kw),
                lambda *a, **kw: dmr.dmr_qlinear_bf16_forward_fused(wb, *a, **kw))
    if fmt == "w3":
        layer = dmr.dmr_qlinear_w3_create(*dmr.dmr_qlinear_quantize_w3(w, G), G)
    else:
        qw, s, z = dmr.dmr_qlinear_quantize(w, G)
        if fmt == "w4flag":
            s[::64, 0] = 0          # a zero scale: the tiled path leaves these columns to the exact kernel
        layer = dmr.dmr_qlinear_create_per_channel(qw, s[:, 0].contiguous()) if fmt == "w4pc" else \
            dmr.dmr_qlinear_create(qw, s, z, G)
    return (lambda x, **kw: dmr.dmr_qlinear_forward(layer, x, **kw),
            lambda *a, **kw: dmr.dmr_qlinear_forward_fused(layer, *a, **kw))


# M x (K, N): every size class of each format, with M, N off the tile sizes
SHAPES = [(1, 128, 272), (1, 384, 272), (1, 14336, 400), (1, 32768, 528), (2, 384, 272), (7, 2048, 400), (12, 512, 16400),
          (9, 14336, 272), (31, 1024, 272), (33, 512, 16400), (40, 640, 16400), (70, 1024, 528), (129, 1024, 17936), (130, 1152, 144), (300, 512, 6160),
          (900, 512, 2576), (1100, 1024, 8208), (2000, 1280, 13328)]


@pytest.mark.parametrize("fmt", ["w4", "w4pc", "w3", "bf16"])
@pytest.mark.parametrize("M,K,N", SHAPES)
def test_residual_is_added_to_the_fp32_result(fmt, M, K, N):
    plain, fused = forwards(fmt, weights(N, K, 71 + K + N))
    x, res = acts((M, K), 72 + M), acts((M, N), 73 + M)
    want = plain(x, out_dtype=torch.float32) + res.float()
    assert torch.equal(fused(dmr.DMR_PRO_NONE, x, residual=res, out_dtype=torch.float32), want)
    y = fused(dmr.DMR_PRO_NONE, x, residual=res)
    assert torch.equal(y, want.to(torch.bfloat16))
    over = res.clone()                                   # the output over the residual
    fused(dmr.DMR_PRO_NONE, x, residual=over, out=over)
    assert torch.equal(over, y)


@pytest.mark.parametrize("M", [300, 1100])
def test_residual_on_flagged_columns(M):
    K, N = 512, 6160
    plain, fused = forwards("w4flag", weights(N, K, 81))
    x, res = acts((M, K), 82), acts((M, N), 83)
    want = plain(x, out_dtype=torch.float32) + res.float()
    y = fused(dmr.DMR_PRO_NONE, x, residual=res)
    assert torch.equal(y, want.to(torch.bfloat16))
    over = res.clone()                                   # a tile stored twice would add the residual twice
    fused(dmr.DMR_PRO_NONE, x, residual=over, out=over)
    assert torch.equal(over, y)


@pytest.mark.parametrize("fmt", ["w4", "w3", "bf16"])
@pytest.mark.parametrize("M", [40, 200, 700])
def test_output_over_the_activations(fmt, M):
    K = N = 4096
    plain, fused = forwards(fmt, weights(N, K, 91))
    x, res = acts((M, K), 92), acts((M, N), 93)
    want = (plain(x, out_dtype=torch.float32) + res.float()).to(torch.bfloat16)
    y = x.clone()
    fused(dmr.DMR_PRO_NONE, y, residual=res, out=y)
    assert torch.equal(y, want)
