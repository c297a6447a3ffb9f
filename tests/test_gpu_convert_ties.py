"""Quantisers at the edges of their fp32 rounding shortcut: quotients on and next to ties, scales at both ends of the fp32
range and beyond the shortcut's, against the oracle's 64-bit arithmetic, bit for bit; and ragged block counts of both."""
import numpy as np
import pytest
import torch

import paper_2602_02711_amd as dmr
from oracle import cpu_oracle as orc
from paper_2602_02711_amd import synth
from gpu_util import bf16_dev, bits_host, u32_dev

pytestmark = pytest.mark.gpu
G = synth.GROUP


def tie_weights(top: int, N: int, K: int) -> np.ndarray:
    """Rows whose groups have scale 2^e (or a fraction of it above 1), with weights on ties and up to three ulps beside them."""
    rng = np.random.default_rng(7700 + top + K)
    w = np.empty((N, K), dtype=np.float32)
    exps = [-146, -140, -133, -126, -101, -100, -99, -20, -6, 0, 3, 99, 100, 101, 118]
    for n in range(N):
        for b in range(K // G):
            i = n * (K // G) + b
            s = np.float32(2.0) ** exps[i % len(exps)] * np.float32(1.0 + (i // len(exps)) % 128 / 128.0)
            low = int(rng.integers(0, top + 1))
            half = rng.integers(-2 * low, 2 * (top - low) + 1, size=G)       # multiples of s / 2: codes and ties
            v = (half.astype(np.float64) * 0.5 * float(s)).astype(np.float32)
            for _ in range(3):
                step = rng.integers(-1, 2, size=G)
                v = np.where(step > 0, np.nextafter(v, np.float32(np.inf)), np.where(step < 0, np.nextafter(v, np.float32(-np.inf)), v))
            v[5], v[77] = np.float32(-low * float(s)), np.float32((top - low) * float(s))
            w[n, b * G:(b + 1) * G] = v
    return w


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("K,N", [(128, 16), (384, 48), (1024, 1040)])
def test_quantise_on_and_beside_ties(K, N, bits):
    w = tie_weights(2 ** bits - 1, N, K)
    wd = torch.from_numpy(w).to("cuda:0")
    q_ref, s_ref, z_ref = orc.quantize_bits(w, G, bits)
    if bits == 4:
        qw, s, z = dmr.dmr_qlinear_quantize(wd, G)
        layer, ref, deq = dmr.dmr_qlinear_create(qw, s, z, G), orc.pack(q_ref), orc.dequantize
    else:
        qw, s, z = dmr.dmr_qlinear_quantize_w3(wd, G)
        layer, ref, deq = dmr.dmr_qlinear_w3_create(qw, s, z, G), orc.pack3(q_ref), orc.dequantize3
    got = bits_host(dmr.dmr_qlinear_dequantize(layer))
    assert np.array_equal(bits_host(s), s_ref)
    assert np.array_equal(bits_host(z), z_ref)
    assert np.array_equal(qw.cpu().numpy().view(np.uint32), ref)
    assert np.array_equal(got, deq(ref, s_ref, z_ref, G))


@pytest.mark.parametrize("K,N", [(128, 16), (384, 48), (1920, 272)])
def test_per_channel_dequantise_of_ragged_block_counts(K, N):
    q = np.random.default_rng(7800 + K).integers(0, 16, size=(N, K)).astype(np.uint8)
    s = synth.to_bf16_bits(np.abs(synth.weights_f32(7801 + K, N, 1)) + np.float32(1e-3))
    words = orc.pack(q)
    layer = dmr.dmr_qlinear_create_per_channel(u32_dev(words), bf16_dev(s.reshape(N)))
    got = bits_host(dmr.dmr_qlinear_dequantize(layer))
    z = synth.to_bf16_bits(np.full((N, K // G), 8.0, dtype=np.float32))
    assert np.array_equal(got, orc.dequantize(words, np.repeat(s.reshape(N, 1), K // G, axis=1), z, G))
