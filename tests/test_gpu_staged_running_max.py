"""Staged output projection with the running maximum: the maximum rising, falling and jumping from block to block of 32 words, and
whole runs of blocks masked (words of probability 0), in front of the first unmasked one too."""
import numpy as np
import pytest

import paper_2007_11794_amd as rn
from workloads import round_to_bf16

from harness import gpu_step, load_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", ["rising", "falling", "jumping"])
@pytest.mark.parametrize("H,V,B", [(64, 16500, 130), (190, 33000, 200), (250, 3000, 257), (512, 25000, 140), (704, 17000, 300)])
def test_maximum_moves_between_blocks(H, V, B, shape):
    rng = np.random.default_rng(H * 1009 + V)
    model = {"U": rng.normal(0, 0.3, (V, H)), "W": rng.normal(0, 1 / np.sqrt(H), (H, H)), "O": rng.normal(0, 2 / np.sqrt(H), (H, V))}
    model = {k: round_to_bf16(v.astype(np.float32)) for k, v in model.items()}
    block = np.arange(V) // 32
    at = {"rising": block / block[-1], "falling": 1 - block / block[-1], "jumping": rng.random(block[-1] + 1)[block]}[shape]
    bias = (300 * at + rng.normal(0, 0.5, V)).astype(np.float32)
    masked = (block < 7) | (block % 11 == 3) | (block > block[-1] - 3)
    bias[masked] = -np.inf
    model["bias"] = bias
    m = load_model(model, "bf16", B)
    m.set_option(rn.OPT_LSE_MODE, 1)
    assert m.outproj_kernel_name(B) == "outproj_staged_kernel"
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    query = rng.choice(np.flatnonzero(~masked), (B, 2)).astype(np.int32)
    h, lp = gpu_step(m, prev, h_in, query)
    assert m.last_error() == 0
    m.close()
    # what the kernel computes, in float64: the rows enter the normaliser as bf16 numbers, times log2(e) where that is folded in
    scale = np.log2(np.e) if -(-max(H, 128) // 64) * 64 in (128, 256, 512) else 1.0
    d = round_to_bf16((h - np.float32(0.5)) * np.float32(scale)).astype(np.float64) / scale
    O = model["O"].astype(np.float64)
    z = d @ O + (bias.astype(np.float64) + 0.5 * O.sum(0))
    top = z.max(1, keepdims=True)
    ref = np.take_along_axis(h.astype(np.float64) @ O + bias, query, 1) - top - np.log(np.exp(z - top).sum(1, keepdims=True))
    # numbers up to 300 (433 in base 2) are rounded half a dozen times on the way: 2^-24 * 512 each, and as in the plain case 1e-4
    assert np.max(np.abs(lp - ref)) <= 1e-4 + 6 * 2.0 ** -15
