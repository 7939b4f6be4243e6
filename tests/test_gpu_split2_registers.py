"""Two-term fp32 output projection with the rows in registers (padded hidden sizes of 128 to 576), against the oracle and the
form that takes rows through LDS: rows around its groups of 256 (from 384 on 128) and 32, vocabularies that end inside a block, a stage and a split, words many powers of
two apart, a maximum that moves from block to block, words of probability 0, row counts known on the device only."""
import numpy as np
import pytest

import oracle
import paper_2007_11794_amd as rn

from harness import gpu_step, gpu_step_dedup, load_model
from test_gpu_split2 import model_of

pytestmark = pytest.mark.gpu

SIZES = [(3, 70, 65), (255, 128, 128), (16500, 100, 300), (8300, 190, 129), (33000, 150, 255), (700, 200, 257), (25000, 256, 140),
         (1000, 256, 8300), (513, 257, 100), (12500, 320, 513), (41000, 300, 161), (16500, 350, 300), (8300, 448, 129), (25000, 512, 140), (700, 500, 257), (300, 512, 8300),
         (33000, 570, 65), (17000, 350, 1300), (16400, 450, 2100)]


@pytest.mark.parametrize("V,H,B", SIZES)
def test_against_the_oracle_and_the_other_form(V, H, B):
    rng = np.random.default_rng(V + B)
    model = model_of(rng, V, H, 1.0)
    m = load_model(model, "f32", B)
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    query = rng.integers(0, V, (B, 2)).astype(np.int32)
    ref = oracle.step(model, prev, h_in, query)
    # fp32 sums of H products: 2^-24 of the running sum per addition at worst, running sums below the sum of |O| / 2
    tol = 1e-5 + 2.0 ** -24 * np.sqrt(H) * 0.5 * np.abs(model["O"]).sum(0).max()
    for lse_mode in (0, 1):
        m.set_option(rn.OPT_LSE_MODE, lse_mode)
        by_form = []
        for kernel in (0, 4):
            m.set_option(rn.OPT_OUTPROJ_KERNEL, kernel)
            assert m.outproj_kernel_name(B) == ("outproj_split2_kernel" if kernel else "outproj_staged_f32_kernel")
            h, lp = gpu_step(m, prev, h_in, query)
            assert np.max(np.abs(h - ref["h_out"])) <= 1e-5
            assert np.max(np.abs(lp - ref["logprob"])) <= tol, (kernel, lse_mode)
            by_form.append(lp)
        # the same products and accumulators; what differs is the order of the sums over words
        assert np.max(np.abs(by_form[0] - by_form[1])) <= 1e-5
    # few of the rows distinct: the row count is then known on the device only
    m.set_option(rn.OPT_OUTPROJ_KERNEL, 0)
    for few in (max(1, B // 9), max(1, B // 2)):
        src = rng.integers(0, few, B)
        out = gpu_step_dedup(m, src.astype(np.uint64) + 5, prev[src], h_in[src], query)
        ref = oracle.step(model, prev[src], h_in[src], query)
        assert np.max(np.abs(out["logprob"] - ref["logprob"])) <= tol
    assert m.last_error() == 0
    m.close()


@pytest.mark.parametrize("shape", ["rising", "falling", "jumping"])
@pytest.mark.parametrize("V,H,B", [(16500, 128, 130), (33000, 190, 200), (3000, 250, 257), (17000, 320, 300), (9000, 500, 200)])
def test_maximum_moves_between_blocks(V, H, B, shape):
    rng = np.random.default_rng(H * 1009 + V)
    model = {"U": rng.normal(0, 0.3, (V, H)), "W": rng.normal(0, 1 / np.sqrt(H), (H, H)), "O": rng.normal(0, 2 / np.sqrt(H), (H, V))}
    model = {k: v.astype(np.float32) for k, v in model.items()}
    block = np.arange(V) // 32
    at = {"rising": block / block[-1], "falling": 1 - block / block[-1], "jumping": rng.random(block[-1] + 1)[block]}[shape]
    bias = (300 * at + rng.normal(0, 0.5, V)).astype(np.float32)
    masked = (block < 7) | (block % 11 == 3) | (block > block[-1] - 3)
    bias[masked] = -np.inf
    model["bias"] = bias
    m = load_model(model, "f32", B)
    m.set_option(rn.OPT_LSE_MODE, 1)
    assert m.outproj_kernel_name(B) == "outproj_staged_f32_kernel"
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    query = rng.choice(np.flatnonzero(~masked), (B, 2)).astype(np.int32)
    h, lp = gpu_step(m, prev, h_in, query)
    assert m.last_error() == 0
    m.close()
    z = h.astype(np.float64) @ model["O"].astype(np.float64) + bias.astype(np.float64)
    top = z.max(1, keepdims=True)
    ref = np.take_along_axis(z, query, 1) - top - np.log(np.exp(z - top).sum(1, keepdims=True))
    # numbers up to 300 (433 in base 2) are rounded half a dozen times on the way: 2^-24 * 512 each; sums as above
    assert np.max(np.abs(lp - ref)) <= 2e-5 + 6 * 2.0 ** -15
