"""Staged output projection at every padded hidden size it is built for, against the oracle: rows around its groups of
256, vocabularies that end inside a block and a split, both forms of the log-sum-exp, row counts known on the device only."""
import numpy as np
import pytest

import oracle
import paper_2007_11794_amd as rn
from workloads import round_to_bf16

from harness import gpu_step, gpu_step_dedup, load_model

pytestmark = pytest.mark.gpu


def logprob_of_rounded_rows(model, h, query, scale):
    """What the kernel computes, in float64: the rows h' - 1/2 enter the normaliser as bf16 numbers, times scale where that is
    folded in.  Also the smallest share in a normaliser that a whole block of 32 words has."""
    O, bias = model["O"].astype(np.float64), model["bias"].astype(np.float64)
    d = round_to_bf16((h - np.float32(0.5)) * np.float32(scale)).astype(np.float64) / scale
    z = d @ O + (bias + 0.5 * O.sum(0))
    top = z.max(1, keepdims=True)
    p = np.exp(z - top)
    blocks = p[:, :p.shape[1] // 32 * 32].reshape(len(p), -1, 32).sum(2) / p.sum(1, keepdims=True)
    exact = np.take_along_axis(h.astype(np.float64) @ O + bias, query, 1)
    return exact - top - np.log(p.sum(1, keepdims=True)), blocks.min()


@pytest.mark.parametrize("H,V,B", [(100, 33, 128), (129, 5000, 129), (192, 8300, 255), (300, 4097, 257), (333, 20000, 130),
                                   (384, 700, 512), (445, 9000, 300), (512, 12345, 200), (570, 6000, 131), (600, 33000, 140),
                                   (640, 1000, 513), (650, 16500, 317), (704, 4100, 128)])
def test_against_the_oracle(H, V, B):
    rng = np.random.default_rng(H * 100003 + B)
    sigma = 1.0 / np.sqrt(H)
    model = {"U": rng.normal(0, 0.3, (V, H)), "W": rng.normal(0, sigma, (H, H)), "O": rng.normal(0, 2 * sigma, (H, V))}
    model = {k: round_to_bf16(v.astype(np.float32)) for k, v in model.items()}
    model["bias"] = rng.normal(0, 0.5, V).astype(np.float32)
    m = load_model(model, "bf16", B)
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    query = rng.integers(0, V, (B, 2)).astype(np.int32)
    ref = oracle.step(model, prev, h_in, query)
    assert m.outproj_kernel_name(B) == "outproj_staged_kernel"
    # h' - 1/2 enters the normaliser rounded to bf16: 2^-10 at most per unit, random signs, weights of 2 / sqrt(H)
    tol = 1e-4 + 2 * 2.0 ** -10
    by_mode = []
    for lse_mode in (0, 1):
        m.set_option(rn.OPT_LSE_MODE, lse_mode)
        h, lp = gpu_step(m, prev, h_in, query)
        assert np.max(np.abs(h - ref["h_out"])) <= 1e-5 and np.max(np.abs(lp - ref["logprob"])) <= tol, lse_mode
        by_mode.append(lp)
        # beside that rounding: fp32 sums, 2^-24 of logits below 40 some hundred times, random signs.  A block of 32 words that
        # the normaliser misses moves it by the block's share, three times that or more at every size here
        scale = np.log2(np.e) if -(-H // 64) * 64 in (128, 256, 512) else 1.0
        tight, share = logprob_of_rounded_rows(model, h, query, scale)
        assert share > 3e-4 and np.max(np.abs(lp - tight)) <= 1e-4, lse_mode
    # the same operands, fp32 sums in another order: 2^-24 of logits below 40 some hundred times, random signs
    assert np.max(np.abs(by_mode[0] - by_mode[1])) <= 1e-4
    m.set_option(rn.OPT_LSE_MODE, 0)
    src = rng.integers(0, max(1, B // 2), B)
    out = gpu_step_dedup(m, src.astype(np.uint64) + 9, prev[src], h_in[src], query)
    ref = oracle.step(model, prev[src], h_in[src], query)
    assert np.max(np.abs(out["logprob"] - ref["logprob"])) <= tol
    assert m.last_error() == 0
    m.close()
