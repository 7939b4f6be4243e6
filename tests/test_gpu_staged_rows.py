"""Staged output projection with row groups that are not full: waves without rows (they only load), and beyond Hp = 512 groups of
128 rows from 257 to 384; counts known to the host and on the device only, both forms of the log-sum-exp, items of one block, a
few and many, three and four LDS stages, weights in either order.  Against float64 on the rows as the kernel rounds them."""
import numpy as np
import pytest

import oracle
import paper_2007_11794_amd as rn
from workloads import round_to_bf16

from harness import gpu_step, gpu_step_dedup, load_model
from test_gpu_staged_sizes import logprob_of_rounded_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,V", [(128, 300), (190, 9000), (500, 10000), (512, 33000), (576, 700), (650, 12000), (704, 5000)])
def test_partly_filled_groups(H, V):
    rng = np.random.default_rng(H)
    sigma = 1.0 / np.sqrt(H)
    model = {"U": rng.normal(0, 0.3, (V, H)), "W": rng.normal(0, sigma, (H, H)), "O": rng.normal(0, 2 * sigma, (H, V))}
    model = {k: round_to_bf16(v.astype(np.float32)) for k, v in model.items()}
    model["bias"] = rng.normal(0, 0.5, V).astype(np.float32)
    N = 700
    m = load_model(model, "bf16", N)
    prev, h_in = rng.integers(0, V, N).astype(np.int32), rng.uniform(0, 1, (N, H)).astype(np.float32)
    query = rng.integers(0, V, (N, 2)).astype(np.int32)
    scale = np.log2(np.e) if -(-H // 64) * 64 in (128, 256, 512) else 1.0
    h_all = oracle.step(model, prev, h_in, query)["h_out"]
    want, share = logprob_of_rounded_rows(model, h_all, query, scale)
    assert share > 3e-4                                            # a lost block of words moves a normaliser three times the bar
    for mode in (0, 1):
        m.set_option(rn.OPT_LSE_MODE, mode)
        for B in (128, 129, 160, 161, 256, 257, 288, 320, 384, 385, 512, 513, 640, 672):      # known to the host
            h, lp = gpu_step(m, prev[:B], h_in[:B], query[:B])
            # fp32 sums, 2^-24 of logits below 40 some hundred times; a unit whose fp32 value differs in the last place may round to
            # the other bf16 number (2^-10 of a weight of 2 / sqrt(H), a few units of a row)
            assert np.max(np.abs(h - h_all[:B])) <= 1e-5 and np.max(np.abs(lp - want[:B])) <= 2e-4, (mode, B)
        for U in (1, 65, 66, 96, 97, 128, 129, 255, 257, 300, 383, 385, 513, 600):             # on the device only
            src = np.concatenate([np.arange(U), rng.integers(0, U, N - U)])
            out = gpu_step_dedup(m, src.astype(np.uint64) + 9, prev[src], h_in[src], query[src])
            assert out["n_unique"] == U and np.max(np.abs(out["logprob"] - want[src])) <= 2e-4, (mode, U)
    assert m.last_error() == 0
    m.close()
