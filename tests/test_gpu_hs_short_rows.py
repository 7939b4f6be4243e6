"""Path kernel of the hierarchical layer for padded hidden sizes that fill 8 of 16 or 24 of 32 lanes of a node row (64 and 192, both
types), against the oracle; and an infinite node weight, which lanes beyond the row must not turn into NaN."""
import numpy as np
import pytest
import torch

import oracle
import paper_2007_11794_amd as rn
from workloads import bf16_bits, round_to_bf16

from harness import DEV

pytestmark = pytest.mark.gpu


def run(V, H, N, K, dtype, spoil=False):
    rng = np.random.default_rng(H + N)
    sigma = 0.5 / np.sqrt(H)
    U, W, theta = (rng.normal(0, s, shape).astype(np.float32) for s, shape in
                   ((0.3, (V, H)), (sigma, (H, H)), (2 * sigma, (V - 1, H))))
    if dtype == "bf16":
        U, W, theta = (round_to_bf16(x) for x in (U, W, theta))
    if spoil:
        theta[V - 2, 0] = np.inf                                   # the root: on every path
    off, entry = rn.rnnlm_huffman_build(np.arange(1, V + 1, dtype=np.float64) ** -1.1)
    code, give = (rn.RNNLM_BF16, bf16_bits) if dtype == "bf16" else (rn.RNNLM_F32, np.ascontiguousarray)
    m = rn.rnnlm_hs_load(V, H, code, give(U), give(W), give(theta), off, entry, N)
    prev, h_in = rng.integers(0, V, N).astype(np.int32), rng.uniform(0, 1, (N, H)).astype(np.float32)
    query = (V ** rng.uniform(0, 1, (N, K))).astype(np.int32) - 1
    h_out, lp = torch.zeros((N, H), device=DEV), torch.zeros((N, K), device=DEV)
    rn.rnnlm_hs_step(m, torch.from_numpy(prev).to(DEV), torch.from_numpy(h_in).to(DEV), torch.from_numpy(query).to(DEV), h_out, lp)
    rows = np.unique(np.linspace(0, N - 1, 25).astype(int))
    out = lp.cpu().numpy()[rows]
    assert m.last_error() == 0
    m.close()
    return out, oracle.hs_step({"U": U, "W": W, "theta": theta, "path_off": off, "path_entry": entry}, prev[rows], h_in[rows], query[rows])["logprob"]


@pytest.mark.parametrize("dtype,H", [("f32", 1), ("f32", 50), ("f32", 64), ("f32", 129), ("f32", 192), ("bf16", 130), ("bf16", 180), ("bf16", 192)])
@pytest.mark.parametrize("N,K", [(3, 4), (256, 25), (257, 25), (300, 60)])
def test_against_the_oracle(dtype, H, N, K):
    out, ref = run(2000, H, N, K, dtype)
    # up to 17 terms of fp32 dot products of H products: 2^-24 of sums below 2, some hundred roundings, random signs
    assert np.max(np.abs(out - ref)) <= 2e-5


@pytest.mark.parametrize("dtype,H", [("f32", 40), ("bf16", 150)])
def test_an_infinite_weight(dtype, H):
    out, _ = run(500, H, 6, 8, dtype, spoil=True)
    clean, _ = run(500, H, 6, 8, dtype)
    gone = np.isneginf(out)                                        # one side of the root has no mass left
    assert not np.isnan(out).any() and gone.any() and not gone.all() and np.isfinite(clean).all()
