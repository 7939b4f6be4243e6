"""Path kernel of the hierarchical layer on both sides of its two limits: queries per launch (twice the threads up to
512, 256 for hidden sizes of 128 and 256) and path entries per query (256), against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2007_11794_amd as rn

from harness import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,N,K", [(100, 256, 20), (100, 257, 20), (250, 256, 4), (250, 257, 4), (300, 512, 30), (300, 513, 30),
                                   (300, 512, 4), (520, 9, 40), (40, 1, 64)])
def test_against_the_oracle(H, N, K):
    V = 3000
    rng = np.random.default_rng(H + N)
    sigma = 0.5 / np.sqrt(H)
    U, W, theta = (rng.normal(0, s, shape).astype(np.float32) for s, shape in
                   ((0.3, (V, H)), (sigma, (H, H)), (2 * sigma, (V - 1, H))))
    off, entry = rn.rnnlm_huffman_build(np.arange(1, V + 1, dtype=np.float64) ** -1.1)
    m = rn.rnnlm_hs_load(V, H, rn.RNNLM_F32, U, W, theta, off, entry, N)
    prev, h_in = rng.integers(0, V, N).astype(np.int32), rng.uniform(0, 1, (N, H)).astype(np.float32)
    query = (V ** rng.uniform(0, 1, (N, K))).astype(np.int32) - 1
    h_out, lp = torch.zeros((N, H), device=DEV), torch.zeros((N, K), device=DEV)
    rn.rnnlm_hs_step(m, torch.from_numpy(prev).to(DEV), torch.from_numpy(h_in).to(DEV), torch.from_numpy(query).to(DEV), h_out, lp)
    rows = np.unique(np.linspace(0, N - 1, 25).astype(int))
    ref = oracle.hs_step({"U": U, "W": W, "theta": theta, "path_off": off, "path_entry": entry}, prev[rows], h_in[rows], query[rows])
    # up to 17 terms of fp32 dot products of H products: 2^-24 of sums below 2, some hundred roundings, random signs
    assert np.max(np.abs(lp.cpu().numpy()[rows] - ref["logprob"])) <= 2e-5
    assert m.last_error() == 0
    m.close()
