"""Steps of the hierarchical layer in one launch (hidden update inside the path kernel): at the limits of its queries and rows, at the
edges of the hidden sizes, with queries mapped to rows and rows nobody asks about, mistakes, base scores, and outputs on inputs."""
import numpy as np
import pytest
import torch

import oracle
import paper_2007_11794_amd as rn
from workloads import bf16_bits, round_to_bf16

from harness import DEV

pytestmark = pytest.mark.gpu
V = 1500


def make(H, dtype, max_B):
    rng = np.random.default_rng(H)
    sigma = 0.5 / np.sqrt(H)
    m = {k: rng.normal(0, s, shape).astype(np.float32) for k, s, shape in
         (("U", 0.3, (V, H)), ("W", sigma, (H, H)), ("theta", 2 * sigma, (V - 1, H)))}
    code, give = rn.RNNLM_F32, np.ascontiguousarray
    if dtype == "bf16":
        m = {k: round_to_bf16(x) for k, x in m.items()}
        code, give = rn.RNNLM_BF16, bf16_bits
    m["path_off"], m["path_entry"] = rn.rnnlm_huffman_build(np.arange(1, V + 1, dtype=np.float64) ** -1.1)
    return m, rn.rnnlm_hs_load(V, H, code, give(m["U"]), give(m["W"]), give(m["theta"]), m["path_off"], m["path_entry"], max_B)


def inputs(H, B, N, K):
    rng = np.random.default_rng(B + N)
    return (rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32),
            (V ** rng.uniform(0, 1, (N, K))).astype(np.int32) - 1, rng.integers(0, B, N).astype(np.int32))


def step(mod, H, prev, h_in, query, row=None, base=None):
    t = lambda x: None if x is None else torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
    h_out = torch.full((len(prev), H), float("nan"), device=DEV)
    lp = torch.full(query.shape, float("nan"), device=DEV)
    rn.rnnlm_hs_step(mod, t(prev), t(h_in), t(query), h_out, lp, row_of_query=t(row), base_score=t(base))
    return h_out.cpu().numpy(), lp.cpu().numpy()


# fp32 sums of up to 256 products and 17 terms of a path: 2^-24 of sums below 2, some hundred roundings, random signs
def close(out, ref):
    assert np.max(np.abs(out[0] - ref["h_out"])) <= 2e-6 and np.max(np.abs(out[1] - ref["logprob"])) <= 2e-5


@pytest.mark.parametrize("dtype,H,N,K", [("f32", 1, 5, 4), ("f32", 63, 3, 9), ("f32", 64, 512, 4), ("f32", 65, 513, 4), ("f32", 128, 40, 64),
                                         ("f32", 129, 256, 5), ("f32", 250, 7, 30), ("f32", 256, 257, 6), ("bf16", 100, 1024, 4),
                                         ("bf16", 128, 1025, 4), ("bf16", 127, 30, 20), ("bf16", 192, 256, 12), ("bf16", 256, 9, 40), ("bf16", 257, 9, 8)])
def test_a_row_per_query(dtype, H, N, K):
    m, mod = make(H, dtype, N)
    prev, h_in, query, _ = inputs(H, N, N, K)
    out = step(mod, H, prev, h_in, query)
    close(out, oracle.hs_step(m, prev, h_in, query))
    assert mod.last_error() == 0
    mod.close()


@pytest.mark.parametrize("dtype,H,B,N", [("f32", 100, 3, 200), ("f32", 180, 128, 256), ("f32", 180, 129, 256), ("bf16", 90, 200, 17), ("bf16", 256, 1, 1), ("bf16", 70, 512, 1024)])
def test_queries_mapped_to_rows(dtype, H, B, N):
    m, mod = make(H, dtype, 1024)
    prev, h_in, query, row = inputs(H, B, N, 6)
    row[row == B - 1] = 0                                          # nobody asks about the last row
    base = np.random.default_rng(1).normal(0, 1, query.shape).astype(np.float32)
    out = step(mod, H, prev, h_in, query, row, base)
    ref = oracle.hs_step(m, prev, h_in, query, row_of_query=row)
    close((out[0], out[1] + base), ref)
    mod.close()


def test_mistakes():
    H, B, N = 120, 6, 12
    m, mod = make(H, "bf16", 16)
    prev, h_in, query, row = inputs(H, B, N, 5)
    row = np.arange(N, dtype=np.int32) % B
    good = step(mod, H, prev, h_in, query, row)
    prev2, query2, row2 = prev.copy(), query.copy(), row.copy()
    prev2[2], query2[3, 1], query2[5, 4], row2[7], row2[10] = -1, V, -5, B, -1
    out = step(mod, H, prev2, h_in, query2, row2)
    assert mod.last_error() == rn.FLAG_BAD_PREV_WORD | rn.FLAG_BAD_QUERY_WORD | rn.FLAG_BAD_ROW and mod.last_error() == 0
    bad = np.zeros((N, 5), bool)
    bad[2], bad[8], bad[7], bad[10], bad[3, 1], bad[5, 4] = True, True, True, True, True, True
    assert np.isnan(out[1][bad]).all() and np.array_equal(out[1][~bad], good[1][~bad])
    assert np.isnan(out[0][2]).all() and np.array_equal(np.delete(out[0], 2, 0), np.delete(good[0], 2, 0))
    mod.close()


def test_answers_on_top_of_the_words_asked_for():
    H, N, K = 64, 9, 5
    m, mod = make(H, "f32", 16)
    prev, h_in, query, _ = inputs(H, N, N, K)
    q, h_out = torch.from_numpy(query).to(DEV), torch.zeros((N, H), device=DEV)
    rn.rnnlm_hs_step(mod, torch.from_numpy(prev).to(DEV), torch.from_numpy(h_in).to(DEV), q, h_out, q.view(torch.float32))
    close((h_out.cpu().numpy(), q.view(torch.float32).cpu().numpy()), oracle.hs_step(m, prev, h_in, query))
    mod.close()
