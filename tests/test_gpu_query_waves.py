"""Waves per raw query in the query kernel: 4, 2 or 1 by the words and the number of queries, at the counts where that changes and
with a last workgroup that is not full, against the oracle."""
import numpy as np
import pytest

import oracle

from harness import gpu_step, gpu_step_dedup, load_model

pytestmark = pytest.mark.gpu
V, H = 60, 70


@pytest.fixture(scope="module")
def model():
    rng = np.random.default_rng(4)
    m = {"U": rng.normal(0, 0.3, (V, H)), "W": rng.normal(0, 0.1, (H, H)), "O": rng.normal(0, 0.1, (H, V)), "bias": rng.normal(0, 0.1, V)}
    return {k: v.astype(np.float32) for k, v in m.items()}


@pytest.mark.parametrize("N,K", [(1024, 17), (1025, 17), (2048, 9), (2048, 33), (2049, 9), (2049, 18), (4096, 8), (4097, 41)])
def test_rows(model, N, K):
    rng = np.random.default_rng(N + K)
    B = 70
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    query, row = rng.integers(0, V, (N, K)).astype(np.int32), rng.integers(0, B, N).astype(np.int32)
    m = load_model(model, "f32", N)
    h, p = gpu_step(m, prev, h_in, query, row)
    ref = oracle.step(model, prev, h_in, query, row_of_query=row)
    assert np.max(np.abs(h - ref["h_out"])) <= 1e-5 and np.max(np.abs(p - ref["logprob"])) <= 1e-5
    m.close()


@pytest.mark.parametrize("N,K", [(2050, 12), (1030, 20)])
def test_grouped(model, N, K):
    rng = np.random.default_rng(N)
    ids = rng.integers(0, 90, N, dtype=np.uint64)
    u, rep, inv = oracle.dedup(ids)
    prev, h_in = rng.integers(0, V, N).astype(np.int32)[rep][inv], rng.uniform(0, 1, (N, H)).astype(np.float32)[rep][inv]
    query = rng.integers(0, V, (N, K)).astype(np.int32)
    m = load_model(model, "f32", N)
    out = gpu_step_dedup(m, ids, prev, h_in, query)
    ref = oracle.step(model, prev[rep], h_in[rep], query, row_of_query=inv)
    assert out["n_unique"] == u and np.max(np.abs(out["logprob"] - ref["logprob"])) <= 1e-5
    m.close()
