"""Grouping of ids inside the hidden update's launch (up to 1024 raw queries): group numbers, representatives and results
against the oracle around its sizes (one and two ids per thread, the limit), for the key that marks a free slot, all ids
equal and all distinct; and the separate launch where an output lies on the ids."""
import numpy as np
import pytest
import torch

import oracle
import paper_2007_11794_amd as rn

from harness import DEV, gpu_step_dedup, keys_tensor, load_model

pytestmark = pytest.mark.gpu
V, H = 50, 72


@pytest.fixture(scope="module")
def model():
    rng = np.random.default_rng(3)
    m = {"U": rng.normal(0, 0.3, (V, H)), "W": rng.normal(0, 0.1, (H, H)), "O": rng.normal(0, 0.1, (H, V)), "bias": np.zeros(V)}
    return {k: v.astype(np.float32) for k, v in m.items()}


@pytest.mark.parametrize("N", [1, 2, 31, 64, 511, 512, 513, 1000, 1023, 1024, 1025])
@pytest.mark.parametrize("kind", ["mixed", "equal", "distinct"])
def test_groups_and_results(model, N, kind):
    rng = np.random.default_rng(N)
    pool = rng.integers(0, 2 ** 63, max(1, N // 3), dtype=np.uint64)
    pool[0] = 0xFFFFFFFFFFFFFFFF
    if len(pool) > 2:
        pool[1], pool[2] = 0, pool[-1] ^ np.uint64(1 << 32)          # zero; a key that differs in its high half only
    ids = {"mixed": pool[rng.integers(0, len(pool), N)], "equal": np.full(N, pool[0]),
           "distinct": np.arange(N, dtype=np.uint64) * np.uint64(0x100000001) + np.uint64(7)}[kind]
    u, rep, inv = oracle.dedup(ids)
    prev, h_in = rng.integers(0, V, N).astype(np.int32), rng.uniform(0, 1, (N, H)).astype(np.float32)
    prev, h_in = prev[rep][inv], h_in[rep][inv]
    query = rng.integers(0, V, (N, 2)).astype(np.int32)
    m = load_model(model, "f32", N)
    out = gpu_step_dedup(m, ids, prev, h_in, query)
    assert out["n_unique"] == u and np.array_equal(out["rep"], rep) and np.array_equal(out["inverse"], inv)
    ref = oracle.step(model, prev[rep], h_in[rep], query, row_of_query=inv)
    assert np.max(np.abs(out["h_out"] - ref["h_out"])) <= 1e-5 and np.max(np.abs(out["logprob"] - ref["logprob"])) <= 1e-5
    assert np.isnan(out["h_out_rest"]).all()                          # rows beyond the groups stay untouched
    m.close()


def test_outputs_on_the_ids(model):
    """inverse written over the ids: allowed when one launch reads them all before another writes."""
    N = 300
    rng = np.random.default_rng(1)
    ids = rng.integers(0, 40, N, dtype=np.uint64)
    u, rep, inv = oracle.dedup(ids)
    prev, h_in = rng.integers(0, V, N).astype(np.int32)[rep][inv], rng.uniform(0, 1, (N, H)).astype(np.float32)[rep][inv]
    query = rng.integers(0, V, (N, 1)).astype(np.int32)
    m = load_model(model, "f32", N)
    k = keys_tensor(ids)
    inverse = k.view(torch.int32)[:N]
    rep_t, nu = torch.zeros(N, dtype=torch.int32, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
    h_out, lp = torch.zeros((N, H), device=DEV), torch.zeros((N, 1), device=DEV)
    ws = torch.empty(rn.rnnlm_dedup_workspace_bytes(N), dtype=torch.uint8, device=DEV)
    rn.rnnlm_step_dedup(m, k, torch.from_numpy(prev).to(DEV), torch.from_numpy(h_in).to(DEV), torch.from_numpy(query).to(DEV),
                        rep_t, inverse, nu, h_out, lp, ws)
    assert int(nu.item()) == u and np.array_equal(inverse.cpu().numpy(), inv)
    ref = oracle.step(model, prev, h_in, query)
    assert np.max(np.abs(lp.cpu().numpy() - ref["logprob"])) <= 1e-5
    m.close()
