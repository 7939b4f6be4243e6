"""Steps of few rows in one launch (grouping, hidden update, output projection, words and normaliser): against the oracle and
against the launches it replaces (option 5 takes them), at the edges of its rows, units, words and pairs."""
import numpy as np
import pytest
import torch

import oracle
import paper_2007_11794_amd as rn
from workloads import round_to_bf16

from harness import DEV, CachedStepper, gpu_step, gpu_step_dedup, load_model

pytestmark = pytest.mark.gpu
BARS = {"f32": (1e-5, 1e-5), "bf16": (1e-3, 2e-3)}
# Both routes round the same hidden vector to bf16 (fp32 models: to two fp16 terms, 2^-23).  A unit whose fp32 value differs in its
# last place may round to the other neighbour, 2^-9 / 2 at most, and moves a log-probability by that times a weight difference of
# at most 8 sigma = 0.4: 4e-4 if it happens to one unit, and it happens to about one in 2^14.
ROUTES = {"f32": 1e-5, "bf16": 4e-4}


def make(V, H, dtype, sigma=0.05, seed=1):
    rng = np.random.default_rng(seed)
    m = {"U": rng.normal(0, sigma, (V, H)), "W": rng.normal(0, sigma, (H, H)), "O": rng.normal(0, sigma, (H, V)), "bias": rng.normal(0, sigma, V)}
    m = {k: v.astype(np.float32) for k, v in m.items()}
    if dtype == "bf16":
        for k in "UWO":
            m[k] = round_to_bf16(m[k])
    return m


def inputs(V, H, B, N, K, seed=2):
    rng = np.random.default_rng(seed)
    return (rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32), rng.integers(0, V, (N, K)).astype(np.int32),
            rng.integers(0, B, N).astype(np.int32))


def check(out, ref, dtype):
    h_bar, p_bar = BARS[dtype]
    assert np.max(np.abs(out[0] - ref["h_out"])) <= h_bar and np.max(np.abs(out[1] - ref["logprob"])) <= p_bar


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V,H,B,K", [(1, 1, 1, 1), (31, 3, 2, 5), (257, 64, 32, 1), (1300, 63, 31, 8), (1300, 65, 17, 3), (1281, 127, 32, 7), (5000, 128, 16, 64),
                                     (2049, 129, 9, 33), (900, 192, 21, 8), (4100, 200, 5, 2), (700, 253, 16, 4), (8000, 256, 8, 8), (20011, 100, 16, 11)])
def test_rows(dtype, V, H, B, K):
    model = make(V, H, dtype)
    m = load_model(model, dtype, 64)
    prev, h_in, query, row = inputs(V, H, B, B, K)
    out = gpu_step(m, prev, h_in, query)
    check(out, oracle.step(model, prev, h_in, query), dtype)
    again = gpu_step(m, prev, h_in, query)                        # the launch leaves its counter as it found it
    assert np.array_equal(out[0], again[0]) and np.array_equal(out[1], again[1])
    if V > 1:
        m.set_option(rn.OPT_OUTPROJ_KERNEL, 5)
        old = gpu_step(m, prev, h_in, query)
        assert np.max(np.abs(out[0] - old[0])) <= 1e-6 and np.max(np.abs(out[1] - old[1])) <= ROUTES[dtype]
    m.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,K", [(1, 8192), (200, 40), (201, 41), (3, 3)])
def test_more_queries_than_rows(dtype, N, K):
    V, H, B = 3000, 96, min(N, 12)                                # (200 x 40 words and more: the separate launches)
    model = make(V, H, dtype)
    m = load_model(model, dtype, 256)
    prev, h_in, query, row = inputs(V, H, B, N, K)
    check(gpu_step(m, prev, h_in, query, row), oracle.step(model, prev, h_in, query, row_of_query=row), dtype)
    m.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,K", [(128, 32), (64, 128), (40, 150), (20, 409), (8, 1024)])
def test_more_words_than_one_round(dtype, N, K):
    """More answers than the last workgroup holds beside the partials, and more than one batch of dot products a wave."""
    V, H, B = 3000, 96, 12
    model = make(V, H, dtype)
    m = load_model(model, dtype, 256)
    assert m.one_launch(B, N, K, mapped=True)
    prev, h_in, query, row = inputs(V, H, B, N, K)
    check(gpu_step(m, prev, h_in, query, row), oracle.step(model, prev, h_in, query, row_of_query=row), dtype)
    m.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,H", [(1, 70), (2, 128), (31, 64), (32, 120), (20, 190), (16, 256)])
def test_grouped(dtype, N, H):
    V, K = 1500, 6
    model = make(V, H, dtype)
    m = load_model(model, dtype, 64)
    prev, h_in, query, _ = inputs(V, H, N, N, K)
    rng = np.random.default_rng(N)
    pool = rng.integers(0, 2 ** 63, max(1, N // 2), dtype=np.uint64)
    pool[0] = 0
    if len(pool) > 2:
        pool[1], pool[2] = 0xFFFFFFFFFFFFFFFF, pool[-1] ^ np.uint64(1 << 32)
    ids = pool[rng.integers(0, len(pool), N)]
    u, rep, inv = oracle.dedup(ids)
    prev, h_in = prev[rep][inv], h_in[rep][inv]
    out = gpu_step_dedup(m, ids, prev, h_in, query)
    assert out["n_unique"] == u and np.array_equal(out["rep"], rep) and np.array_equal(out["inverse"], inv)
    assert np.isnan(out["h_out_rest"]).all()                      # rows beyond the groups stay untouched
    check((out["h_out"], out["logprob"]), oracle.step(model, prev[rep], h_in[rep], query, row_of_query=inv), dtype)
    m.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_running_maximum_and_mistakes(dtype):
    V, H, B, K = 1000, 100, 8, 6
    model = make(V, H, dtype, sigma=0.3)
    m = load_model(model, dtype, 16)
    prev, h_in, query, row = inputs(V, H, B, B, K)
    ref = oracle.step(model, prev, h_in, query)
    for mode in (1, 0):
        m.set_option(rn.OPT_LSE_MODE, mode)
        out = gpu_step(m, prev, h_in, query)
        assert np.max(np.abs(out[0] - ref["h_out"])) <= BARS[dtype][0]
        assert np.max(np.abs(out[1] - ref["logprob"])) <= 6 * BARS[dtype][1]      # weights six times those of the bars
    good = gpu_step(m, prev, h_in, query, row)
    prev2, query2, row2 = prev.copy(), query.copy(), row.copy()
    prev2[3], query2[1, 2], query2[4, 0], row2[6], row2[7], row2[1], row2[4] = V, -1, V, -1, B, 0, 1
    row2[[0, 2, 3, 5]] = [3, 0, 1, 2]
    good = gpu_step(m, prev, h_in, query, np.clip(row2, 0, B - 1))
    assert m.last_error() == 0
    h, p = gpu_step(m, prev2, h_in, query2, row2)
    assert m.last_error() == rn.FLAG_BAD_PREV_WORD | rn.FLAG_BAD_QUERY_WORD | rn.FLAG_BAD_ROW and m.last_error() == 0
    bad = np.zeros((B, K), bool)
    bad[0], bad[6], bad[7], bad[1, 2], bad[4, 0] = True, True, True, True, True
    assert np.isnan(p[bad]).all() and np.array_equal(p[~bad], good[1][~bad])
    assert np.isnan(h[3]).all() and np.array_equal(np.delete(h, 3, 0), np.delete(good[0], 3, 0))
    m.close()


def test_answers_on_top_of_the_words_asked_for():
    """Outputs that share memory with inputs take the launches that read them all first."""
    V, H, B, K = 2000, 64, 8, 4
    model = make(V, H, "f32")
    m = load_model(model, "f32", 16)
    prev, h_in, query, _ = inputs(V, H, B, B, K)
    q = torch.from_numpy(query).to(DEV)
    h_out = torch.zeros((B, H), device=DEV)
    rn.rnnlm_step(m, torch.from_numpy(prev).to(DEV), torch.from_numpy(h_in).to(DEV), q, h_out, q.view(torch.float32))
    check((h_out.cpu().numpy(), q.view(torch.float32).cpu().numpy()), oracle.step(model, prev, h_in, query), "f32")
    m.close()


def test_rows_in_single_floats():
    """h_in that does not begin on 16 bytes."""
    V, H, B, K = 1500, 96, 20, 5
    model = make(V, H, "bf16")
    m = load_model(model, "bf16", 32)
    prev, h_in, query, _ = inputs(V, H, B, B, K)
    flat = torch.zeros(B * H + 1, device=DEV)
    flat[1:] = torch.from_numpy(h_in).to(DEV).flatten()
    h_out, lp = torch.zeros((B, H), device=DEV), torch.zeros((B, K), device=DEV)
    rn.rnnlm_step(m, torch.from_numpy(prev).to(DEV), flat[1:].view(B, H), torch.from_numpy(query).to(DEV), h_out, lp)
    check((h_out.cpu().numpy(), lp.cpu().numpy()), oracle.step(model, prev, h_in, query), "bf16")
    m.close()


@pytest.mark.parametrize("dtype,V,H,B,K", [("f32", 1300, 65, 17, 3), ("f32", 4000, 128, 24, 8), ("f32", 15000, 100, 16, 7), ("f32", 20011, 100, 8, 11), ("f32", 30011, 50, 16, 5),
                                           ("bf16", 900, 192, 16, 8), ("bf16", 8000, 117, 32, 6), ("bf16", 4100, 200, 5, 2), ("bf16", 16000, 251, 8, 4), ("bf16", 30011, 128, 16, 9)])
def test_rows_up_to_the_lines(dtype, V, H, B, K):
    """The largest steps that are one launch, and that they are."""
    model = make(V, H, dtype)
    m = load_model(model, dtype, 64)
    assert m.one_launch(B, B, K)
    prev, h_in, query, _ = inputs(V, H, B, B, K)
    out = gpu_step(m, prev, h_in, query)
    check(out, oracle.step(model, prev, h_in, query), dtype)
    m.set_option(rn.OPT_OUTPROJ_KERNEL, 5)
    assert not m.one_launch(B, B, K)
    old = gpu_step(m, prev, h_in, query)
    assert np.max(np.abs(out[0] - old[0])) <= 1e-6 and np.max(np.abs(out[1] - old[1])) <= ROUTES[dtype]
    m.close()


# (32, 100): more answers than the last workgroup holds beside the partials
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,K", [(1, 5), (16, 7), (32, 3), (32, 100)])
def test_grouped_with_base_scores(dtype, N, K):
    V, H = 1500, 90
    model = make(V, H, dtype)
    m = load_model(model, dtype, 64)
    assert m.one_launch(0, N, K, grouped=True)
    prev, h_in, query, _ = inputs(V, H, N, N, K)
    rng = np.random.default_rng(N + K)
    ids = rng.integers(0, 2 ** 63, max(1, N // 2), dtype=np.uint64)[rng.integers(0, max(1, N // 2), N)]
    u, rep, inv = oracle.dedup(ids)
    prev, h_in = prev[rep][inv], h_in[rep][inv]
    base = rng.normal(0, 2, (N, K)).astype(np.float32)
    st = CachedStepper(m, None, N, K)
    plain, less = st.step(ids, prev, h_in, query), st.step(ids, prev, h_in, query, base)
    assert plain["n_unique"] == less["n_unique"] == u and np.array_equal(plain["rep"], rep) and np.array_equal(less["inverse"], inv)
    assert np.array_equal(less["score"], plain["score"] - base)             # one fp32 subtraction
    assert np.array_equal(less["h_out"], plain["h_out"])
    check((plain["h_out"], plain["score"]), oracle.step(model, prev[rep], h_in[rep], query, row_of_query=inv), dtype)
    # the answers in the place of the base scores: the launches that read them first
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
    both, h_out = t(base), torch.zeros((N, H), device=DEV)
    r, i, nu = (torch.zeros(n, dtype=torch.int32, device=DEV) for n in (N, N, 1))
    rn.rnnlm_step_cached(m, None, t(ids.view(np.int64)), t(prev), t(h_in), t(query), r, i, nu, h_out, both, st.ws, base_score=both)
    assert np.max(np.abs(both.cpu().numpy() - less["score"])) <= ROUTES[dtype] + 1e-6         # (one more rounding of sums below 16)
    m.close()
