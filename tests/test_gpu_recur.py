"""Hidden update against the oracle where its shapes change: row counts around a tile and around the limits of the small
shape (one and two workgroups per compute unit), hidden sizes that end inside a tile of 128 units or are no multiple of
four, buffers that are not 16-byte aligned, row counts known on the device only."""
import numpy as np
import pytest
import torch

import oracle
import paper_2007_11794_amd as rn
from workloads import round_to_bf16

from harness import DEV, gpu_step, gpu_step_dedup, load_model

pytestmark = pytest.mark.gpu
V = 40


def model_of(rng, H, dtype):
    m = {"U": rng.normal(0, 0.3, (V, H)).astype(np.float32), "W": rng.normal(0, 1.0 / np.sqrt(H), (H, H)).astype(np.float32),
         "O": rng.normal(0, 0.1, (H, V)).astype(np.float32), "bias": np.zeros(V, np.float32)}
    return {k: round_to_bf16(v) if k != "bias" and dtype == "bf16" else v for k, v in m.items()}


# hidden size, rows: small_rows is 256 * (32 / (padded H / 64)) rows, with 64 in the place of 32 beyond them (rounded down)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H,B", [(64, 31), (64, 33), (150, 64), (130, 65), (333, 257), (512, 1024), (512, 1025), (1022, 513),
                                 (1024, 1024), (1024, 1025), (1100, 500), (1100, 931), (2048, 513), (4096, 257),
                                 (64, 300), (64, 4096), (64, 4097), (61, 1), (192, 1344), (190, 1345), (256, 1024), (512, 512), (650, 16), (1024, 256),
                                 (1100, 64), (2048, 64), (700, 513), (704, 1280), (704, 1281), (512, 2049), (1088, 769), (320, 3073)])
def test_against_the_oracle(H, B, dtype):
    rng = np.random.default_rng(H * 10000 + B)
    model = model_of(rng, H, dtype)
    m = load_model(model, dtype, B)
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    query = rng.integers(0, V, (B, 1)).astype(np.int32)
    rows = np.unique(np.concatenate([np.arange(0, B, 29), np.arange(max(0, B - 40), B), np.arange(min(B, 40))]))
    ref = oracle.step(model, prev[rows], h_in[rows], query[rows])
    # |h'| error: a quarter of that of the sum, which rounds 2^-24 of sums below 2 some tens of times (and, bf16
    # models, drops 2^-17 of the centred inputs, 2^-18 at most, with random signs, over H weights of 1 / sqrt(H))
    tol_h = 2e-6 if dtype == "f32" else 1e-5
    # log-probabilities: the normaliser of bf16 models takes h' - 1/2 rounded to bf16, 2^-10 at most per unit, random
    # signs, H weights of 0.1
    tol_lp = 1e-5 if dtype == "f32" else 1e-4 + 0.1 * np.sqrt(H) * 2.0 ** -10
    for shift in (0, 1):                                       # base of h_in and h_out: 16-byte aligned, 4-byte aligned
        buf_in = torch.zeros(B * H + 4, device=DEV)
        buf_out = torch.full((B * H + 4,), float("nan"), device=DEV)
        h_t, out = buf_in[shift:shift + B * H].view(B, H), buf_out[shift:shift + B * H].view(B, H)
        h_t.copy_(torch.from_numpy(h_in))
        lp = torch.zeros((B, 1), device=DEV)
        rn.rnnlm_step(m, torch.from_numpy(prev).to(DEV), h_t, torch.from_numpy(query).to(DEV), out, lp)
        assert torch.isfinite(out).all() and torch.isnan(buf_out[B * H + shift:]).all()
        assert np.max(np.abs(out.cpu().numpy()[rows] - ref["h_out"])) <= tol_h
        assert np.max(np.abs(lp.cpu().numpy()[rows] - ref["logprob"])) <= tol_lp
    # the same rows through ids, a third of them distinct
    src = rng.integers(0, max(1, B // 3), B)
    res = gpu_step_dedup(m, src.astype(np.uint64) * 77 + 1, prev[src], h_in[src], query)
    u, rep, _ = oracle.dedup(src.astype(np.uint64) * 77 + 1)
    assert res["n_unique"] == u
    some = np.unique(np.linspace(0, u - 1, 50).astype(int))
    ref = oracle.step(model, prev[src][rep][some], h_in[src][rep][some], query[:len(some)])
    assert np.max(np.abs(res["h_out"][some] - ref["h_out"])) <= tol_h
    assert m.last_error() == 0
    m.close()


@pytest.mark.parametrize("H,B", [(64, 7), (77, 40), (256, 300), (1022, 513)])
def test_fp32_inputs_beyond_a_16_bit_term(H, B):
    """fp32 models: infinities, and finite numbers that round to one in bf16, in h_in and W saturate the units they reach
    (one such term per sum, so the sign is certain), in any position of the row."""
    rng = np.random.default_rng(H + B)
    model = model_of(rng, H, "f32")
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    query = rng.integers(0, V, (B, 2)).astype(np.int32)
    big = np.finfo(np.float32).max
    rows = np.unique(np.linspace(0, B - 1, 7).astype(int))
    for i, r in enumerate(rows):
        h_in[r, (0, H - 1, H // 2, 3, 1, 5, 0)[i]] = (np.inf, -np.inf, -np.inf, big, -big, np.float32(3.395e38), -big)[i]
    model["W"][2, 7] = np.inf                                  # 7: no row above has its large element there
    h_in[:, 7] = 0.75
    a = model["U"][prev].astype(np.float64)
    with np.errstate(over="ignore"):
        # no sum holds two infinities of different sign but unit 2's, where W is infinite too: left out of the check
        a += np.einsum("bi,ji->bj", h_in.astype(np.float64), model["W"].astype(np.float64))
        ref = 1.0 / (1.0 + np.exp(-a))
    keep = np.ones((B, H), bool)
    keep[rows, 2] = False
    assert np.isfinite(ref[keep]).all()
    m = load_model(model, "f32", B)
    for grouped in (False, True):
        if grouped:
            res = gpu_step_dedup(m, np.arange(B, dtype=np.uint64) * 3 + 5, prev, h_in, query)
            h_out, lp = res["h_out"], res["logprob"]
        else:
            h_out, lp = gpu_step(m, prev, h_in, query)
        assert np.max(np.abs(h_out[keep] - ref[keep])) <= 2e-6              # as above
        # the normaliser of a row whose units are all known: the vectors handed out, in 64 bits
        known = np.isfinite(h_out).all(1)
        assert known.sum() >= B - len(rows)
        z = h_out.astype(np.float64) @ model["O"].astype(np.float64)
        want = np.take_along_axis(z, query.astype(np.int64), 1) - np.log(np.exp(z).sum(1))[:, None]
        assert np.max(np.abs(lp[known] - want[known])) <= 1e-5
    assert m.last_error() == 0
    m.close()


@pytest.mark.parametrize("H,B", [(63, 7), (77, 20), (100, 32), (77, 40), (130, 9), (250, 70), (300, 12), (1022, 5)])
def test_fp32_rows_with_an_infinity_and_padded_units(H, B):
    """An infinity in h_in, which the zero weights of units beyond H meet as well: every unit of the row saturates, and
    its log-probabilities are those of the saturated units, grouped and not."""
    rng = np.random.default_rng(H * B)
    model = model_of(rng, H, "f32")
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    query = rng.integers(0, V, (B, 3)).astype(np.int32)
    rows = np.unique(np.linspace(0, B - 1, 5).astype(int))
    for i, r in enumerate(rows):
        h_in[r, (0, H - 1, H // 2, 3, 1)[i]] = (np.inf, -np.inf, -np.inf, np.inf, -np.inf)[i]
    a = model["U"][prev].astype(np.float64) + np.einsum("bi,ji->bj", h_in.astype(np.float64), model["W"].astype(np.float64))
    with np.errstate(over="ignore"):
        h_ref = 1.0 / (1.0 + np.exp(-a))
    z = h_ref @ model["O"].astype(np.float64)
    want = np.take_along_axis(z, query.astype(np.int64), 1) - np.log(np.exp(z).sum(1))[:, None]
    m = load_model(model, "f32", B)
    for grouped in (False, True):
        if grouped:
            res = gpu_step_dedup(m, np.arange(B, dtype=np.uint64) * 3 + 5, prev, h_in, query)
            h_out, lp = res["h_out"], res["logprob"]
        else:
            h_out, lp = gpu_step(m, prev, h_in, query)
        # as in test_against_the_oracle
        assert np.max(np.abs(h_out - h_ref)) <= 2e-6 and np.max(np.abs(lp - want)) <= 1e-5, grouped
    assert m.last_error() == 0
    m.close()
