"""Two-term fp16 form of the fp32 output projection, against the oracle: edges of its row and word tiles, both tile
shapes, both forms of the log-sum-exp, and words whose weights lie many powers of two apart (every word is brought into
the range of fp16 by a power of two of its own)."""
import numpy as np
import pytest

import oracle
import paper_2007_11794_amd as rn

from harness import gpu_step, gpu_step_dedup, load_model

pytestmark = pytest.mark.gpu


def model_of(rng, V, H, big):
    O = rng.normal(0, big, (H, V))
    O *= 2.0 ** rng.integers(-30, 1, (H, V))               # a wide range inside every word
    O[:, ::5] *= 1e-6
    O[:, 1::7] *= 1e-30
    O[:, 2::11] = 0.0
    O[:, 3::13] *= 1e-40                                   # denormal or zero as fp32
    sigma = 0.4 / np.sqrt(H)
    return {"U": rng.normal(0, 0.3, (V, H)).astype(np.float32), "W": rng.normal(0, sigma, (H, H)).astype(np.float32),
            "O": O.astype(np.float32), "bias": rng.normal(0, 0.5, V).astype(np.float32)}


# 64-word granularity of the tiles (256 words from 1024 tiles of 256 x 128 on), rows around 64 and 128
@pytest.mark.parametrize("V,H,B,big", [(2, 64, 1, 1.0), (255, 65, 63, 1.0), (257, 128, 64, 1.0), (511, 64, 65, 4.0),
                                       (513, 200, 127, 1.0), (1000, 64, 128, 4.0), (700, 576, 129, 0.5),
                                       (33000, 64, 1000, 1.0), (66000, 32, 449, 4.0), (4100, 1030, 140, 0.5)])
def test_against_the_oracle(V, H, B, big):
    rng = np.random.default_rng(V + B)
    model = model_of(rng, V, H, big)
    m = load_model(model, "f32", B)
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    query = rng.integers(0, V, (B, 3)).astype(np.int32)
    ref = oracle.step(model, prev, h_in, query)
    # fp32 sums of H products: 2^-24 of the running sum per addition at worst, running sums below the sum of |O| / 2
    tol = 1e-5 + 2.0 ** -24 * np.sqrt(H) * 0.5 * np.abs(model["O"]).sum(0).max()
    for lse_mode in (0, 1):
        m.set_option(rn.OPT_LSE_MODE, lse_mode)
        for kernel in (0, 4, 5):
            m.set_option(rn.OPT_OUTPROJ_KERNEL, kernel)
            h, lp = gpu_step(m, prev, h_in, query)
            assert np.max(np.abs(h - ref["h_out"])) <= 1e-5
            assert np.max(np.abs(lp - ref["logprob"])) <= tol, (kernel, lse_mode)
    # few of the rows distinct: the row count is then known on the device only
    m.set_option(rn.OPT_OUTPROJ_KERNEL, 4)
    src = rng.integers(0, max(1, B // 9), B)
    out = gpu_step_dedup(m, src.astype(np.uint64) + 5, prev[src], h_in[src], query)
    ref = oracle.step(model, prev[src], h_in[src], query)
    assert np.max(np.abs(out["logprob"] - ref["logprob"])) <= tol
    assert m.last_error() == 0
    m.close()


@pytest.mark.parametrize("V,H,B", [(300, 1000, 8), (300, 1000, 33), (700, 128, 20), (700, 128, 130)])
def test_a_word_masked_by_an_infinite_weight(V, H, B):
    """A word with a weight of -inf on a unit that is above one half in every row has probability 0; the others keep theirs."""
    rng = np.random.default_rng(V + H + B)
    model = model_of(rng, V, H, 1.0)
    model["U"][:, 3] = 9.0                                   # h' of unit 3 is close to 1
    model["O"][3, 17] = -np.inf
    m = load_model(model, "f32", B)
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    query = rng.integers(18, V, (B, 3)).astype(np.int32)
    query[:, 2] = 17
    h, lp = gpu_step(m, prev, h_in, query)
    others = np.delete(np.arange(V), 17)
    z = h.astype(np.float64) @ model["O"][:, others].astype(np.float64) + model["bias"][others]
    full = np.zeros((B, V))
    full[:, others] = z - np.log(np.exp(z).sum(1))[:, None]
    tol = 1e-5 + 2.0 ** -24 * np.sqrt(H) * 0.5 * np.abs(model["O"][:, others]).sum(0).max()      # as above
    assert np.max(np.abs(lp[:, :2] - np.take_along_axis(full, query[:, :2].astype(np.int64), 1))) <= tol
    assert np.all(lp[:, 2] == -np.inf)
    m.close()


# The tiles (on request where the rows fit the registers): both terms of 64 and of 32 rows in LDS, one term of 32 rows, neither; rows
# around what each takes; a vocabulary of fewer blocks of 32 words than there are workgroups, one with a remainder
@pytest.mark.parametrize("V,H,N,unique", [(300, 64, 300, 1), (9000, 256, 1024, 64), (9000, 256, 1024, 65), (20011, 320, 513, 32),
                                          (20011, 320, 513, 33), (9000, 576, 300, 31), (9000, 640, 300, 32), (9000, 832, 300, 20),
                                          (9000, 832, 300, 40), (3000, 1024, 300, 9), (66000, 900, 513, 32), (3000, 1300, 300, 9)])
def test_few_rows_known_on_the_device_only(V, H, N, unique):
    rng = np.random.default_rng(V + H + unique)
    model = model_of(rng, V, H, 1.0)
    m = load_model(model, "f32", N)
    src = np.concatenate([np.arange(unique), rng.integers(0, unique, N - unique)])
    prev, h_in = rng.integers(0, V, unique).astype(np.int32)[src], rng.uniform(0, 1, (unique, H)).astype(np.float32)[src]
    query = rng.integers(0, V, (N, 2)).astype(np.int32)
    ref = oracle.step(model, prev[:unique], h_in[:unique], query, row_of_query=src.astype(np.int32))
    tol = 1e-5 + 2.0 ** -24 * np.sqrt(H) * 0.5 * np.abs(model["O"]).sum(0).max()                 # as above
    for kernel in (0, 4):
        m.set_option(rn.OPT_OUTPROJ_KERNEL, kernel)
        in_registers = kernel == 0 and 64 < H <= 576
        assert m.outproj_kernel_name(N) == ("outproj_staged_f32_kernel" if in_registers else "outproj_split2_kernel")
        for lse_mode in (0, 1):
            m.set_option(rn.OPT_LSE_MODE, lse_mode)
            out = gpu_step_dedup(m, src.astype(np.uint64) + 5, prev, h_in, query)
            assert out["n_unique"] == unique and np.max(np.abs(out["logprob"] - ref["logprob"])) <= tol
    assert m.last_error() == 0
    m.close()


@pytest.mark.parametrize("V", [2, 300, 1100])
def test_more_row_groups_than_workgroups(V):
    """Workgroups take several row groups, of vocabulary splits that hold no word at all where there are few (64 units: the tiles)."""
    H, B = 64, 9000
    rng = np.random.default_rng(V)
    model = model_of(rng, V, H, 1.0)
    m = load_model(model, "f32", B)
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    query = rng.integers(0, V, (B, 1)).astype(np.int32)
    ref = oracle.step(model, prev, h_in, query)
    tol = 1e-5 + 2.0 ** -24 * np.sqrt(H) * 0.5 * np.abs(model["O"]).sum(0).max()                 # as above
    for lse_mode in (0, 1):
        m.set_option(rn.OPT_LSE_MODE, lse_mode)
        assert np.max(np.abs(gpu_step(m, prev, h_in, query)[1] - ref["logprob"])) <= tol
    m.close()


@pytest.mark.parametrize("V,H,B", [(600, 64, 20), (600, 64, 130), (600, 700, 30), (600, 700, 130), (66000, 64, 513)])
def test_words_with_one_dominant_weight(V, H, B):
    """One weight of every word a hundred times the others: a logit is then one product, whose split cannot hide behind the
    roundings of many."""
    rng = np.random.default_rng(V + H + B)
    O = rng.normal(0, 0.2, (H, V))
    O[rng.integers(0, H, V), np.arange(V)] *= 100.0
    model = {"U": rng.normal(0, 0.3, (V, H)).astype(np.float32), "W": rng.normal(0, 0.4 / np.sqrt(H), (H, H)).astype(np.float32),
             "O": O.astype(np.float32), "bias": rng.normal(0, 0.5, V).astype(np.float32)}
    m = load_model(model, "f32", B)
    prev, h_in = rng.integers(0, V, B).astype(np.int32), rng.uniform(0, 1, (B, H)).astype(np.float32)
    query = rng.integers(0, V, (B, 3)).astype(np.int32)
    for kernel in (0, 1, 4):
        m.set_option(rn.OPT_OUTPROJ_KERNEL, kernel)
        h, lp = gpu_step(m, prev, h_in, query)
        # the normaliser of the vector handed out, in 64 bits
        z = h.astype(np.float64) @ model["O"].astype(np.float64) + model["bias"]
        top = z.max(1, keepdims=True)
        want = np.take_along_axis(z, query.astype(np.int64), 1) - (top + np.log(np.exp(z - top).sum(1, keepdims=True)))
        # 2^-21 of a word's products, and one rounding of 2^-24 of the running sum per matrix instruction (three per 16
        # units) or product; the same for the word asked, in plain fp32; constants and results of the size of the logits
        size = 0.5 * np.abs(model["O"]).sum(0).max()
        tol = (2.0 ** -21 + (3 * (H // 16 + 1) + 64) * 2.0 ** -24) * size
        assert np.max(np.abs(lp - want)) <= tol, kernel
        assert np.sqrt(np.mean((lp - want) ** 2)) <= 2.0 ** -21 * size            # roundings do not all add up
    m.close()
