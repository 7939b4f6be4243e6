"""Host-side checks of the index arithmetic and of the splits of fp32 operands the HIP kernels rely on.

Nothing here touches the GPU or the oracle: the formulas are restated in numpy and checked for
the properties the kernels need (bijections, bank spreading, exactness of the split and the size
of what it drops).  A kernel that used another formula would fail its parity test; these tests
say WHY the formulas are safe to use."""
import numpy as np
import pytest

from workloads import round_to_bf16


# ------------------------------------------------------------------ LDS rows: bank spreading
# A ds_read_b128 serves 16 lanes together; they read the same logical 16-byte piece c of 16
# consecutive rows.  LDS has 64 banks of 4 bytes = 16 groups of 16 bytes: the 16 reads must fall in
# 16 different groups.  Physical piece index of (row, c):
LAYOUTS = {
    "128-byte rows, c ^ ((r >> 1) & 7)": (8, lambda r, c: c ^ ((r >> 1) & 7)),          # tiled kernels
    "128-byte rows of 1 KB words, c ^ (r & 15)": (64, lambda r, c: c ^ (r & 15)),       # staged kernel (Hp = 512)
}


@pytest.mark.parametrize("name", list(LAYOUTS))
def test_lds_row_layout_is_a_bijection_and_conflict_free(name):
    pieces, pos = LAYOUTS[name]
    swizzled = min(pieces, 16)          # only the low bits of the piece index take part
    for r in range(64):
        assert sorted(pos(r, c) for c in range(swizzled)) == list(range(swizzled)), (name, r)
    for base in range(0, 64, 16):
        for c in range(swizzled):
            groups = {(pieces * r + pos(r, c)) % 16 for r in range(base, base + 16)}
            assert len(groups) == 16, (name, base, c)


def test_direct_load_side_inverts_the_rotation():
    """The direct global->LDS loads write LDS linearly, so lane i must fetch the logical piece that
    belongs at physical position i: the inverse map used by the loaders."""
    for r in range(64):
        for p in range(8):
            c = p ^ ((r >> 1) & 7)
            assert c ^ ((r >> 1) & 7) == p


# ------------------------------------------------------------------ MFMA-operand ("fragment") order
def frag_index(row, unit, KS):
    """Element index of (row, unit) in [rows / 32][KS][64 lanes][8]: lane 32 g + c of fragment
    (rb, ks) holds row 32 rb + c, units 16 ks + 8 g .. + 7."""
    rb, c = divmod(row, 32)
    ks, rest = divmod(unit, 16)
    g, e = divmod(rest, 8)
    return ((rb * KS + ks) * 64 + 32 * g + c) * 8 + e


@pytest.mark.parametrize("rows,H", [(32, 64), (64, 128), (96, 512)])
def test_fragment_order_is_a_bijection(rows, H):
    KS = H // 16
    idx = np.array([[frag_index(r, u, KS) for u in range(H)] for r in range(rows)])
    assert sorted(idx.ravel().tolist()) == list(range(rows * H))
    # one operand of a wave (fixed row block and k-step) is 1 KB contiguous
    block = idx[:32, :16].ravel()
    assert block.min() == 0 and block.max() == 511


def test_two_term_fragment_order_is_a_bijection():
    """fp32 models, [row block][k-step][term][64 lanes][8]: the two terms of an operand are 2 KB contiguous."""
    H, rows = 128, 64
    KS = H // 16
    idx = [frag_index(r, u, KS) // 512 * 1024 + t * 512 + frag_index(r, u, KS) % 512
           for r in range(rows) for u in range(H) for t in range(2)]
    assert sorted(idx) == list(range(2 * rows * H))


# ------------------------------------------------------------------ two-term fp16 split (output projection)
def split2(x):
    """Values below 2^15 in magnitude, as the kernels scale them."""
    x1 = x.astype(np.float32).astype(np.float16)
    return x1, (x - x1.astype(np.float32)).astype(np.float16)


def scaled_words(O):
    """Every word's weights times the power of two that brings its largest into [2^13, 2^14)."""
    e = np.frexp(np.abs(O).max(0))[1]
    return np.ldexp(O, 14 - e).astype(np.float32)


def test_two_fp16_terms_miss_the_fp32_number_by_one_unit_in_its_last_place_at_most():
    # (or by half of the smallest fp16 step, 2^-24, where that is more)
    rng = np.random.default_rng(8)
    x = np.concatenate([rng.uniform(2.0 ** -3, 2.0 ** 14, 50000), np.exp2(rng.uniform(-3, 14, 50000)),
                        np.array([0.0, 2.0 ** 13, 2.0 ** 14 - 2.0 ** -10])]).astype(np.float32)
    x1, x2 = split2(x)
    off = np.abs(x1.astype(np.float64) + x2.astype(np.float64) - x)
    unit = np.exp2(np.floor(np.log2(np.maximum(x, 1e-30))) - 23)
    assert np.all(off <= np.maximum(unit, 2.0 ** -25)) and 0.1 < np.mean(off > 0) < 0.3
    # centred hidden values above one half of a unit's range are exact
    h = (rng.integers(2 ** 22, 2 ** 24, 50000) / 2.0 ** 24).astype(np.float32)
    d = (h - np.float32(0.5)) * np.float32(2.0 ** 14)
    d1, d2 = split2(d)
    assert np.array_equal(d1.astype(np.float64) + d2.astype(np.float64), d.astype(np.float64))


@pytest.mark.parametrize("big", [1.0, 100.0, 1e5])
def test_the_three_kept_products_of_the_fp16_split(big):
    """One weight of every word `big` times the others: a product of weights not far below the word's largest is off by
    2^-21 of itself at most, any other by what the second term's smallest step leaves, 2^-38 of the largest weight."""
    rng = np.random.default_rng(9)
    O = rng.normal(0, 0.2, (64, 500)).astype(np.float32)
    O[rng.integers(0, 64, 500), np.arange(500)] *= np.float32(big)
    w = scaled_words(O)
    d = ((rng.uniform(0, 1, 64).astype(np.float32) - np.float32(0.5)) * np.float32(2.0 ** 14))[:, None]
    w1, w2 = (t.astype(np.float64) for t in split2(w))
    d1, d2 = (t.astype(np.float64) for t in split2(d))
    kept = w1 * d1 + w1 * d2 + w2 * d1
    exact = w.astype(np.float64) * d.astype(np.float64)
    assert np.all(np.abs(kept - exact) <= 2.0 ** -21 * np.abs(exact) + 2.0 ** -25 * (np.abs(w) + np.abs(d)) * 1.01 + 2.0 ** -40)


# ------------------------------------------------------------------ three-term bf16 split (hidden update)
def split3(x):
    x = x.astype(np.float32)
    x1 = round_to_bf16(x)
    r1 = (x - x1).astype(np.float32)
    x2 = round_to_bf16(r1)
    r2 = (r1 - x2).astype(np.float32)
    x3 = round_to_bf16(r2)
    return x1, x2, x3


def test_three_bf16_terms_add_up_to_the_fp32_number_exactly():
    rng = np.random.default_rng(5)
    x = np.concatenate([rng.normal(0, 1, 20000), rng.normal(0, 1e-3, 20000), rng.uniform(-0.5, 0.5, 20000),
                        np.array([0.0, 1.0, -1.0, 0.5, 2.0 ** -20, 1.0 + 2.0 ** -23, 1e30, 1.2e-30])]).astype(np.float32)
    # (holds up to the largest finite bf16; a number that rounds to infinity as bf16 is no weight)
    x1, x2, x3 = split3(x)
    total = x1.astype(np.float64) + x2.astype(np.float64) + x3.astype(np.float64)
    assert np.array_equal(total, x.astype(np.float64))
    # each term is at most half a unit in the last place of the one before it
    big = np.abs(x) > 1e-30
    assert np.all(np.abs(x2[big]) <= np.abs(x1[big]) * 2.0 ** -8)
    assert np.all(np.abs(x3[big]) <= np.abs(x1[big]) * 2.0 ** -16)


def test_the_six_kept_cross_terms_leave_less_than_three_ulp_of_bf16_cubed():
    """(w1 + w2 + w3)(d1 + d2 + d3) minus the six kept products = w2 d3 + w3 d2 + w3 d3, each at
    most 2^-24 |w1 d1|: the sum of the kept products is within 3 * 2^-24 of the fp32 product,
    relative, before any accumulation error."""
    rng = np.random.default_rng(6)
    w = rng.normal(0, 0.05, 50000).astype(np.float32)
    d = rng.uniform(-0.5, 0.5, 50000).astype(np.float32)
    w1, w2, w3 = (t.astype(np.float64) for t in split3(w))
    d1, d2, d3 = (t.astype(np.float64) for t in split3(d))
    kept = w1 * d1 + w1 * d2 + w2 * d1 + w1 * d3 + w3 * d1 + w2 * d2
    exact = w.astype(np.float64) * d.astype(np.float64)
    ok = np.abs(exact) > 1e-12
    assert np.max(np.abs(kept - exact)[ok] / np.abs(exact)[ok]) <= 3 * 2.0 ** -24
